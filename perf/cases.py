"""The work that programs around an FX correlator give this library, as cases
that can be timed: each is a call (or the few calls of one integration)
through the public entry points of ``paper_2406_19013_amd.xcorr``.

A case is a dict of plain values; its ``op`` says which entry points it runs:

* ``corr``    one integration held in one buffer: ``Correlator.ingest_dump``
              (4+4-bit int8 MFMA), or the 8+8-bit int8 and FP16 paths;
* ``blocks``  an integration of several device blocks handed over together:
              ``Correlator.ingest_blocks`` and ``Correlator.dump``;
* ``pipe``    the streaming loop: ``Pipe.push`` of device blocks, one launch
              per block, with the dump on the last one;
* ``batch``   several arrays of uneven size in one ``Batch.ingest``, then one
              dump per array;
* ``fengine`` raw ADC codes to packed 4+4-bit channels: ``xcorr_fengine``;
* ``stokes``  a dump to full-Stokes visibilities: ``xcorr_stokes``.

Ranges: 2 to 512 inputs (even and odd counts), 1 to 4096 channels, 32 to 8192
samples per channel (8 to 4096 spectra for the front end).
"""
import math

import torch

from paper_2406_19013_amd import synth
from paper_2406_19013_amd import xcorr as X

PATHS = {"i8": (4, X.PATH_I8_MFMA), "i8x8": (8, X.PATH_I8_MFMA), "f16x8": (8, X.PATH_F16_MFMA)}
TONE = synth.Tone(amp=2.5, delta=0.01)
FE_TONES = (synth.AdcTone(freq=300.0 / 2048, amp=12.0), synth.AdcTone(freq=700.5 / 2048, amp=8.0))


def listed():
    return [
        # the smallest call: 8 dual-polarisation feeds, a few channels; the
        # launch and the host path are all of it
        {"name": "tiny_16x8x256", "op": "corr", "path": "i8", "N": 16, "F": 8, "T": 256},
        # one instance of the X-engine node: 192 inputs x 32 channels
        {"name": "instance_192x32x4096", "op": "corr", "path": "i8", "N": 192, "F": 32, "T": 4096},
        # the whole band of the 192-input array, 33.55 ms of sky
        {"name": "band_192x1024x4096", "op": "corr", "path": "i8", "N": 192, "F": 1024, "T": 4096},
        # an array whose input count is no multiple of 16, ragged sample count
        {"name": "odd_100x512x1000", "op": "corr", "path": "i8", "N": 100, "F": 512, "T": 1000},
        # an array wider than one triangle
        {"name": "wide_512x512x2048", "op": "corr", "path": "i8", "N": 512, "F": 512, "T": 2048},
        # unpacked samples: exact int8 and FP16 with FP32 accumulation
        {"name": "fluffed_i8_192x512x8192", "op": "corr", "path": "i8x8", "N": 192, "F": 512, "T": 8192},
        {"name": "fluffed_f16_192x512x8192", "op": "corr", "path": "f16x8", "N": 192, "F": 512, "T": 8192},
        # 1024-sample blocks of a 96-input array, eight to an integration
        {"name": "blocks_96x2048x1024", "op": "blocks", "N": 96, "F": 2048, "T": 1024, "blocks": 8},
        # the streaming loop of the 192-input array, 4096 channels
        {"name": "stream_192x4096x1024", "op": "pipe", "N": 192, "F": 4096, "T": 1024, "blocks": 4},
        # four arrays of uneven input and channel counts in one launch
        {"name": "batch_4_arrays", "op": "batch", "N": 64, "F": 256, "N2": 192, "F2": 1024, "N3": 256, "F3": 512,
         "N4": 512, "F4": 128, "T": 2048},
        # the front end of the 192-input array, 33.55 ms of samples
        {"name": "fengine_192x4096", "op": "fengine", "N": 192, "T": 4096},
        # full Stokes of the whole band's dump
        {"name": "stokes_192x1024", "op": "stokes", "N": 192, "F": 1024},
    ]


def _log(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _inputs(rng, lo=2, hi=512):
    """Half the arrays have a multiple of 16 inputs, the rest any number."""
    n = _log(rng, lo, hi)
    return max(16, n // 16 * 16) if rng.random() < 0.5 else n


def draw(rng):
    op = rng.choice(["corr", "corr", "corr", "corr", "blocks", "pipe", "batch", "fengine", "stokes"])
    if op == "fengine":
        return {"op": op, "N": 16 * rng.randint(1, 12), "T": _log(rng, 8, 4096)}
    if op == "stokes":
        return {"op": op, "N": 2 * _log(rng, 2, 128), "F": _log(rng, 1, 1024)}
    if op == "batch":
        return {"op": op, "N": 16 * rng.randint(1, 12), "F": _log(rng, 4, 1024), "N2": 16 * rng.randint(1, 24),
                "F2": _log(rng, 4, 512), "T": _log(rng, 64, 2048)}
    if op in ("blocks", "pipe"):
        c = {"op": op, "N": _inputs(rng, 8, 256), "F": _log(rng, 4, 2048), "T": 64 * _log(rng, 1, 16),
             "blocks": rng.randint(2, 8)}
        if rng.random() < 0.25:
            c["T"] = max(32, c["T"] - rng.randint(1, 31))
    else:
        c = {"op": op, "path": rng.choice(["i8", "i8", "i8", "i8x8", "f16x8"]), "N": _inputs(rng),
             "F": _log(rng, 1, 4096), "T": _log(rng, 32, 8192)}
    while not _fits(c):
        c["F"] = max(1, c["F"] // 2)
    return c


def _fits(c):
    """No drawn case costs more than the largest listed ones."""
    w = work(c)
    return w["bytes"] <= 1.5e9 and w["flops"] <= 6e11


def _arrays(c):
    return [(c["N" + k], c["F" + k]) for k in ("", "2", "3", "4") if "N" + k in c]


def _volts(c, seed, a=0, N=None, F=None, block=0):
    N, F = N or c["N"], F or c["F"]
    bits = PATHS[c.get("path", "i8")][0]
    return synth.gaussian_volts(N, F, c["T"], sigma=2.5 if bits == 4 else 20.0, bits=bits, seed=(seed, a),
                                tone=TONE if bits == 4 else None, block=block, t0=block * c["T"], device="cuda")


def _vis(N, F, dtype=torch.int32):
    return torch.empty((F, N * (N + 1) // 2, 2), dtype=dtype, device="cuda")


def prepare(case, seed):
    c = case
    op = c["op"]
    st = {"case": c}
    if op == "corr":
        bits, path = PATHS[c["path"]]
        st["cor"] = X.Correlator(c["N"], c["F"], bits, path)
        st["volts"] = _volts(c, seed)
        st["out"] = _vis(c["N"], c["F"], torch.float32 if path == X.PATH_F16_MFMA else torch.int32)
    elif op in ("blocks", "pipe"):
        st["cor"] = X.Correlator(c["N"], c["F"])
        st["volts"] = [_volts(c, seed, block=b) for b in range(c["blocks"])]
        st["out"] = _vis(c["N"], c["F"])
        if op == "pipe":
            st["pipe"] = X.Pipe(st["cor"], c["T"], c["blocks"], host_blocks=False)
    elif op == "batch":
        st["cors"] = [X.Correlator(N, F) for N, F in _arrays(c)]
        st["batch"] = X.Batch(st["cors"])
        st["volts"] = [_volts(c, seed, a, N, F) for a, (N, F) in enumerate(_arrays(c))]
        st["outs"] = [_vis(N, F) for N, F in _arrays(c)]
    elif op == "fengine":
        N, T = c["N"], c["T"]
        st["adc"] = synth.adc_samples(N, (T + 3) * 2048, sigma=synth.FE_ADC_SIGMA, seed=(seed, 6), tones=FE_TONES,
                                      device="cuda")
        st["gains"] = synth.eq_gains(N, 1024, base=synth.FE_EQ_BASE, seed=(seed, 7), device="cuda")
        st["h"] = torch.from_numpy(X.xcorr_pfb_prototype()).cuda()
        st["out"] = torch.empty((T, 1024, N), dtype=torch.uint8, device="cuda")
    else:
        # a dump of about 4096 samples: integer visibilities with the powers
        # of such an integration
        g = torch.Generator(device="cuda")
        g.manual_seed(synth.seed_of(seed, 8))
        N, F = c["N"], c["F"]
        P = N * (N + 1) // 2
        st["vis"] = torch.empty((F, P, 2), dtype=torch.int32, device="cuda")
        for f in range(0, F, 64):
            n = min(64, F - f)
            st["vis"][f:f + n] = (torch.randn((n, P, 2), generator=g, device="cuda") * 26000.0).to(torch.int32)
        st["out"] = torch.empty((F, (N // 2) * (N // 2 + 1) // 2, 4, 2), dtype=torch.int64, device="cuda")
    return st


def run(state):
    c = state["case"]
    op = c["op"]
    if op == "corr":
        out, _, _ = state["cor"].ingest_dump(state["volts"], state["out"])
        return out
    if op == "blocks":
        state["cor"].ingest_blocks(state["volts"])
        out, _, _ = state["cor"].dump(state["out"])
        return out
    if op == "pipe":
        last = c["blocks"] - 1
        for b, v in enumerate(state["volts"]):
            state["pipe"].push(v, state["out"] if b == last else None)
        return state["out"]
    if op == "batch":
        state["batch"].ingest(state["volts"])
        for cor, out in zip(state["cors"], state["outs"]):
            cor.dump(out)
        return state["outs"]
    if op == "fengine":
        X.xcorr_fengine(state["adc"], state["h"], state["gains"], state["out"])
        return state["out"]
    return X.xcorr_stokes(state["vis"], c["N"], state["out"])


def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: 8 per
    (pair, channel, sample); for the front end the filter, the real FFT by
    the usual count and the EQ."""
    c = case
    op = c["op"]

    def pairs(N):
        return N * (N + 1) // 2

    if op == "fengine":
        n = c["N"] * c["T"]
        return {"bytes": c["N"] * (c["T"] + 3) * 2048 + n * 1024 + c["N"] * 4096 + 32768,
                "flops": n * (8 * 2048 + 2.5 * 2048 * 11 + 2 * 1024)}
    if op == "stokes":
        return {"bytes": c["F"] * (pairs(c["N"]) * 8 + pairs(c["N"] // 2) * 64), "flops": c["F"] * pairs(c["N"] // 2) * 8}
    per_sample = PATHS[c.get("path", "i8")][0] // 4
    T = c["T"] * c.get("blocks", 1)
    return {"bytes": sum(N * F * T * per_sample + F * pairs(N) * 8 for N, F in _arrays(c)),
            "flops": sum(8 * F * pairs(N) * T for N, F in _arrays(c))}


def _correlate64(blocks, N, F, bits):
    """Visibilities [F][P][2] in float64 from the blocks [T][F][N](2)."""
    i, j = torch.tril_indices(N, N, device="cuda")
    out = torch.zeros((F, N * (N + 1) // 2, 2), dtype=torch.float64, device="cuda")
    for v in blocks:
        step = max(1, int(2e8 // (v.shape[0] * N)))
        for f in range(0, F, step):
            x = v[:, f:f + step]
            if bits == 4:
                re, im = synth.unpack4(x)
            else:
                re, im = x[..., 0], x[..., 1]
            re = re.to(torch.float64).permute(1, 2, 0).contiguous()
            im = im.to(torch.float64).permute(1, 2, 0).contiguous()
            ret, imt = re.transpose(1, 2).contiguous(), im.transpose(1, 2).contiguous()
            out[f:f + step, :, 0] += (torch.bmm(re, ret) + torch.bmm(im, imt))[:, i, j]
            out[f:f + step, :, 1] += (torch.bmm(im, ret) - torch.bmm(re, imt))[:, i, j]
    return out


def _fengine64(st, N, T):
    """Packed codes [T][1024][N] of the filter bank in float64."""
    h = st["h"].to(torch.float64).view(4, 2048)
    out = torch.empty((T, 1024, N), dtype=torch.uint8, device="cuda")
    for i in range(N):
        x = st["adc"][i].to(torch.float64).view(T + 3, 2048)
        y = sum(h[k] * x[k:k + T] for k in range(4))
        s = torch.fft.rfft(y, dim=1)[:, :1024] * st["gains"][i].to(torch.float64)
        out[:, :, i] = synth.pack4(torch.clamp(torch.round(s.real), -8, 7), torch.clamp(torch.round(s.imag), -8, 7))
    return out


def exact(case, seed):
    c = case
    op = c["op"]
    st = prepare(c, seed)
    if op == "corr":
        v = _correlate64([st["volts"]], c["N"], c["F"], PATHS[c["path"]][0])
        return v if c["path"] == "f16x8" else v.to(torch.int32)
    if op in ("blocks", "pipe"):
        return _correlate64(st["volts"], c["N"], c["F"], 4).to(torch.int32)
    if op == "batch":
        return [_correlate64([v], N, F, 4).to(torch.int32) for v, (N, F) in zip(st["volts"], _arrays(c))]
    if op == "fengine":
        return _fengine64(st, c["N"], c["T"])
    N, F = c["N"], c["F"]
    nf = N // 2
    a, b = torch.tril_indices(nf, nf, device="cuda")
    vis = st["vis"].to(torch.int64)

    def at(i, j):
        return vis[:, i * (i + 1) // 2 + j]

    xx, yy, yx = at(2 * a, 2 * b), at(2 * a + 1, 2 * b + 1), at(2 * a + 1, 2 * b)
    conj = torch.tensor([1, -1], dtype=torch.int64, device="cuda")
    same = (a == b)[None, :, None]
    # V(2a, 2b + 1) lies above the diagonal for a = b: there it is conj V(2a + 1, 2a)
    xy = torch.where(same, yx * conj, at(2 * a, torch.where(a == b, 2 * b, 2 * b + 1)))
    d = xy - yx
    return torch.stack([xx + yy, xx - yy, xy + yx, torch.stack([d[..., 1], -d[..., 0]], dim=-1)], dim=2)
