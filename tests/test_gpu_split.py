"""The time-split 4+4-bit kernel (few channels, rows off the 16-byte
boundaries) and the persistent kernel on rows that start on 4-byte boundaries
only: exact parity, against the oracle where it is quick and against the plain
path (itself checked against the oracle elsewhere) on the larger outputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2406_19013_amd import synth
from paper_2406_19013_amd import xcorr as X

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)


def _at(v, offset):
    """A copy of v on the GPU whose first byte lies `offset` bytes past a
    256-byte boundary, at the very end of its allocation."""
    raw = torch.empty(v.numel() + offset, dtype=torch.uint8, device="cuda")
    raw[offset:] = v.reshape(-1).cuda()
    return raw[offset:].view(v.shape)


def _run(v, N, F, splits, path=X.PATH_I8_MFMA):
    c = X.Correlator(N, F, 4, path)
    t0 = 0
    for n in splits:
        c.ingest(v[t0:t0 + n], n)
        t0 += n
    out, n, _ = c.dump()
    torch.cuda.synchronize()
    assert n == sum(splits)
    c.close()
    return out


# inputs around the 32-input block and the 64-input region, by alignment of
# the rows; samples around the 32-sample step and the 8 waves' first round
SHAPES = [(n, f) for n in (4, 32, 64, 68, 100, 192, 260) for f in (1, 3)] + \
         [(n, f) for n in (1, 2, 31, 33, 66, 99, 130) for f in (1, 3)]


@pytest.mark.parametrize("T", [1, 31, 33, 256, 289])
@pytest.mark.parametrize("N,F", SHAPES, ids=[f"N{n}F{f}" for n, f in SHAPES])
def test_few_channels_exact(N, F, T):
    _say(f"split N={N} F={F} T={T}")
    v = synth.uniform_volts4(N, F, T, seed=(2101, N, F, T))
    want = oracle.to_int32(oracle.xcorr(v.numpy(), 4, T, F, N))
    assert np.array_equal(_run(_at(v, 0), N, F, [T]).cpu().numpy(), want)


@pytest.mark.parametrize("N,offset", [(n, o) for n in (33, 100, 192) for o in (1, 2, 4, 12)])
def test_any_start_address_and_running_sums(N, offset):
    """Inputs that start off the 16-byte boundaries and end with their
    allocation; the second and third ingest add to running sums."""
    F, splits = 3, [64, 7, 300]
    _say(f"split N={N} offset={offset}")
    v = synth.uniform_volts4(N, F, sum(splits), seed=(2102, N, offset))
    want = oracle.to_int32(oracle.xcorr(v.numpy(), 4, sum(splits), F, N))
    assert np.array_equal(_run(_at(v, offset), N, F, splits).cpu().numpy(), want)


@pytest.mark.parametrize("N", [4, 64, 100, 200])
def test_few_channel_blocks(N):
    """Block tables of the time-split kernel: several blocks to a launch,
    stored and accumulated."""
    F, B = 3, 128
    _say(f"split blocks N={N}")
    v = synth.uniform_volts4(N, F, 11 * B, seed=(2103, N))
    want = oracle.to_int32(oracle.xcorr(v.numpy(), 4, 11 * B, F, N))
    d = v.cuda()
    c = X.Correlator(N, F)
    c.ingest_blocks([d[b * B:(b + 1) * B].clone() for b in range(9)])
    c.ingest_blocks([d[b * B:(b + 1) * B].clone() for b in (9, 10)])
    out, n, _ = c.dump()
    torch.cuda.synchronize()
    c.close()
    assert n == 11 * B and np.array_equal(out.cpu().numpy(), want)


def test_extreme_samples_at_the_launch_limit():
    """130,560 samples of -8-8i, the most one launch takes: every real sum is
    128 T, every imaginary one 0."""
    T = 130_560
    _say("split extremes")
    for N in (5, 64):
        v = torch.full((T, 1, N), 0x88, dtype=torch.uint8, device="cuda")
        out = _run(v, N, 1, [T]).cpu().numpy()
        assert np.all(out[..., 0] == 128 * T) and np.all(out[..., 1] == 0)


# enough channels that the persistent kernel is the faster: pairs, a single
# triangle, several segments; the plain path is the reference
@pytest.mark.parametrize("N,F,T,offset", [(20, 2050, 70, 0), (60, 1030, 130, 4), (92, 515, 130, 8), (124, 515, 65, 0),
                                          (180, 515, 130, 12), (300, 260, 130, 4)])
def test_persistent_kernel_on_word_rows(N, F, T, offset):
    _say(f"word rows N={N} F={F} T={T} offset={offset}")
    v = _at(synth.uniform_volts4(N, F, 2 * T, seed=(2104, N)), offset)
    got = _run(v, N, F, [T, T])
    assert torch.equal(got, _run(v, N, F, [T, T], X.PATH_PLAIN))
    c = X.Correlator(N, F)
    c.ingest_blocks([v[:64], v[64:128]])
    a, _, _ = c.dump()
    torch.cuda.synchronize()
    c.close()
    assert torch.equal(a, _run(v, N, F, [128], X.PATH_PLAIN))


@pytest.mark.parametrize("N,F,T", [(99, 300, 161), (99, 300, 100), (66, 700, 40), (250, 60, 200)])
def test_unaligned_rows_of_many_channels(N, F, T):
    _say(f"unaligned rows N={N} F={F} T={T}")
    v = _at(synth.uniform_volts4(N, F, T, seed=(2105, N)), 0)
    assert torch.equal(_run(v, N, F, [T]), _run(v, N, F, [T], X.PATH_PLAIN))


def _run8(v, N, F, splits, path, last_dumps=False):
    c = X.Correlator(N, F, 8, path)
    t0 = 0
    for k, n in enumerate(splits):
        if last_dumps and k + 1 == len(splits):
            out, total, _ = c.ingest_dump(v[t0:t0 + n])
        else:
            c.ingest(v[t0:t0 + n], n)
        t0 += n
    if not last_dumps:
        out, total, _ = c.dump()
    torch.cuda.synchronize()
    assert total == sum(splits)
    c.close()
    return out


@pytest.mark.parametrize("T", [1, 15, 17, 128, 145, 300])
@pytest.mark.parametrize("N,F", [(n, f) for n in (1, 2, 31, 32, 33, 64, 66, 99, 130, 192) for f in (1, 3)])
def test_8bit_few_channels(N, F, T):
    """int8 exact; FP16 equal to the float64 oracle (every sum stays an
    integer below 2^24).  Around the 32-input block, the 64-input region, the
    16-sample step and the waves' first round of 128."""
    _say(f"split 8bit N={N} F={F} T={T}")
    v = synth.uniform_volts8(N, F, T, seed=(2106, N, F, T))
    d = v.cuda()
    want = oracle.xcorr(v.numpy(), 8, T, F, N)
    assert np.array_equal(_run8(d, N, F, [T], X.PATH_I8_MFMA).cpu().numpy(), oracle.to_int32(want))
    assert np.abs(want).max() < 2 ** 24
    assert np.array_equal(_run8(d, N, F, [T], X.PATH_F16_MFMA).cpu().numpy().astype(np.float64), want)


@pytest.mark.parametrize("path", [X.PATH_I8_MFMA, X.PATH_F16_MFMA], ids=["int8", "fp16"])
@pytest.mark.parametrize("N,F,offset", [(33, 3, 0), (33, 3, 1), (34, 3, 2), (34, 3, 4), (192, 3, 8), (130, 515, 4),
                                        (36, 1030, 8), (192, 300, 0)])
def test_8bit_starts_and_running_sums(N, F, offset, path):
    """Start addresses off the 16-byte boundaries, few and many channels; the
    last ingest adds to the running sums straight into the dump."""
    splits = [70, 33, 90]
    _say(f"split 8bit N={N} F={F} offset={offset}")
    v = synth.uniform_volts8(N, F, sum(splits), seed=(2107, N, offset))
    d = _at(v.view(torch.uint8), offset).view(torch.int8)
    want = _run8(d, N, F, splits, X.PATH_PLAIN)
    assert int(want.abs().max()) < 2 ** 24
    for last_dumps in (False, True):
        assert torch.equal(_run8(d, N, F, splits, path, last_dumps).to(torch.int32), want)


def test_8bit_dumping_ingest_leaves_nothing_behind():
    """Integrations that end with ingest_dump, one launch and several, one
    after another on a context."""
    N, F = 64, 40
    v = synth.uniform_volts8(N, F, 500, seed=(2108,)).cuda()
    c = X.Correlator(N, F, 8)
    spans = [(0, 100, 200), (50, 90), (10, 200, 260, 400)]
    for span in spans:
        for a, b in zip(span[:-2], span[1:-1]):
            c.ingest(v[a:b])
        out, n, _ = c.ingest_dump(v[span[-2]:span[-1]])
        assert n == span[-1] - span[0]
        assert torch.equal(out, _run8(v[span[0]:span[-1]], N, F, [n], X.PATH_PLAIN))
    c.close()
