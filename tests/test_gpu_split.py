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
