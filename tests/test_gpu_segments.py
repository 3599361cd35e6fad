"""The 4+4-bit kernels for 128-input segments (97 to 128 inputs and more than
192) and for one triangle of 129 to 192 inputs: exact parity, against the
oracle where it is quick and against the plain path on larger inputs.  Sums of
4-bit samples over the launch limits stay within int32, so every comparison is
of whole numbers."""
import numpy as np
import pytest
import torch

import oracle
from paper_2406_19013_amd import synth
from paper_2406_19013_amd import xcorr as X

pytestmark = pytest.mark.gpu


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


# inputs at the edges of the 16-, 32- and 48-input blocks and of the 128-input
# segments; samples around a 64- and a 128-row slot; channels enough that the
# few-channel kernel is not taken
@pytest.mark.parametrize("T", [1, 64, 65, 129, 700])
@pytest.mark.parametrize("N", [100, 128, 132, 144, 148, 160, 164, 192, 196, 260, 388])
def test_edges_match_plain(N, T):
    F = 260 if N <= 192 else 130
    print(f"segments N={N} F={F} T={T}", flush=True)
    v = synth.uniform_volts4(N, F, T, seed=(2301, N, T), device="cuda")
    assert torch.equal(_run(v, N, F, [T]), _run(v, N, F, [T], X.PATH_PLAIN))


@pytest.mark.parametrize("N", [128, 180, 256])
def test_running_sums_from_any_word(N):
    """Rows that start on 4-byte boundaries only and end with their
    allocation; later ingests add to running sums, the last one dumps."""
    F, splits = 270, [64, 7, 300]
    T = sum(splits)
    v = synth.uniform_volts4(N, F, T, seed=(2302, N), device="cuda")
    raw = torch.empty(v.numel() + 4, dtype=torch.uint8, device="cuda")
    raw[4:] = v.reshape(-1)
    w = raw[4:].view(v.shape)
    want = _run(v, N, F, [T], X.PATH_PLAIN)
    assert torch.equal(_run(w, N, F, splits), want)
    c = X.Correlator(N, F, 4, X.PATH_I8_MFMA)
    c.ingest(w[:71], 71)
    out = torch.empty_like(want)
    c.ingest_dump(w[71:], out=out)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    c.close()


@pytest.mark.parametrize("N", [112, 176, 272])
def test_blocks_of_odd_count(N):
    """A block table whose 64-row chunks leave the last 128-row slot half full."""
    F, nb, B = 300, 5, 64
    blocks = [synth.uniform_volts4(N, F, B, seed=(2303, N, k), device="cuda") for k in range(nb)]
    c = X.Correlator(N, F, 4, X.PATH_I8_MFMA)
    c.ingest_blocks(blocks)
    c.ingest_blocks(blocks[:2])
    out, n, _ = c.dump()
    torch.cuda.synchronize()
    assert n == (nb + 2) * B
    v = torch.cat(blocks + blocks[:2])
    assert torch.equal(out, _run(v, N, F, [v.shape[0]], X.PATH_PLAIN))
    c.close()


@pytest.mark.parametrize("N,T", [(128, 65472), (128, 65473), (192, 130560), (256, 65472)])
def test_extreme_samples_at_the_launch_limits(N, T):
    """Every sample -8 - 8i, whose sums reach 128 per sample: the int32 bounds
    of a launch, on a few channels' worth of memory."""
    F = 4 if N > 128 else 8
    v = torch.full((T, F, N), 0x88, dtype=torch.uint8, device="cuda")
    c = X.Correlator(N, F, 4, X.PATH_I8_MFMA)
    c.ingest(v, T)
    out, _, _ = c.dump()
    torch.cuda.synchronize()
    assert (out[..., 0] == 128 * T).all() and (out[..., 1] == 0).all()
    c.close()
    del v, out
    torch.cuda.empty_cache()


def test_oracle_parity():
    for N, F, T in ((128, 260, 40), (192, 260, 40), (200, 130, 40)):
        v = synth.uniform_volts4(N, F, T, seed=(2304, N))
        want = oracle.to_int32(oracle.xcorr(v.numpy(), 4, T, F, N))
        assert np.array_equal(_run(v.cuda(), N, F, [T]).cpu().numpy(), want)


@pytest.mark.parametrize("T", [64, 1100])
def test_batch_members_launched_by_themselves(T):
    """Members that fill the chip beside ones that share a launch, and alone;
    the second ingest adds to running sums."""
    arrays = [(256, 264), (64, 8), (192, 256), (512, 128)]
    for pick in (arrays, arrays[:1]):
        vs = [synth.uniform_volts4(N, F, T, seed=(2305, T, N), device="cuda") for N, F in pick]
        cors = [X.Correlator(N, F) for N, F in pick]
        b = X.Batch(cors)
        for _ in range(2):
            b.ingest(vs)
        for (N, F), v, c in zip(pick, vs, cors):
            out, n, _ = c.dump()
            torch.cuda.synchronize()
            assert n == 2 * T and c.stats()["kernel_launches"] == 3
            assert torch.equal(out, 2 * _run(v, N, F, [T], X.PATH_PLAIN)), (N, F)
        b.close()


@pytest.mark.parametrize("N,F,T", [(512, 601, 5056), (260, 1001, 5056)])
def test_long_launches_in_two(N, F, T):
    """Channels of an odd count in two launches: stored, added, from a block
    table and dumped, against the three-product kernel."""
    print(f"two launches N={N} F={F} T={T}", flush=True)
    v = synth.uniform_volts4(N, F, T, seed=(2306, N), device="cuda")
    assert X.xcorr_ingest_kernel(X.make_config(N, F), v, T) == "xc_duo4_kernel"
    ref = X.Correlator(N, F, tile=4)
    want, _, _ = ref.ingest_dump(v)
    ref.close()
    c = X.Correlator(N, F)
    out, _, _ = c.ingest_dump(v)
    assert torch.equal(out, want)
    c.ingest(v)
    out, _, _ = c.ingest_dump(v)
    assert torch.equal(out, 2 * want)
    if N % 16 == 0:
        c.ingest_blocks([v, v])
        out, _, _ = c.dump()
        assert torch.equal(out, 2 * want)
    torch.cuda.synchronize()
    c.close()
