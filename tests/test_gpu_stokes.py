"""GPU full-Stokes formation against the Stokes oracle, bit for bit (int64)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from oracle import stokes as st  # noqa: E402
from paper_2406_19013_amd import synth  # noqa: E402
from paper_2406_19013_amd import xcorr as X  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("N,F", [(2, 1), (6, 3), (192, 4)])
def test_random_dumps(N, F):
    """Any int32 visibilities, including the extremes: the int64 sums are exact."""
    rng = np.random.default_rng(N * 7 + F)
    P = N * (N + 1) // 2
    v = rng.integers(-2 ** 31, 2 ** 31, size=(F, P, 2), dtype=np.int64).astype(np.int32)
    v[0, 0] = [2 ** 31 - 1, -2 ** 31]
    got = X.xcorr_stokes(torch.from_numpy(v).to(DEV), N).cpu().numpy()
    assert np.array_equal(got, st.stokes(v, N))


def test_polarised_source_end_to_end():
    """4+4-bit voltages: each feed's X carries a common signal s plus noise
    and Y carries s too (linear at 45 degrees), so U dominates Q and V in
    every feed pair; GPU X-engine + GPU Stokes equal the oracles exactly."""
    N, F, T = 32, 4, 512
    g = torch.Generator().manual_seed(synth.seed_of(synth.BASE_SEED, 70))
    s_re = torch.randint(-3, 4, (T, F, 1), generator=g)
    s_im = torch.randint(-3, 4, (T, F, 1), generator=g)
    n_re = torch.randint(-2, 3, (T, F, N), generator=g)
    n_im = torch.randint(-2, 3, (T, F, N), generator=g)
    v = synth.pack4(s_re + n_re, s_im + n_im)
    c = X.Correlator(N, F, 4, X.PATH_I8_MFMA, device=DEV)
    vis, _, _ = c.ingest_dump(v.to(DEV))
    c.close()
    got = X.xcorr_stokes(vis, N).cpu().numpy()
    want = st.stokes(oracle.xcorr(v.numpy(), 4, T, F, N), N)
    assert np.array_equal(got, want)
    Q, U, V = (np.abs(want[:, :, k, 0]) for k in (1, 2, 3))
    assert (U > 4 * Q).mean() > 0.9 and (U > 4 * V).mean() > 0.9


def test_refusals():
    v = torch.zeros((1, 6, 2), dtype=torch.int32, device=DEV)
    with pytest.raises(X.XcorrError):
        X.xcorr_stokes(v, 3)


@pytest.mark.parametrize("N,F", [(18, 5), (22, 8), (514, 2), (1030, 1)])
def test_channel_groups_and_many_feeds(N, F):
    """Channel counts on both sides of the four a thread takes, pair counts
    off the work-group's 64, and many feeds (the pair index is found from a
    float square root)."""
    rng = np.random.default_rng(N + F)
    v = rng.integers(-2 ** 31, 2 ** 31, size=(F, N * (N + 1) // 2, 2), dtype=np.int64).astype(np.int32)
    got = X.xcorr_stokes(torch.from_numpy(v).to(DEV), N).cpu().numpy()
    assert np.array_equal(got, st.stokes(v, N))


def test_more_lanes_than_a_grid_row_counts():
    """92,682 inputs: four lanes for each of 2^30 feed pairs are more threads
    than 32 bits count.  Every element must be written; pairs at the start, on
    both sides of the 2^32nd lane and at the end against the definition."""
    N = 92_682
    nf = N // 2
    P, Pf = N * (N + 1) // 2, nf * (nf + 1) // 2
    assert 4 * Pf > 2 ** 32
    if torch.cuda.mem_get_info()[0] < 8 * P + 64 * Pf + (2 << 30):
        pytest.skip("needs 106 GB of GPU memory")
    vis = torch.empty((1, P, 2), dtype=torch.int32, device=DEV)
    flat = vis.view(-1)
    step = 1 << 28
    for k in range(0, 2 * P, step):        # every int32 of its own: the element's index, mixed
        i = torch.arange(k, min(2 * P, k + step), dtype=torch.int64, device=DEV)
        flat[k:k + step] = ((i * 2654435761) >> 3).to(torch.int32)
    never = -(1 << 62)
    out = torch.full((1, Pf, 4, 2), never, dtype=torch.int64, device=DEV)
    X.xcorr_stokes(vis, N, out)
    left = sum(int((out[0, k:k + step] == never).sum()) for k in range(0, Pf, step))
    assert left == 0

    def v(i, j):
        return [int(x) for x in vis[0, i * (i + 1) // 2 + j].tolist()]

    a1 = int((2 * 2 ** 30) ** 0.5) - 1     # about the pair of the 2^32nd lane
    pairs = [(0, 0), (1, 0), (1, 1), (nf - 1, 0), (nf - 1, nf - 2), (nf - 1, nf - 1)] + \
            [(a, b) for a in range(a1 - 1, min(nf, a1 + 3)) for b in (0, a // 2, a - 1, a)]
    for a, b in pairs:
        xx, yy, yx = v(2 * a, 2 * b), v(2 * a + 1, 2 * b + 1), v(2 * a + 1, 2 * b)
        xy = v(2 * a, 2 * b + 1) if a > b else [yx[0], -yx[1]]
        d = [xy[0] - yx[0], xy[1] - yx[1]]
        want = [[xx[0] + yy[0], xx[1] + yy[1]], [xx[0] - yy[0], xx[1] - yy[1]],
                [xy[0] + yx[0], xy[1] + yx[1]], [d[1], -d[0]]]
        assert out[0, a * (a + 1) // 2 + b].tolist() == want, (a, b)
    del vis, out, flat
    torch.cuda.empty_cache()
