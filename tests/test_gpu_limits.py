"""The persistent 4+4-bit kernels at the most samples one launch gives them,
and with many short items to a work-group; each test asserts that the kernel
it is about is the one that runs.  Whole numbers throughout: every comparison
is exact."""
import pytest
import torch

from paper_2406_19013_amd import synth
from paper_2406_19013_amd import xcorr as X

pytestmark = pytest.mark.gpu

# what the parts of a sample can reach: the products of input i with input j
# run from -112 - 120i to 128 per sample, and every partial sum of a kernel to
# its largest of either sign
EXTREMES = torch.tensor([[-8, -8], [-8, 7], [7, -8], [7, 7], [-8, 0], [0, -8]])


def _constant_inputs(N, F, T):
    """Input k holds EXTREMES[k % 6] throughout."""
    e = EXTREMES[torch.arange(N) % 6]
    row = synth.pack4(e[:, 0], e[:, 1]).cuda()
    return row.expand(T, F, N).contiguous()


def _want(N, T):
    e = EXTREMES[torch.arange(N) % 6].to(torch.int64)
    i, j = torch.tril_indices(N, N)
    re = e[i, 0] * e[j, 0] + e[i, 1] * e[j, 1]
    im = e[i, 1] * e[j, 0] - e[i, 0] * e[j, 1]
    return (torch.stack([re, im], dim=1) * T).to(torch.int32).cuda()


def _correlator(N, F, T, kernel, v, tile=0):
    assert X.xcorr_ingest_kernel(X.make_config(N, F, tile=tile), v, T) == kernel
    return X.Correlator(N, F, tile=tile)


# launch limits: 65,472 samples for 128-input segments (2^15 a sample), 130,560
# for the others; one sample more than the segments take
LIMITS = [(128, 160, 65_472, 0, "xc_duo4_kernel"), (256, 160, 65_472, 0, "xc_duo4_kernel"),
          (512, 48, 65_472, 0, "xc_duo4_kernel"), (192, 128, 130_560, 0, "xc_tri48_kernel"),
          (256, 160, 65_473, 0, "xc_gauss4_kernel"), (256, 160, 130_560, 0, "xc_gauss4_kernel"),
          (16, 1, 130_560, 2, "xc_gauss4_kernel"), (96, 2, 130_560, 3, "xc_gauss4_kernel"),
          (128, 2, 130_560, 4, "xc_gauss4_kernel"), (192, 2, 130_560, 6, "xc_gauss4_kernel"),
          (512, 2, 130_560, 4, "xc_gauss4_kernel"), (96, 2, 130_560, 0, "xc_split_kernel"),
          (99, 2, 130_560, 0, "xc_split_kernel"), (100, 2, 130_560, 3, "xc_mfma4f_kernel")]


@pytest.mark.parametrize("N,F,T,tile,kernel", LIMITS, ids=[f"N{n}T{t}D{d}_{k[3:-7]}" for n, f, t, d, k in LIMITS])
def test_extreme_constants_at_the_launch_limit(N, F, T, tile, kernel):
    print(f"limit N={N} F={F} T={T} tile={tile} {kernel}", flush=True)
    v = _constant_inputs(N, F, T)
    c = _correlator(N, F, T, kernel, v, tile)
    c.ingest(v)
    out, n, _ = c.dump()
    torch.cuda.synchronize()
    c.close()
    assert n == T and torch.equal(out, _want(N, T).expand(F, -1, -1))
    del v, out
    torch.cuda.empty_cache()


@pytest.mark.parametrize("N,F,T,kernel", [(128, 160, 65_472, "xc_duo4_kernel"), (256, 160, 65_472, "xc_duo4_kernel"),
                                          (192, 128, 130_560, "xc_tri48_kernel")])
def test_extreme_mix_at_the_launch_limit(N, F, T, kernel):
    """Re and im drawn from {-8, 7}, a pattern of 977 rows repeated."""
    print(f"mix N={N} F={F} T={T} {kernel}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(2402)
    pick = torch.tensor([-8, 7], device="cuda")
    part = [pick[torch.randint(0, 2, (977, F, N), generator=g, device="cuda")] for _ in range(2)]
    p = synth.pack4(*part)
    v = p.repeat((T + 976) // 977, 1, 1)[:T].contiguous()
    c = _correlator(N, F, T, kernel, v)
    out, n, _ = c.ingest_dump(v)
    del v
    # T = k 977 + r rows: the plain path's sums of the pattern and of its first r
    k, r = divmod(T, 977)
    ref = X.Correlator(N, F, 4, X.PATH_PLAIN)
    whole, _, _ = ref.ingest_dump(p)
    rest = ref.ingest_dump(p[:r])[0] if r else 0
    torch.cuda.synchronize()
    assert n == T and torch.equal(out, whole * k + rest)
    c.close()
    ref.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("N,F,block,n,kernel", [(256, 160, 8192, 9, "xc_gauss4_kernel"),
                                                (128, 160, 16_384, 8, "xc_split_kernel"),
                                                (192, 128, 16_384, 8, "xc_tri48_kernel")])
def test_blocks_past_the_segment_bound(N, F, block, n, kernel):
    """Groups of blocks of 65,536 and 114,688 samples, then a last one added."""
    print(f"blocks N={N} F={F} {n} x {block}", flush=True)
    v = _constant_inputs(N, F, block)
    group = min(8, 130_560 // block) * block
    c = _correlator(N, F, group, kernel, v)
    c.ingest_blocks([v] * n)
    out, total, _ = c.dump()
    torch.cuda.synchronize()
    assert c.stats()["kernel_launches"] == 3
    c.close()
    assert total == n * block and torch.equal(out, _want(N, n * block).expand(F, -1, -1))
    del v, out
    torch.cuda.empty_cache()


SHORT = [(192, 1200, "xc_tri48_kernel"), (132, 1100, "xc_tri48_kernel"), (128, 2048, "xc_duo4_kernel"),
         (100, 2048, "xc_duo4_kernel"), (512, 400, "xc_duo4_kernel"), (260, 900, "xc_duo4_kernel"),
         (16, 4097, "xc_gauss4_kernel"), (32, 4096, "xc_gauss4_kernel"), (80, 3000, "xc_gauss4_kernel")]


@pytest.mark.parametrize("T", [1, 64, 65, 128, 200])
@pytest.mark.parametrize("N,F,kernel", SHORT, ids=[f"N{n}F{f}" for n, f, _ in SHORT])
def test_many_short_items_per_workgroup(N, F, kernel, T):
    """Three and more items of one to four ring slots to a work-group: an
    item's stores are still in flight when the next ones' samples are waited
    for, and its per-input sums make way for the next item's.  Stored, added,
    and dumped by the launch."""
    print(f"short items N={N} F={F} T={T}", flush=True)
    v = synth.uniform_volts4(N, F, T, seed=(2403, N, T), device="cuda")
    if T <= 64 and N in (132, 192):   # at most half a slot
        kernel = "xc_gauss4_kernel"
    c = _correlator(N, F, T, kernel, v)
    ref = X.Correlator(N, F, 4, X.PATH_PLAIN)
    want, _, _ = ref.ingest_dump(v)
    ref.close()
    for _ in range(2):
        stored, _, _ = c.ingest_dump(v)
        c.ingest(v)
        added, _, _ = c.ingest_dump(v)
        torch.cuda.synchronize()
        assert torch.equal(stored, want) and torch.equal(added, 2 * want)
    if T % 64 == 0 and N % 16 == 0:
        c.ingest_blocks([v, v, v])
        out, _, _ = c.dump()
        torch.cuda.synchronize()
        assert torch.equal(out, 3 * want)
    c.close()
