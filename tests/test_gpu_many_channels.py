"""More work-groups than one grid dimension counts the threads of (32 bits):
every channel must be written, whichever kernel runs."""
import pytest
import torch

from paper_2406_19013_amd import synth
from paper_2406_19013_amd import xcorr as X

pytestmark = pytest.mark.gpu

CASES = {"split4": (4, X.PATH_I8_MFMA, 0, ""), "fused4": (4, X.PATH_I8_MFMA, 2, ""),
         "roles4": (4, X.PATH_I8_MFMA, 2, "roles"), "plain4": (4, X.PATH_PLAIN, 0, ""),
         "split8": (8, X.PATH_I8_MFMA, 0, ""), "split8_f16": (8, X.PATH_F16_MFMA, 0, ""),
         "mfma8": (8, X.PATH_I8_MFMA, 2, ""), "mfma8_f16": (8, X.PATH_F16_MFMA, 2, ""),
         "plain8": (8, X.PATH_PLAIN, 0, "")}


@pytest.mark.parametrize("name", CASES)
def test_every_channel_is_written(name, monkeypatch):
    """One input, 2^24 + 5 channels (a work-group each, of 256 threads on the
    plain path and 512 on the others), stored and added."""
    bits, path, tile, variant = CASES[name]
    if variant:
        monkeypatch.setenv("XCORR_MFMA4_VARIANT", variant)
    else:
        monkeypatch.delenv("XCORR_MFMA4_VARIANT", raising=False)
    F, T = (1 << 24) + 5, 3
    print(f"many channels {name} F={F}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(2401)
    x = torch.randint(-8 if bits == 4 else -127, 8 if bits == 4 else 128, (T, F, 1, 2), generator=g, device="cuda",
                      dtype=torch.int8)
    v = synth.pack4(x[..., 0], x[..., 1]) if bits == 4 else x
    c = X.Correlator(1, F, bits, path, tile=tile)
    c.ingest(v)
    c.ingest(v[:1])
    out, n, _ = c.dump()
    torch.cuda.synchronize()
    c.close()
    p = x.to(torch.int32).square().sum(dim=(2, 3))
    assert n == T + 1
    assert torch.equal(out[:, 0, 0].to(torch.int32), p.sum(dim=0, dtype=torch.int32) + p[0])
    assert not out[:, 0, 1].any()
