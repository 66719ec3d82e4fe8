"""FP8 encoder (cm_fp8_encode) at the edges of its tiles and of its short form:
the codes of plain values (0 <= x < 2^100) must not depend on whether a value
beside them takes the general form, at scales on both sides of the short
form's range."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SCALES = [2.0 ** e for e in (-41, -40, -3, 0, 4, 13, 14)]


@pytest.mark.parametrize("scale", SCALES)
def test_short_form_equals_general_form(scale):
    import torch
    import paper_2012_07145_amd as cm
    # every 2,003rd bit pattern from 0 to just below 2^100, and the values
    # around the points where 1 + x, the form or the code changes
    bits = torch.arange(0, 0x71800000, 2003, dtype=torch.int64, device="cuda")
    near = torch.tensor([b + o for b in (0x0, 0x33000000, 0x33800000, 0x34000000, 0x3f800000,
                                         0x71800000) for o in range(-8, 9) if 0 <= b + o < 0x71800000],
                        dtype=torch.int64, device="cuda")
    x = torch.cat([bits, near]).to(torch.int32).view(torch.float32)
    short = cm.cm_fp8_encode(x, scale)
    # a NaN in every 64 values sends every wave to the general form
    n = x.numel()
    mixed = torch.full((-(-n // 63), 64), float("nan"), device="cuda")
    padded = torch.zeros(mixed.shape[0] * 63, device="cuda")
    padded[:n] = x
    mixed[:, :63] = padded.view(-1, 63)
    general = cm.cm_fp8_encode(mixed.reshape(-1), scale).view(-1, 64)
    torch.cuda.synchronize()
    assert (general[:, 63] == 0x7F).all()
    assert torch.equal(general[:, :63].reshape(-1)[:n], short)


@pytest.mark.parametrize("n", [1, 3, 255, 4095, 4096, 4097, 8191, 8192 + 17, 40000])
def test_encode_tile_edges(oracle_mod, n):
    import torch
    import paper_2012_07145_amd as cm
    rng = np.random.default_rng(n)
    x = np.exp(rng.normal(4.0, 2.0, n)).astype(np.float32)
    x[:: 7] = 0.0
    out = torch.full((n + 32,), 0xEE, dtype=torch.uint8, device="cuda")
    cm.cm_fp8_encode(torch.from_numpy(x).cuda(), 16.0, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    want = oracle_mod.fp8_codes(x, 16.0)
    assert np.all(got[n:] == 0xEE)
    # a code may differ by one step where log1p(x) * s is within 1e-6 of a
    # midpoint: the float32 log1p is within a few ulps
    bad = np.nonzero(got[:n] != want)[0]
    assert np.all(np.abs(got[bad].astype(int) - want[bad].astype(int)) == 1)
    dec = np.array([oracle_mod.e4m3_decode(c) for c in range(256)])
    y = np.log1p(x[bad].astype(np.float64)) * 16.0
    mid = 0.5 * (dec[got[bad]] + dec[want[bad]])
    assert np.all(np.abs(y - mid) <= 1e-6 * np.abs(mid))
