"""FP32 / BF16 products that test half tiles for negligible pairs (GPU).

Up to four coordinates and above 100 tiles the symmetric product tests the two
halves of a row tile on their own.  Each size ends on another fill of the last
tile (one point: its second half is empty; one point in the second half; both
partly filled), on sets where many pairs, and single halves of pairs, are left
out.  Against the same product with nothing left out: what is left out is below
2^-40 of a row, so with a positive vector each entry agrees within two FP32
roundings of the sum (2^-22), and the profile says that pairs were left out.
"""
import numpy as np
import pytest
import torch

from paper_1408_1237_amd import api, native, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("n", [100 * 256 + 1, 100 * 256 + 129, 30_000])
@pytest.mark.parametrize("d,kernel", [(1, "gauss"), (2, "gauss"), (4, "gauss"), (3, "matern")])
def test_half_tiles_left_out(d, kernel, n, prec, monkeypatch):
    x = torch.from_numpy(workloads.random_points(60 + d, n, d, 1.0)).cuda()
    q = torch.from_numpy(0.1 + np.abs(workloads.random_vector(61, n))).float().cuda()
    f, sigma = (api.kmvp_matern, 0.01) if kernel == "matern" else (api.kmvp_gauss, 0.02)
    with native.profile() as prof:
        y = f(x, sigma, q, shift=1e-2, prec=prec)
        torch.cuda.synchronize()
    st = prof.stats[prec]
    assert 0 < st["pairs_skipped"] < st["pairs"]
    monkeypatch.setenv("KRR_NO_TILE_SKIP", "1")
    want = f(x, sigma, q, shift=1e-2, prec=prec)
    assert bool(torch.isfinite(y).all())
    assert float(((y - want).abs() / want).max()) <= 2.0 ** -22
