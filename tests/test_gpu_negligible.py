"""Tile pairs left out as negligible, for vectors of any size distribution (GPU).

The symmetric products leave out a pair of tiles whose sources, by the tile's sum of
|q|, are below 2^-40 (FP64 2^-69) of what the rows of the other tile hold, by a floor
from the rows' own |q|.  Every kernel that produces a product's vector writes these
bounds.  Products, truncated CG solves and FGMRES steps with nothing left out
(KRR_NO_TILE_SKIP=1) against the same calls as they are, on clusters whose pairs lie
between negligible and out of range, with vectors that make the floors differ:
signed, a single nonzero entry, clusters of zeros, one cluster 1e15 times larger or
smaller.  Per row, relative to sum_j k_ij |q_j|: two roundings of the sum (2^-22,
FP64 2^-51); what is left out is 2^-16 of one.
"""
import numpy as np
import pytest
import torch

from paper_1408_1237_amd import api, native

pytestmark = pytest.mark.gpu

DT = {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.float32}
ROUND2 = {"fp64": 2.0 ** -51, "fp32": 2.0 ** -22, "bf16": 2.0 ** -22}
VECTORS = ["signed", "one", "zeros", "large", "small"]
SIZES = [(12, 250, 2), (12, 600, 6), (12, 600, 16), (10, 2600, 3), (6, 700, 8)]


def _clusters(k, m, d, kernel):
    """k clusters of m points along the diagonal (so that the space-filling order of
    the tiles keeps them apart), neighbours 10 (Matern 40) scaled units apart."""
    rng = np.random.default_rng(100 * k + d)
    gap = 10.0 / np.sqrt(np.log2(np.e) / 2) if kernel == "gauss" else 40.0 / np.sqrt(3.0)
    x = 0.3 / np.sqrt(d) * rng.standard_normal((k, m, d))
    x += gap / np.sqrt(d) * np.arange(k)[:, None, None]
    return torch.from_numpy(x.reshape(-1, d)[rng.permutation(k * m)].copy()).cuda()


def _vector(kind, x, prec):
    n = x.shape[0]
    q = torch.from_numpy(np.random.default_rng(n).standard_normal(n)).cuda()
    lo, hi = float(x[:, 0].min()), float(x[:, 0].max())
    part = (x[:, 0] - lo) / (hi - lo)  # along the row of clusters
    if kind == "one":
        keep = int(torch.argmin((part - 0.5).abs()))
        q = torch.where(torch.arange(n, device="cuda") == keep, q, torch.zeros_like(q))
    elif kind == "zeros":
        q = torch.where((part > 0.3) & (part < 0.7), torch.zeros_like(q), q)
    elif kind in ("large", "small"):
        q = torch.where(part > 0.9, q * (1e15 if kind == "large" else 1e-15), q)
    return q.to(DT[prec])


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("kernel", ["gauss", "matern"])
@pytest.mark.parametrize("k,m,d", SIZES)
def test_products_with_and_without(k, m, d, kernel, prec, monkeypatch):
    x = _clusters(k, m, d, kernel)
    f = api.kmvp_matern if kernel == "matern" else api.kmvp_gauss
    for kind in VECTORS:
        q = _vector(kind, x, prec)
        with native.profile() as prof:
            y = f(x, 1.0, q, shift=0.0, prec=prec)
            torch.cuda.synchronize()
        if kind == "signed":
            assert prof.stats[prec]["pairs_skipped"] > 0
        monkeypatch.setenv("KRR_NO_TILE_SKIP", "1")
        want, size = f(x, 1.0, q, shift=0.0, prec=prec), f(x, 1.0, q.abs(), shift=0.0, prec=prec)
        monkeypatch.delenv("KRR_NO_TILE_SKIP")
        off = (y.double() - want.double()).abs()
        assert bool(torch.isfinite(y).all())
        assert bool((off <= ROUND2[prec] * size.double()).all()), kind


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("kernel", ["gauss", "matern"])
@pytest.mark.parametrize("d", [2, 8])
def test_a_nan_is_never_left_out(d, kernel, prec):
    x = _clusters(2, 700, d, kernel)
    q = _vector("signed", x, prec)
    q[5] = float("nan")
    f = api.kmvp_matern if kernel == "matern" else api.kmvp_gauss
    assert bool(torch.isnan(f(x, 1.0, q, shift=0.0, prec=prec)).all())


# the vectors that the solvers' own kernels produce: well-conditioned systems, whose
# iterates carry a few roundings of the products (BF16: of the direction as well)
CG_BAR = {"fp64": 1e-13, "fp32": 1e-5, "bf16": 1e-2}


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("k,m,d", SIZES)
def test_truncated_cg_with_and_without(k, m, d, prec, monkeypatch):
    x = _clusters(k, m, d, "gauss")
    for kind in VECTORS:
        v = _vector(kind, x, prec)
        z = api.cg_inner_solve(x, 1.0, 1e3, v, 3, prec=prec)[0].double()
        monkeypatch.setenv("KRR_NO_TILE_SKIP", "1")
        want = api.cg_inner_solve(x, 1.0, 1e3, v, 3, prec=prec)[0].double()
        monkeypatch.delenv("KRR_NO_TILE_SKIP")
        assert bool((z - want).norm() <= CG_BAR[prec] * want.norm()), kind


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("k,m,d", [(12, 250, 2), (12, 600, 6)])
def test_fgmres_steps_with_and_without(k, m, d, prec, monkeypatch):
    x = _clusters(k, m, d, "gauss")
    for kind in VECTORS:
        y = _vector(kind, x, "fp64")
        opts = dict(tol=1e-10, max_outer=30, inner_prec=prec)
        w, info = api.fgmres_solve(x, 1.0, 1e3, y, **opts)
        monkeypatch.setenv("KRR_NO_TILE_SKIP", "1")
        want, info2 = api.fgmres_solve(x, 1.0, 1e3, y, **opts)
        monkeypatch.delenv("KRR_NO_TILE_SKIP")
        assert info["status"] == 0 and info2["status"] == 0
        assert bool((w - want).norm() <= 1e-8 * want.norm()), kind
