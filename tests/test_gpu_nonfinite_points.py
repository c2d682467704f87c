"""NaN coordinates in the products and the gradient pass (GPU).

The product calls do not check their points (the solvers do); a NaN coordinate
makes every row NaN, although the symmetric products leave tile pairs out by boxes
whose minima and maxima pass a NaN over: also where a whole tile or half tile is
NaN, and whatever the workspace held before.
"""
import numpy as np
import pytest
import torch

from paper_1408_1237_amd import api, native

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _used_workspace(which, n, d):
    """A workspace that holds finite numbers, as after an earlier call."""
    ws = api.workspace((native.workspace_size(which, [(n, d)]) + 7) // 8 * 8, "cuda")
    ws.view(torch.float64).fill_(1.0)
    return ws


def _points(kind, n, d):
    x = np.random.default_rng(n).random((n, d))
    if kind == "column":
        x[:, d - 1] = np.nan
    elif kind == "point":
        x[n // 2, 0] = np.nan
    else:  # the first tile and half of the next one in the sorted order
        assert kind == "tiles"
        x[:384] = np.nan
    return x


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("kernel", ["gauss", "matern"])
@pytest.mark.parametrize("kind,n,d", [("column", 1, 2), ("column", 300, 3), ("column", 26_000, 2), ("column", 700, 16),
                                      ("point", 2000, 2), ("point", 26_000, 2), ("tiles", 2000, 2),
                                      ("tiles", 26_000, 2), ("tiles", 2000, 8)])
def test_products_with_nan_points(kind, n, d, kernel, prec):
    x = _points(kind, n, d)
    q = torch.ones(n, dtype=torch.float64 if prec == "fp64" else torch.float32, device="cuda")
    f, sigma = (api.kmvp_matern, 0.1) if kernel == "matern" else (api.kmvp_gauss, 0.1)
    y = f(_t(x), sigma, q, shift=0.5, prec=prec, ws=_used_workspace(native.KRR_WS_KMVP, n, d))
    assert bool(torch.isnan(y).all())


@pytest.mark.parametrize("d", [3, 9, 12, 16])
@pytest.mark.parametrize("same", [False, True])
def test_gradient_with_a_nan_point(d, same):
    n = 600
    rng = np.random.default_rng(d)
    x = rng.standard_normal((n, d))
    x[7, 2] = np.nan
    lam = _t(rng.standard_normal(n))
    w = lam if same else _t(rng.standard_normal(n))
    gx, gs, gg = api.kmvp_grad(_t(x), np.sqrt(d), 0.1, lam, w)
    assert bool(torch.isnan(gx[:, 2]).all()) and bool(torch.isnan(gs)) and bool(torch.isfinite(gg))
