"""Point preparation at the edges of its two sorting forms (GPU).

Sets up to 8192 points are ordered by counting ranks, larger ones by a radix
sort; both order by (Morton key, index).  Products through either are held to
the oracle at the bars of tests/parity.py, on sets with many equal keys (points
on a coarse grid, and d = 41, where a key has one bit per coordinate) and with a
few points far outside (tiles too wide to fold take the median anchor).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1408_1237_amd import api, workloads
from parity import DT, call_vector, check

pytestmark = pytest.mark.gpu


def _points(kind, n):
    rng = np.random.default_rng(n)
    if kind == "grid":
        return np.ascontiguousarray(rng.integers(0, 6, size=(n, 3)).astype(np.float64)), 1.5
    if kind == "wide41":
        return np.ascontiguousarray(rng.standard_normal((n, 41))), np.sqrt(41.0)
    x = rng.standard_normal((n, 2))
    x[rng.choice(n, max(1, n // 100), replace=False)] *= 500.0
    return np.ascontiguousarray(x), 0.7


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("kind,n", [("grid", 63), ("grid", 64), ("grid", 65), ("grid", 1025), ("outliers", 2000),
                                    ("outliers", 8191), ("grid", 8192), ("outliers", 8193), ("wide41", 1100),
                                    ("wide41", 8200)])
def test_products_at_the_sorting_edges(prec, kind, n):
    x, sigma = _points(kind, n)
    q = workloads.random_vector(n, n)
    y = api.kmvp_gauss(torch.from_numpy(x).cuda(), sigma, torch.from_numpy(q).to(DT[prec]).cuda(), shift=0.02,
                       prec=prec)
    rows = np.random.default_rng(n + 1).choice(n, min(n, 200), replace=False)
    want = oracle.mvp_rows(x, sigma, call_vector(q, prec), rows, shift=0.02)
    check(y.double().cpu().numpy()[rows], want, prec, what=(kind, n))
