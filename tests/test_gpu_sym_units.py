"""Square products of small sets, where several blocks share a pair of tiles (GPU).

The number of blocks per pair changes with the tile count (FP64: 4 to 12 tiles, 2
to 32; FP32 / BF16: 2 to 20) and the row groups per wave with it and the compiled
dimension.  Sizes on both sides of each change, the last tile full or of one
point, against the oracle's rows, for both kernels; a set with far tiles takes the
skipped-pair path of a share.  Positive vectors, so that no row cancels and the
bars of tests/parity.py hold with no format floor.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1408_1237_amd import api, workloads
from parity import call_vector, check

pytestmark = pytest.mark.gpu


def _run(x, sigma, kernel, prec, seed):
    n = x.shape[0]
    dt = torch.float64 if prec == "fp64" else torch.float32
    q = torch.from_numpy(0.1 + np.abs(workloads.random_vector(seed, n))).to(dt).cuda()
    f, rows_of = ((api.kmvp_matern, oracle.matern_mvp_rows) if kernel == "matern" else
                  (api.kmvp_gauss, oracle.mvp_rows))
    y = f(torch.from_numpy(x).cuda(), sigma, q, shift=1e-2, prec=prec).double().cpu().numpy()
    rows = np.unique(np.r_[0, n - 1, np.random.default_rng(seed).integers(0, n, 40)])
    want = rows_of(x, sigma, call_vector(q.double().cpu().numpy(), prec), rows, shift=1e-2)
    check(y[rows], want, prec, what=(kernel, n, x.shape[1]))


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("n", [1, 257, 12 * 256, 12 * 256 + 1, 20 * 256, 20 * 256 + 1, 32 * 256, 32 * 256 + 1])
@pytest.mark.parametrize("d", [2, 6, 8, 16])
@pytest.mark.parametrize("kernel", ["gauss", "matern"])
def test_shared_tile_pairs(kernel, d, n, prec):
    x = workloads.random_points(900 + d, n, d, 1.0, kind="normal")
    _run(x, 0.7 * np.sqrt(d), kernel, prec, 900 + n % 97)


@pytest.mark.parametrize("kernel", ["gauss", "matern"])
def test_shared_tile_pairs_far(kernel):
    # clusters further apart than the kernel reaches: whole pairs are left out.  FP64
    # only: a tile across two clusters holds offsets of 10^4 widths, whose FP32
    # rounding alone (5e-4 of a width) is beyond the FP32 bar
    x = workloads.random_points(77, 2500, 2, 1.0, kind="normal")
    x[:, 0] += 5000.0 * (np.arange(2500) % 3)
    _run(x, 0.5, kernel, "fp64", 5)
