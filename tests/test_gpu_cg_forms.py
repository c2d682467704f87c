"""The forms of a CG iteration's vector part (GPU).

Up to 4096 padded points one block does everything after the product; above, the
finish with the step length, the update and the direction are three launches;
sets of a single tile at d > 16 take the separate dot product (the product writes
its result itself).  Truncated solves in every precision on both sides of those
sizes against the oracle's FP64 CG (the FP32 bar of the existing inner-solve test,
2e-4 over 5 iterations; BF16 products carry 2^-9 per entry of q into every step, about
1e-2 over 5 steps, held to 1e-1).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1408_1237_amd import api, workloads
from parity import DT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-11), ("fp32", 2e-4), ("bf16", 1e-1)])
@pytest.mark.parametrize("n,d", [(1, 2), (200, 3), (257, 2), (4095, 3), (4096, 3), (4097, 3), (5000, 8), (250, 20),
                                 (3000, 20)])
def test_truncated_cg_matches_oracle(prec, bar, n, d):
    x = workloads.random_points(60 + n, n, d, 1.0, kind="normal")
    v = workloads.random_vector(61 + n, n)
    vt = torch.from_numpy(v).to(DT[prec]).cuda()
    sigma, shift, its = 0.5 * np.sqrt(d), 2.0, 5
    z, info = api.cg_inner_solve(torch.from_numpy(x).cuda(), sigma, shift, vt, its, prec=prec)
    want, _, iters, _, _ = oracle.cg(x, sigma, shift, vt.double().cpu().numpy(), its, 0.0, confirm=False)
    assert info["inner_iters"] == iters or n == 1
    z = z.double().cpu().numpy()
    assert np.linalg.norm(z - want) <= bar * np.linalg.norm(want)


@pytest.mark.parametrize("n", [2000, 4096, 4097])
def test_plain_cg_forms_agree_with_cholesky(n):
    x = workloads.random_points(70, n, 2, 1.0)
    y = workloads.random_vector(71, n)
    (w,), (info,) = api.krr_solve([torch.from_numpy(x).cuda()], [0.1], [0.1], [torch.from_numpy(y).cuda()], mode="cg64",
                                  tol=1e-10)
    assert info["status"] == 0 and 0.0 < info["lambda_min_est"] < info["lambda_max_est"]
    wd = oracle.direct_solve(x, 0.1, 0.1, y)
    assert np.linalg.norm(w.cpu().numpy() - wd) <= 1e-8 * np.linalg.norm(wd)
