"""Where a CG iteration's vector part changes from one block to three launches (GPU).

One block takes it up to 104 bytes of partial sums per entry: 4 tiles in FP64 and 13
in FP32 / BF16 up to d = 16, 13 and 16 tiles above (13 slots of 8 bytes; 4096
points).  Truncated solves on both sides against the oracle's FP64 CG, at the bars
of the other forms' test, and the time of an iteration, which must not be longer
at 12 tiles than at 17 (in one block it was, by a third).
"""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_1408_1237_amd import api, native, workloads
from parity import DT

pytestmark = pytest.mark.gpu

EDGES = [("fp64", 1024, 2), ("fp64", 1025, 2), ("fp64", 1280, 8), ("fp64", 3328, 20), ("fp64", 3329, 20),
         ("fp32", 3328, 3), ("fp32", 3329, 3), ("bf16", 3328, 8), ("bf16", 3329, 8), ("fp32", 4096, 20)]


@pytest.mark.parametrize("prec,n,d", EDGES)
def test_truncated_cg_at_the_edges(prec, n, d):
    x = workloads.random_points(80 + n, n, d, 1.0, kind="normal")
    vt = torch.from_numpy(workloads.random_vector(81 + n, n)).to(DT[prec]).cuda()
    sigma, shift, its = 0.5 * np.sqrt(d), 2.0, 5
    z, info = api.cg_inner_solve(torch.from_numpy(x).cuda(), sigma, shift, vt, its, prec=prec)
    want, _, iters, _, _ = oracle.cg(x, sigma, shift, vt.double().cpu().numpy(), its, 0.0, confirm=False)
    assert info["inner_iters"] == iters
    bar = {"fp64": 1e-11, "fp32": 2e-4, "bf16": 1e-1}[prec]
    assert np.linalg.norm(z.double().cpu().numpy() - want) <= bar * np.linalg.norm(want)


def test_iteration_time_across_the_edge():
    def iteration(n):
        x = torch.from_numpy(workloads.random_points(90, n, 2, 1.0)).cuda()
        v = torch.from_numpy(workloads.random_vector(91, n)).cuda()
        ws = api.workspace(native.workspace_size(native.KRR_WS_CG_INNER, [(n, 2)]), "cuda")

        def run(its):
            t0 = time.perf_counter()
            api.cg_inner_solve(x, 0.4, 1e-2, v, its, prec="fp64", ws=ws)
            torch.cuda.synchronize()
            return time.perf_counter() - t0

        run(210)
        return min(run(210) for _ in range(7)) - min(run(10) for _ in range(7))

    assert iteration(12 * 256) <= 1.1 * iteration(17 * 256)
