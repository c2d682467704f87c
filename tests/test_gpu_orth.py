"""Orthogonalisation of short and long vectors, and small batched work items (GPU).

Up to 8192 padded points one block does a whole Arnoldi orthogonalisation with its
Givens step; above, one launch per basis vector.  Both forms, modified and
twice-classical Gram-Schmidt, in the single and the batched solver, on both
sides of that size: the true residual (oracle, FP64) meets the tolerance, and the
step counts of neighbouring sizes and of the two Gram-Schmidt forms agree
closely (the same Arnoldi process up to rounding).  Small systems of a batch are
cut down to single column tiles; every cut gives the same solution up to the
solver's tolerance.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1408_1237_amd import api, workloads

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _problem(n, seed=5):
    x = workloads.random_points(seed, n, 3, 1.0, kind="normal")
    return x, workloads.random_vector(seed + 1, n), 1.2, 0.05


@pytest.mark.parametrize("n", [1, 2, 255, 257, 8192, 8193])
def test_single_solver_both_orthogonalisations(n):
    x, y, sigma, gamma = _problem(n)
    steps = {}
    for gs in ("mgs", "cgs2"):
        w, info = api.fgmres_solve(_t(x), sigma, gamma, _t(y), gs=gs, restart_m=60, inner_maxit=20, tol=1e-8)
        assert info["status"] == 0
        assert oracle.true_relres(x, sigma, gamma, y, w.cpu().numpy()) <= 1e-8
        steps[gs] = info["outer_iters"]
    assert abs(steps["mgs"] - steps["cgs2"]) <= 2, steps


@pytest.mark.parametrize("gs", ["mgs", "cgs2"])
@pytest.mark.parametrize("sizes", [(300, 8192), (300, 8193), (40, 1)])
def test_batched_solver_both_forms(gs, sizes):
    probs = [_problem(n, seed=20 + k) for k, n in enumerate(sizes)]
    ys = [np.asfortranarray(np.stack([p[1], p[1][::-1]], 1)) for p in probs]
    Ws, infos = api.krr_solve([_t(p[0]) for p in probs], [p[2] for p in probs], [p[3] for p in probs],
                              [torch.from_numpy(np.ascontiguousarray(y.T)).cuda().t() for y in ys], gs=gs,
                              restart_m=60, inner_maxit=20, tol=1e-8)
    assert all(i["status"] == 0 for i in infos)
    for p, y, W in zip(probs, ys, Ws):
        for r in range(2):
            yr = np.ascontiguousarray(y[:, r])
            assert oracle.true_relres(p[0], p[2], p[3], yr, W.cpu().numpy()[:, r]) <= 1e-8


@pytest.mark.parametrize("n,d,nrhs", [(200, 2, 1), (1100, 4, 17), (4200, 8, 3), (9000, 3, 2)])
def test_small_systems_cut_into_items(monkeypatch, n, d, nrhs):
    x = workloads.random_points(31, n, d, 1.0, kind="normal")
    Y = workloads.random_vector(32, n, nrhs)
    Yt = torch.from_numpy(np.ascontiguousarray(Y.T)).cuda().t()
    for tps in ("16", "128"):
        monkeypatch.setenv("KRR_BATCH_TPS", tps)
        for mode in ("fgmres", "cg64"):
            (W,), infos = api.krr_solve([_t(x), ], [np.sqrt(d)], [0.1], [Yt], mode=mode, tol=1e-8, inner_maxit=20)
            assert all(i["status"] == 0 for i in infos)
            for r in (0, nrhs - 1):
                yr = np.ascontiguousarray(Y[:, r])
                wr = W.reshape(n, -1).cpu().numpy()[:, r]
                assert oracle.true_relres(x, np.sqrt(d), 0.1, yr, wr) <= 1e-8
    monkeypatch.delenv("KRR_BATCH_TPS")
