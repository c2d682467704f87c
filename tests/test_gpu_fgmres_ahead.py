"""FGMRES with the next inner solve enqueued before a step's status is read (GPU).

Under launch timing the solver reads every status first, so the two orders of the
same solve can be compared: the same kernels run on the same data, so the solution
and the counts are equal bit for bit, for solves that stop inside a cycle, at its
end, on the step limit and at once, with each kind of inner solve.
"""
import numpy as np
import pytest
import torch

from paper_1408_1237_amd import api, native, workloads

pytestmark = pytest.mark.gpu

CASES = [
    dict(),
    dict(inner_prec="fp64"),
    dict(inner_prec="bf16"),
    dict(inner="none"),
    dict(restart_m=1),
    dict(restart_m=3),
    dict(max_outer=1),
    dict(max_outer=5, restart_m=5),
    dict(max_outer=4, restart_m=3),
    dict(tol=0.5),
]


@pytest.mark.parametrize("kw", CASES, ids=lambda kw: "-".join("%s_%s" % i for i in kw.items()) or "default")
@pytest.mark.parametrize("n", [300, 9000])
def test_order_of_status_reads(n, kw):
    p = workloads.plain_small(n=n)
    x, b = torch.from_numpy(p.x).cuda(), torch.from_numpy(workloads.random_vector(31, n)).cuda()
    opts = dict(dict(tol=1e-6, max_outer=40, restart_m=10), **kw)
    run = lambda: api.fgmres_solve(x, p.sigma, p.gamma, b, **opts)  # noqa: E731
    w, info = run()
    with native.profile():
        w2, info2 = run()
    assert torch.equal(w, w2)
    for key in ("status", "outer_iters", "inner_iters", "cycles", "mvp64", "mvp32", "mvp16", "relres_true"):
        assert info[key] == info2[key], key
    assert info["outer_iters"] <= opts["max_outer"]
