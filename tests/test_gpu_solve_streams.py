"""Solves beside other streams and threads (GPU).

A solve synchronises its own stream only: it returns while another stream still
works.  Solves on several threads and streams at once borrow their host status
copies from one array and give the solutions of the same solves one by one, bit
for bit.
"""
import threading
import time

import numpy as np
import pytest
import torch

from paper_1408_1237_amd import api, native, workloads

pytestmark = pytest.mark.gpu


def _problem(n, seed):
    p = workloads.plain_small(n=n)
    return torch.from_numpy(p.x).cuda(), p.sigma, p.gamma, torch.from_numpy(workloads.random_vector(seed, n)).cuda()


def test_solve_returns_beside_a_busy_stream():
    x, sigma, gamma, y = _problem(1000, 1)
    solve = lambda: api.fgmres_solve(x, sigma, gamma, y, tol=1e-4)  # noqa: E731
    solve()  # the first one also tunes
    torch.cuda.synchronize()
    t0 = time.time()
    solve()
    alone = time.time() - t0
    n = 100_000
    xb = torch.rand((n, 16), dtype=torch.float64, device="cuda")
    q = torch.randn(n, dtype=torch.float64, device="cuda")
    ws = api.workspace(native.workspace_size(native.KRR_WS_KMVP, [(n, 16)]), "cuda")
    product = lambda: api.kmvp_gauss(xb, 1.0, q, ws=ws)  # noqa: E731
    product()
    torch.cuda.synchronize()
    t0 = time.time()
    product()
    torch.cuda.synchronize()
    one = time.time() - t0
    # the solve shares the card with the products: it may take several times as long
    busy, done = torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(busy):
        for _ in range(int(max(2.0, 20 * alone) / one)):
            product()
        done.record()
    with torch.cuda.stream(torch.cuda.Stream()):
        solve()
    still = not done.query()
    torch.cuda.synchronize()
    assert still


def test_solves_on_several_threads():
    probs = [_problem(400 + 300 * k, 10 + k) for k in range(4)]
    opts = dict(tol=1e-8, max_outer=60)
    want = [api.fgmres_solve(*p, **opts)[0] for p in probs]
    torch.cuda.synchronize()
    got = [[] for _ in probs]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(5):
                got[k].append(api.fgmres_solve(*probs[k], **opts)[0].cpu().numpy())

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(probs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k, w in enumerate(want):
        assert len(got[k]) == 5
        for g in got[k]:
            assert np.array_equal(g, w.cpu().numpy())
