"""One-launch solves of contexts in threads of their own, and beside other work
on the device: each wants a workgroup on every CU and its workgroups wait for
each other, so launches that got half of the device each would wait for good.
Results are those of the same solves one after another, bit for bit, and no
wait runs out."""
import threading

import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

H, TOL = 4e-9, 1e-9


def _work(n, seed, precision):
    case = w.small_cube(n, seed=seed, L=(n - 1) * H, jitter=0.15)
    sim = gspm.Simulation(case.mesh, case.params, precision=precision)
    x = case.mesh.per_site(np.random.default_rng(seed).standard_normal((case.mesh.n_sites, 3)))
    loads = [(op, eps, np.ascontiguousarray(sim.apply(op, x, eps=eps)))
             for op, eps in ((gspm.GSPM_OP_ELASTIC, 0.0), (gspm.GSPM_OP_GS, 2 * H * H), (gspm.GSPM_OP_MS, 0.0))]
    return sim, loads


def _solve_all(sim, loads, out):
    for op, eps, b in loads:
        out.append(sim.solve(op, b, eps=eps, tol=TOL))


@pytest.mark.parametrize("sizes", [(47, 47), (47, 11, 24)])
def test_contexts_in_threads(sizes):
    work = [_work(n, 900 + k, (gspm.GSPM_FP64, gspm.GSPM_MIXED)[k % 2]) for k, n in enumerate(sizes)]
    alone = [[] for _ in work]
    for (sim, loads), out in zip(work, alone):
        _solve_all(sim, loads, out)
    for _ in range(3):
        together = [[] for _ in work]
        threads = [threading.Thread(target=_solve_all, args=(sim, loads, out)) for (sim, loads), out in zip(work, together)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for (sim, _), a, b in zip(work, alone, together):
            assert sim.get_solve_path() == gspm.GSPM_PATH_AUTO
            assert len(a) == len(b)
            for (xa, ia), (xb, ib) in zip(a, b):
                assert ia == ib and np.array_equal(xa, xb)
    for sim, _ in work:
        sim.close()


def test_beside_other_work():
    import torch
    sim, loads = _work(47, 950, gspm.GSPM_MIXED)
    alone, beside = [], []
    _solve_all(sim, loads, alone)
    a = torch.randn(4096, 4096, device="cuda", dtype=torch.bfloat16)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for _ in range(200):
            c = a @ a
    _solve_all(sim, loads, beside)
    torch.cuda.synchronize()
    assert torch.isfinite(c.float()).all()
    assert sim.get_solve_path() == gspm.GSPM_PATH_AUTO
    for (xa, ia), (xb, ib) in zip(alone, beside):
        assert ia == ib and np.array_equal(xa, xb)
    sim.close()
