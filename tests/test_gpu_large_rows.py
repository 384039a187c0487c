"""One-launch solves with several rows a thread: 896 rows a workgroup (two a
thread; 226,981 nodes, the elastic solve among them), 1280 (four; 314,432) and
2240 (eight, mixed only: FP64 stops at four and solves by launches; 571,787).

As for the smaller meshes, gspm_apply (a different kernel) recomputes the
residual: twice tol in FP64, whose recurrence follows the true residual to a
few per cent at 1e-9, tol in the mixed form.  The solution by launches meets
the same rule; one-launch results repeat bit for bit.
"""
import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

H, TOL = 4e-9, 1e-9
EPS = 2 * H * H


@pytest.fixture(scope="module", params=[62, 69, 84])
def case(request):
    n = request.param
    return w.small_cube(n, seed=500 + n, L=(n - 1) * H, jitter=0.15, sphere=0.2)


@pytest.mark.parametrize("precision", [gspm.GSPM_FP64, gspm.GSPM_MIXED])
def test_solves_meet_their_residual(case, precision):
    n = case.mesh.n_axis
    sim = gspm.Simulation(case.mesh, dict(case.params, gs_precond=gspm.GSPM_PRECOND_JACOBI), precision=precision)
    x0 = case.mesh.per_site(np.random.default_rng(n).standard_normal((case.mesh.n_sites, 3)))
    first = np.unique(case.mesh.site, return_index=True)[1]
    ops = [(gspm.GSPM_OP_GS, EPS), (gspm.GSPM_OP_MS, 0.0)] + ([(gspm.GSPM_OP_ELASTIC, 0.0)] if n == 62 else [])
    for op, eps in ops:
        b = np.ascontiguousarray(sim.apply(op, x0, eps=eps))
        b[:, 1] *= 1e-2                          # components stop apart
        if op == gspm.GSPM_OP_ELASTIC:
            b = np.ascontiguousarray(sim.apply(op, x0))
        for path in (gspm.GSPM_PATH_AUTO, gspm.GSPM_PATH_LAUNCHES):
            sim.set_solve_path(path)
            x, it = sim.solve(op, b, eps=eps, tol=TOL)
            assert sim.get_solve_path() == path
            r = (b - sim.apply(op, x, eps=eps))[first]
            for c in ([slice(0, 3)] if op == gspm.GSPM_OP_ELASTIC else [0, 1, 2]):
                rel = np.linalg.norm(r[:, c]) / np.linalg.norm(b[first, c])
                print(f"n={n} op={op} precision={precision} path={path}: residual {rel:.2e}, {it} iterations", flush=True)
                assert rel <= (2.0 if precision == gspm.GSPM_FP64 else 1.01) * TOL
            if path == gspm.GSPM_PATH_AUTO and (precision == gspm.GSPM_MIXED or n < 84):
                again, it2 = sim.solve(op, b, eps=eps, tol=TOL)
                assert it2 == it and np.array_equal(again, x)
    sim.close()
