"""Mixed solves whose start is already the solution: after one of a kind, the next
start of that kind is tested before a one-launch solve is made of it.  The
answers stay those of the full path: no iteration and x untouched while the
start holds, zero where the right-hand side is zero, a full solve (bit for bit
that of a context that never rested) as soon as it does not, the recorded
residual of a step, and errors."""
import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

H = 4e-9
EPS = 2 * H * H


@pytest.mark.parametrize("op,eps", [(gspm.GSPM_OP_GS, EPS), (gspm.GSPM_OP_ELASTIC, 0.0), (gspm.GSPM_OP_MS, 0.0)])
@pytest.mark.parametrize("n", [9, 24])
def test_rest_and_departure(n, op, eps):
    case = w.small_cube(n, seed=70 + n, L=(n - 1) * H, jitter=0.15)
    sim, other = (gspm.Simulation(case.mesh, case.params, precision=gspm.GSPM_MIXED) for _ in range(2))
    rng = np.random.default_rng(n)
    b = np.ascontiguousarray(sim.apply(op, case.mesh.per_site(rng.standard_normal((case.mesh.n_sites, 3))), eps=eps))
    b2 = np.ascontiguousarray(sim.apply(op, case.mesh.per_site(rng.standard_normal((case.mesh.n_sites, 3))), eps=eps))
    x, it = sim.solve(op, b, eps=eps, tol=1e-10)
    assert it > 0
    for _ in range(3):
        y, it = sim.solve(op, b, x0=x, eps=eps, tol=1e-8)
        assert it == 0 and np.array_equal(y, x)
    z, it = sim.solve(op, b2, x0=x, eps=eps, tol=1e-9)            # no longer at rest
    ref, it2 = other.solve(op, b2, x0=x, eps=eps, tol=1e-9)
    assert it == it2 > 0 and np.array_equal(z, ref)
    sim.solve(op, b, x0=x, eps=eps, tol=1e-8)
    y, it = sim.solve(op, np.zeros_like(b), x0=x, eps=eps, tol=1e-8)
    assert it == 0 and not np.any(y)
    if op != gspm.GSPM_OP_ELASTIC:                                # one component at rest, another not
        mixed_b = b.copy()
        mixed_b[:, 2] = b2[:, 2]
        sim.solve(op, b, x0=x, eps=eps, tol=1e-8)
        z, it = sim.solve(op, mixed_b, x0=x, eps=eps, tol=1e-8)
        ref, it2 = other.solve(op, mixed_b, x0=x, eps=eps, tol=1e-8)
        assert it == it2 > 0 and np.array_equal(z, ref)
    for s in (sim, other):
        s.close()


def test_steps_that_come_to_rest():
    """A noisy state along the field relaxes around an inclusion; the solves of its last steps start converged in part.  Every residual is
    reported and below tol, and the run ends where one by launches ends (both solve to 1e-8)."""
    case = w.small_cube(9, seed=3, L=8 * H, jitter=0.1, sphere=0.3, m="noisy")
    out = []
    for path in (gspm.GSPM_PATH_AUTO, gspm.GSPM_PATH_LAUNCHES):
        sim = gspm.Simulation(case.mesh, dict(case.params, alpha=0.5), hext=(5e5, 0.0, 0.0), precision=gspm.GSPM_MIXED,
                              local_demag=True)
        sim.set_solve_path(path)
        sim.set_gs_start(gspm.GSPM_GS_START_CORRECTED)
        sim.set_m(case.m0)
        first = sim.step(5e-12, 1)["gs_iters"]
        for _ in range(8):
            st = sim.step(5e-12, 50)
            res = st["final_residual"]
            assert all(0.0 <= v <= 1e-8 for v in (res.values() if isinstance(res, dict) else res))
        print(f"path {path}: GS iterations {first} in the first step, {st['gs_iters'] / 50} a step at the end", flush=True)
        assert st["gs_iters"] / 50 < first
        out.append((sim.get_m(), sim.get_u()))
        sim.close()
    (m, u), (mr, ur) = out
    assert np.linalg.norm(m - mr) <= 1e-6 * np.linalg.norm(mr) and np.linalg.norm(u - ur) <= 1e-5 * np.linalg.norm(ur)
