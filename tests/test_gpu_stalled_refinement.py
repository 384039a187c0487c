"""Mixed solves whose residual is below the range of FP32.

The inner solve of a refinement then starts from zeros, ends without an
iteration and leaves x as it was, and so would every refinement after it: the
solve has to end, with GSPM_E_NOCONV, however many iterations are left.  Inside
one launch (closed cells; GS and K^ms) and by launches (the elastic solve of a
cell with a cavity, and the preconditioned one) alike.  Near the edge of the
range, where some of the residual survives, a solve may also converge or meet a
non-finite scalar; it ends, and what it reports as solved is solved.
"""
import ctypes

import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

N, H, TOL = 8, 4e-9, 1e-9


def _case(cavity=False):
    case = w.small_cube(N, seed=61, L=(N - 1) * H, jitter=0.15)
    if cavity:
        plain = w.kuhn_cube(N, float(N - 1))
        keep = ~np.all(np.floor(plain.xyz[plain.tets].mean(1)).astype(int) == N // 2, axis=1)
        case.mesh.tets = np.ascontiguousarray(case.mesh.tets[keep])
        case.mesh.tags = np.ascontiguousarray(case.mesh.tags[keep])
    return case


def _solve(sim, op, b, eps, maxit=2000):
    x, it = np.zeros_like(b), ctypes.c_int32(0)
    st = gspm.load().gspm_solve(sim.ctx, op, eps, gspm._dp(b), gspm._dp(x), b.shape[0], TOL, maxit, ctypes.byref(it))
    return st, x, it.value


def _load(sim, case, op, eps, seed):
    x = case.mesh.per_site(np.random.default_rng(seed).standard_normal((case.mesh.n_sites, 3)))
    return np.ascontiguousarray(sim.apply(op, x, eps=eps))


CASES = [("one launch", gspm.GSPM_OP_ELASTIC, 0.0, False, False), ("one launch", gspm.GSPM_OP_MS, 0.0, False, False),
         ("one launch", gspm.GSPM_OP_GS, 2 * H * H, False, False),
         ("by launches", gspm.GSPM_OP_ELASTIC, 0.0, True, False),
         ("preconditioned", gspm.GSPM_OP_ELASTIC, 0.0, False, True)]


@pytest.mark.parametrize("form,op,eps,cavity,green", CASES)
def test_a_residual_below_fp32_ends_the_solve(form, op, eps, cavity, green):
    case = _case(cavity)
    p = dict(case.params)
    if green:
        p["elastic_precond"] = gspm.GSPM_PRECOND_GREEN
    sim = gspm.Simulation(case.mesh, p, precision=gspm.GSPM_MIXED)
    fresh = gspm.Simulation(case.mesh, p, precision=gspm.GSPM_MIXED)
    b = _load(sim, case, op, eps, 1)
    st, x, it = _solve(sim, op, b * 1e-100, eps)
    print(f"{form} op={op}: status {st}, {it} iterations: {gspm.gspm_last_error(sim.ctx)}", flush=True)
    assert st == gspm.GSPM_E_NOCONV and it == 0 and not np.any(x)
    # the context goes on as one that never failed
    st, x, _ = _solve(sim, op, b, eps)
    st2, x2, _ = _solve(fresh, op, b, eps)
    assert st == st2 == 0
    assert np.linalg.norm(x - x2) <= (0.0 if form == "one launch" else 1e-6) * np.linalg.norm(x2)
    sim.close()
    fresh.close()


def test_one_component_below_fp32():
    """Two components converge, the third cannot: the call ends and the two are solved."""
    case = _case()
    eps = 2 * H * H
    sim = gspm.Simulation(case.mesh, case.params, precision=gspm.GSPM_MIXED)
    b = _load(sim, case, gspm.GSPM_OP_GS, eps, 2)
    b[:, 2] *= 1e-100
    st, x, it = _solve(sim, gspm.GSPM_OP_GS, b, eps)
    r = b - sim.apply(gspm.GSPM_OP_GS, x, eps=eps)
    assert st == gspm.GSPM_E_NOCONV and 0 < it < 2000
    for c in (0, 1):
        assert np.linalg.norm(r[:, c]) <= 1.01 * TOL * np.linalg.norm(b[:, c])
    sim.close()


@pytest.mark.parametrize("form,op,eps,cavity,green", CASES)
def test_solves_end_through_the_edge_of_the_range(form, op, eps, cavity, green):
    case = _case(cavity)
    p = dict(case.params)
    if green:
        p["elastic_precond"] = gspm.GSPM_PRECOND_GREEN
    sim = gspm.Simulation(case.mesh, p, precision=gspm.GSPM_MIXED)
    b = _load(sim, case, op, eps, 3)
    # FP32 residuals of about 1e-34 (x of order one has scaled residuals between 1e-2 and 1e18 for these operators) down
    for e in range(-60, -28, 4):
        st, x, it = _solve(sim, op, b * 10.0 ** e, eps)
        print(f"{form} op={op} 1e{e}: status {st}, {it} iterations", flush=True)
        assert st in (0, gspm.GSPM_E_NOCONV, gspm.GSPM_E_NONFINITE)
        if st == 0 and not green:
            r = b * 10.0 ** e - sim.apply(op, x, eps=eps)
            first = np.unique(case.mesh.site, return_index=True)[1]
            assert np.linalg.norm(r[first]) <= 1.01 * np.sqrt(3.0) * TOL * np.linalg.norm(b[first] * 10.0 ** e)
    sim.close()
