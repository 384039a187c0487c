"""Solves that run in one launch (a workgroup per CU, halo and sums exchanged
inside the kernel), at the sizes where their split changes.

A mesh of N unique nodes is dealt out in blocks of 64 k rows to at most one
workgroup per CU; 64 rows take eight lanes each, 256 take two, 512 one, and
larger blocks two to eight rows per thread.  Up to 16 workgroups read each
other's sums directly, more of them through leaders.  The sizes below lie on
both sides of these edges, with ragged last blocks, a last block of a single
row, inclusions (rows without entries), node orders whose halo lists are longer
than a launch polls at once, and valences above and below the 14 neighbours
whose coefficients stay in registers.

Each solve is held to its own stopping rule by the operator as gspm_apply
evaluates it (a different kernel): the recomputed ||b - A x|| may exceed
tol ||b|| by the rounding of FP64 residuals, which is far below tol here; CG in
FP64 tests the recurrence's residual, which follows the true one to a few per
cent at these tolerances, so twice tol is allowed.  Results repeat bit for bit.
"""
import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

TOL = 1e-9
# axis nodes -> unique nodes: 5 -> 64 (one full block), 6 -> 125 (a block and 61 rows), 9 -> 512, 17 -> 4096 (64
# blocks of 64, four leaders), 18 -> 4913, 25 -> 13824, 27 -> 17576 (blocks of 128), 35 -> 39304, 48 -> 103823, 53 -> 140608 (two rows per thread)
CASES = [(5, "kuhn", 0.0, gspm.GSPM_REORDER_MORTON), (6, "kuhn", 0.0, gspm.GSPM_REORDER_MORTON),
         (9, "kuhn", 0.3, gspm.GSPM_REORDER_MORTON), (17, "kuhn", 0.0, gspm.GSPM_REORDER_MORTON),
         (18, "kuhn", 0.3, gspm.GSPM_REORDER_NONE), (19, "five", 0.25, gspm.GSPM_REORDER_MORTON),
         (25, "five", 0.0, gspm.GSPM_REORDER_RCM), (27, "kuhn", 0.3, gspm.GSPM_REORDER_MORTON),
         (35, "kuhn", 0.0, gspm.GSPM_REORDER_NONE), (48, "kuhn", 0.3, gspm.GSPM_REORDER_MORTON),
         (53, "kuhn", 0.2, gspm.GSPM_REORDER_MORTON)]


def _setup(n, split, sphere, reorder, precision, precond):
    case = w.small_cube(n, seed=100 + n, L=n * 4e-9, jitter=0.15, sphere=sphere, shuffle=n % 2 == 0, split=split)
    params = case.params
    if precond:
        params["gs_precond"] = gspm.GSPM_PRECOND_JACOBI
    sim = gspm.Simulation(case.mesh, params, precision=precision, reorder=reorder)
    return case, sim


def _load(case, sim, op, eps, rng):
    """A right-hand side in the operator's range: A applied to a random periodic field."""
    x = case.mesh.per_site(rng.standard_normal((case.mesh.n_sites, 3)))
    return np.ascontiguousarray(sim.apply(op, x, eps=eps))


@pytest.mark.parametrize("precision", [gspm.GSPM_FP64, gspm.GSPM_MIXED])
@pytest.mark.parametrize("n,split,sphere,reorder", CASES)
def test_gs_solve_meets_its_residual(n, split, sphere, reorder, precision):
    case, sim = _setup(n, split, sphere, reorder, precision, precond=n % 3 != 0)
    rng = np.random.default_rng(n)
    eps = 2.0 * (4e-9) ** 2
    b = _load(case, sim, gspm.GSPM_OP_GS, eps, rng)
    b[:, 2] *= 1e-3                       # components of different size stop at different iterations
    x, it = sim.solve(gspm.GSPM_OP_GS, b, eps=eps, tol=TOL)
    r = b - sim.apply(gspm.GSPM_OP_GS, x, eps=eps)
    site = case.mesh.site
    first = np.unique(site, return_index=True)[1]
    for c in range(3):
        rel = np.linalg.norm(r[first, c]) / np.linalg.norm(b[first, c])
        print(f"n={n} {split} precision={precision} component {c}: residual {rel:.2e}, {it} iterations", flush=True)
        assert rel <= (2.0 if precision == gspm.GSPM_FP64 else 1.01) * TOL
    again, it2 = sim.solve(gspm.GSPM_OP_GS, b, eps=eps, tol=TOL)
    assert it2 == it and np.array_equal(again, x)
    sim.close()


@pytest.mark.parametrize("precision", [gspm.GSPM_FP64, gspm.GSPM_MIXED])
@pytest.mark.parametrize("op", [gspm.GSPM_OP_ELASTIC, gspm.GSPM_OP_MS])
@pytest.mark.parametrize("n,split,sphere,reorder", CASES)
def test_pinned_solves_meet_their_residual(n, split, sphere, reorder, op, precision):
    """K^mech (3x3 blocks) and K^ms (scalar) over all elements: the rows are
    assembled for these solves, gspm_apply evaluates the operators element by
    element, so this also compares the two forms."""
    case, sim = _setup(n, split, sphere, reorder, precision, precond=False)
    rng = np.random.default_rng(n + 1)
    b = _load(case, sim, op, 0.0, rng)
    x, it = sim.solve(op, b, tol=TOL)
    r = b - sim.apply(op, x)
    first = np.unique(case.mesh.site, return_index=True)[1]
    cols = [slice(0, 3)] if op == gspm.GSPM_OP_ELASTIC else [0, 1, 2]
    for c in cols:
        rel = np.linalg.norm(r[first, c]) / np.linalg.norm(b[first, c])
        print(f"n={n} {split} op={op} precision={precision}: residual {rel:.2e}, {it} iterations", flush=True)
        assert rel <= (2.0 if precision == gspm.GSPM_FP64 else 1.01) * TOL
    again, it2 = sim.solve(op, b, tol=TOL)
    assert it2 == it and np.array_equal(again, x)
    sim.close()


def test_rotated_stiffness_rows_follow_set_params():
    """The rows of K^mech are rebuilt when the stiffness changes, and only then."""
    r111 = np.array([[1, 1, 1], [1, -1, 0], [1, 1, -2]]) / np.sqrt([[3.0], [2.0], [6.0]])
    case, sim = _setup(12, "kuhn", 0.25, gspm.GSPM_REORDER_MORTON, gspm.GSPM_FP64, precond=False)
    rng = np.random.default_rng(7)
    for rot, hx in ((None, 0.0), (r111, 0.0), (r111, 1e5), (None, 1e5)):
        params = case.params
        if rot is not None:
            params["crystal_rot"] = rot
        sim.set_params(params, hext=(hx, 0.0, 0.0))
        b = _load(case, sim, gspm.GSPM_OP_ELASTIC, 0.0, rng)
        x, it = sim.solve(gspm.GSPM_OP_ELASTIC, b, tol=TOL)
        r = b - sim.apply(gspm.GSPM_OP_ELASTIC, x)
        assert it > 0 and np.linalg.norm(r) <= 2.0 * TOL * np.linalg.norm(b)
    sim.close()


# axis nodes -> unique nodes: 11 -> 1000 (16 blocks of 64: one hop), 12 -> 1331 (11 of 128), 13 -> 1728, 14 -> 2197 (35 of
# 64: a third leader with three), 26 -> 15625 (245), 33 -> 32768 (256 of 128), 34 -> 35937 (188 of 192: two lanes a row)
@pytest.mark.parametrize("precision", [gspm.GSPM_FP64, gspm.GSPM_MIXED])
@pytest.mark.parametrize("n", [11, 12, 13, 14, 26, 33, 34])
def test_hops_and_lanes(n, precision):
    case, sim = _setup(n, "kuhn", 0.0, gspm.GSPM_REORDER_MORTON, precision, precond=False)
    rng = np.random.default_rng(n + 2)
    b = _load(case, sim, gspm.GSPM_OP_ELASTIC, 0.0, rng)
    x, _ = sim.solve(gspm.GSPM_OP_ELASTIC, b, tol=TOL)
    sites = np.unique(case.mesh.per_site(np.arange(case.mesh.n_sites, dtype=float)[:, None] + np.zeros((1, 3)))[:, 0],
                      return_index=True)[1]
    r = (b - sim.apply(gspm.GSPM_OP_ELASTIC, x))[sites]
    held = np.any(x[sites] != 0, axis=1)          # the pinned node has no equation
    assert np.count_nonzero(~held) <= 1
    assert np.linalg.norm(r[held]) <= 2 * TOL * np.linalg.norm(b[sites][held])
    again, _ = sim.solve(gspm.GSPM_OP_ELASTIC, b, tol=TOL)
    assert np.array_equal(again, x)
    sim.close()
