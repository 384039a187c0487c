"""Solves whose workgroups give up waiting for each other, and the switch
between the two ways a solve runs.

The longest wait of a one-launch solve is set from the host.  Bounds around the
few microseconds that an exchange takes make some waits run out and others not,
in any workgroup and round, so that launches end with workgroups that stored
their rows and others that did not.  Whatever they did, the call has to return
a solution that meets its stopping rule by gspm_apply (twice tol in FP64, whose
recurrence follows the true residual to a few per cent at 1e-9), and the
context has to say that it solves by launches from then on.
"""
import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

H, TOL = 4e-9, 1e-9
EPS = 2 * H * H
OPS = [(gspm.GSPM_OP_ELASTIC, 0.0), (gspm.GSPM_OP_MS, 0.0), (gspm.GSPM_OP_GS, EPS)]


def _sim(n, precision, **kw):
    shuffled = n == 35
    if shuffled:
        kw["reorder"] = gspm.GSPM_REORDER_NONE
    case = w.small_cube(n, seed=80 + n, L=(n - 1) * H, jitter=0.15, shuffle=shuffled)
    return case, gspm.Simulation(case.mesh, case.params, precision=precision, **kw)


def _load(sim, case, op, eps):
    x = case.mesh.per_site(np.random.default_rng(op).standard_normal((case.mesh.n_sites, 3)))
    return np.ascontiguousarray(sim.apply(op, x, eps=eps))


def _check(sim, case, op, eps, b, x, precision):
    first = np.unique(case.mesh.site, return_index=True)[1]
    r = (b - sim.apply(op, x, eps=eps))[first]
    for c in ([slice(0, 3)] if op == gspm.GSPM_OP_ELASTIC else [0, 1, 2]):
        rel = np.linalg.norm(r[:, c]) / np.linalg.norm(b[first, c])
        assert rel <= (2.0 if precision == gspm.GSPM_FP64 else 1.01) * TOL, (op, c, rel)


# 16 workgroups (one hop), 64 (leaders), 250; then 205 of 192 rows in shuffled order, whose 2500 halo nodes are more than
# a launch fetches before the sums (in FP64 they do not fit LDS)
@pytest.mark.parametrize("n,precision", [(11, gspm.GSPM_FP64), (11, gspm.GSPM_MIXED), (17, gspm.GSPM_FP64),
                                         (17, gspm.GSPM_MIXED), (41, gspm.GSPM_FP64), (41, gspm.GSPM_MIXED),
                                         (35, gspm.GSPM_MIXED)])
def test_a_wait_that_runs_out_costs_no_accuracy(n, precision):
    case, sim = _sim(n, precision)
    loads = [(op, eps, _load(sim, case, op, eps)) for op, eps in OPS]
    gave_up = kept = 0
    for wait in (1e-8, 2e-7, 5e-7, 1e-6, 1.5e-6, 2e-6, 3e-6, 4e-6, 6e-6, 8e-6):
        for op, eps, b in loads:
            sim.set_solve_path(gspm.GSPM_PATH_AUTO, wait)
            assert sim.get_solve_path() == gspm.GSPM_PATH_AUTO
            x, _ = sim.solve(op, b, eps=eps, tol=TOL)
            up = sim.get_solve_path() == gspm.GSPM_PATH_GAVE_UP
            gave_up += up
            kept += not up
            _check(sim, case, op, eps, b, x, precision)
    print(f"n={n} precision={precision}: gave up {gave_up}, kept {kept}", flush=True)
    assert gave_up > 0                      # 10 ns is below any exchange
    # back to one launch: the buffers are in step again and results repeat those of a context that never gave up
    sim.set_solve_path(gspm.GSPM_PATH_AUTO)
    other = _sim(n, precision)[1]
    for op, eps, b in loads:
        x, it = sim.solve(op, b, eps=eps, tol=TOL)
        ref, it2 = other.solve(op, b, eps=eps, tol=TOL)
        assert it == it2 and np.array_equal(x, ref)
    assert sim.get_solve_path() == gspm.GSPM_PATH_AUTO
    sim.close()
    other.close()


def test_steps_go_on_by_launches():
    """A step whose solves give up ends as one that runs by launches throughout."""
    out = []
    for wait in (0.0, 1e-8):
        case, sim = _sim(12, gspm.GSPM_FP64, hext=(2e5, 0.0, 0.0), local_demag=True)
        sim.set_solve_path(gspm.GSPM_PATH_AUTO if wait else gspm.GSPM_PATH_LAUNCHES, wait)
        sim.set_m(case.m0)
        sim.step(1e-12, 3)
        assert sim.get_solve_path() == (gspm.GSPM_PATH_GAVE_UP if wait else gspm.GSPM_PATH_LAUNCHES)
        out.append((sim.get_m(), sim.get_u(), sim.get_ud()))
        sim.close()
    for a, b in zip(*out):
        # both solve to the configured 1e-8 from different starts
        assert np.linalg.norm(a - b) <= 1e-6 * np.linalg.norm(b)


def test_switch_arguments():
    case, sim = _sim(5, gspm.GSPM_FP64)
    for path, wait in ((2, 0.0), (-1, 0.0), (0, -1.0), (0, float("nan")), (0, 1e9)):
        with pytest.raises(gspm.GspmError) as e:
            sim.set_solve_path(path, wait)
        assert e.value.status == gspm.GSPM_E_ARG
    sim.set_solve_path(gspm.GSPM_PATH_LAUNCHES)
    gspm.gspm_upload_mesh(sim.ctx, case.mesh.xyz, case.mesh.tets, case.mesh.tags, case.mesh.lo, case.mesh.hi)
    assert sim.get_solve_path() == gspm.GSPM_PATH_LAUNCHES     # the caller's choice outlives the mesh
    sim.close()
