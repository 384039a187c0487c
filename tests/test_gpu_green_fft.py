"""The elastic preconditioner's grid transforms over the lengths a grid can
have: primes (one stage), even and odd factors, squares and unequal axes.

B x is compared with the oracle's (plain DFTs, its own symbol) at the 1e-12
the preconditioner's other tests ask: both sides sum at most a few hundred
terms per axis in FP64.  The FP32 form is held to the FP64 solve: a mixed solve
must meet the same residual in at most one iteration more per FP32 inner solve
and refinement than the FP64 solve takes in all, which a wrong mode would not.
"""
import numpy as np
import pytest

import oracle as O
import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

H = 200e-9 / 46
# axis nodes and stretch per axis -> grid points per axis: 3, 4 = 2 2, 6, 9 = 3 3, 13, 19, 24 = 4 6, 31, 36 = 6 6;
# (17, 9, 7); (102, 51, 8);
# then two the bound does not hold for, on this path or the library's: a two-cell axis, whose neighbour is its own
# image, and cells of aspect 108, which the library transforms (planes beyond LDS) and the oracle resolve to 1.01e-12
CASES = [(4, (1, 1, 1)), (5, (1, 1, 1)), (7, (1, 1, 1)), (10, (1, 1, 1)), (14, (1, 1, 1)),
         (20, (1, 1, 1)), (25, (1, 1, 1)), (32, (1, 1, 1)), (37, (1, 1, 1)), (11, (1.8, 0.9, 0.7)),
         (35, (3, 1.5, 1 / 4.5)),
         pytest.param(3, (1, 1, 1), marks=pytest.mark.xfail(reason="images of a two-cell axis are ambiguous")),
         pytest.param(35, (6, 3, 1 / 18), marks=pytest.mark.xfail(reason="1.01e-12 with the library's transforms"))]


def _case(n, stretch):
    case = w.small_cube(n, seed=300 + n, L=(n - 1) * H, jitter=0.1)
    s = np.asarray(stretch, float)
    case.mesh.xyz = case.mesh.xyz * s
    case.mesh.hi = case.mesh.hi * s
    p = dict(case.params)
    p["elastic_precond"] = gspm.GSPM_PRECOND_GREEN
    return case, p


@pytest.mark.parametrize("n,stretch", CASES)
def test_preconditioner_over_grid_lengths(n, stretch):
    case, p = _case(n, stretch)
    orc = O.Oracle.from_mesh(case.mesh)
    orc.set_params(p)
    sim = gspm.Simulation(case.mesh, p)
    rng = np.random.default_rng(n)
    x = case.mesh.per_site(rng.standard_normal((case.mesh.n_sites, 3)))
    nmap = orc.node_map()
    xu = np.zeros((orc.n, 3))
    xu[nmap] = x
    y = sim.apply(gspm.GSPM_OP_PRECOND, x)
    ref = orc.precond_apply(xu)[nmap]
    err = np.abs(y - ref).max() / np.abs(ref).max()
    print(f"B x: grid {orc.precond_grid()}, max rel err {err:.2e}", flush=True)
    assert err < 1e-12
    assert np.array_equal(sim.apply(gspm.GSPM_OP_PRECOND, x), y)
    sim.close()


@pytest.mark.parametrize("n,stretch", [(5, (1, 1, 1)), (14, (1, 1, 1)), (25, (1, 1, 1)), (32, (1, 1, 1)),
                                       (11, (1.8, 0.9, 0.7)), (62, (1, 1, 1)),
                                       (82, (1, 1, 1))])    # 531441 nodes: several a thread in the prolongation
def test_fp32_transforms_precondition_as_fp64(n, stretch):
    case, p = _case(n, stretch)
    rng = np.random.default_rng(n + 1)
    b = 1e8 * H ** 2 * rng.standard_normal((case.mesh.n_sites, 3))
    b = case.mesh.per_site(b - b.mean(0))
    its = {}
    for prec in (gspm.GSPM_FP64, gspm.GSPM_MIXED):
        sim = gspm.Simulation(case.mesh, p, precision=prec)
        x, its[prec] = sim.solve(gspm.GSPM_OP_ELASTIC, b, tol=1e-8)
        if prec == gspm.GSPM_FP64:
            ref = x
        sim.close()
    err = np.linalg.norm(x - ref) / np.linalg.norm(ref)
    print(f"n={n} {stretch}: iterations FP64 {its[gspm.GSPM_FP64]} mixed {its[gspm.GSPM_MIXED]}, difference {err:.1e}",
          flush=True)
    assert its[gspm.GSPM_MIXED] <= its[gspm.GSPM_FP64] + 4
    assert err < 1e-6
