"""Cells that their elements do not fill: a cavity, a slab that leaves a gap
along one axis, and a body that touches no max face of its box.

On a closed cell of one stiffness the 3x3 blocks of K^mech are symmetric
(integration by parts leaves no boundary term), and the one-launch elastic
solve stores six numbers for each.  A free surface breaks that: blocks of the
surface's edges differ from their transposes by the area it cuts, so these
meshes must be solved with the elements.  Every solve is held to its own
stopping rule by gspm_apply, which evaluates the operator element by element:
the recomputed ||b - A x|| may exceed tol ||b|| by the drift of the FP64
recurrence only, a few per cent at 1e-9, so twice tol is allowed; in the mixed
form the last test is on the true residual.  Whole steps are compared with the
oracle, which assembles from the elements, at the 1e-9 of the parity tests.
"""
import numpy as np
import pytest

import oracle as O
import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

TOL = 1e-9
H = 4e-9


def _lattice_cells(n):
    """The lattice cell of every tetrahedron of an n-node Kuhn cube."""
    plain = w.kuhn_cube(n, float(n - 1))
    return np.floor(plain.xyz[plain.tets].mean(1)).astype(int)


def _open_case(kind, n, sphere=0.0):
    case = w.small_cube(n, seed=40 + n, L=(n - 1) * H, jitter=0.15, sphere=sphere)
    mesh, cell = case.mesh, _lattice_cells(n)
    if kind == "cavity":
        keep = ~np.all(cell == n // 2, axis=1)
    elif kind == "slab":                       # one layer of cells left out: free surfaces across z
        keep = cell[:, 2] != n // 2
    else:                                      # "body": the box is larger than the mesh
        keep = np.ones(len(cell), bool)
        mesh.hi = mesh.hi + 0.5 * H
        mesh.site = np.arange(mesh.n_nodes)
    mesh.tets, mesh.tags = np.ascontiguousarray(mesh.tets[keep]), np.ascontiguousarray(mesh.tags[keep])
    return case


def _field(case, rng):
    site = case.mesh.site
    return np.ascontiguousarray(rng.standard_normal((site.max() + 1, 3))[site])


@pytest.mark.parametrize("precision", [gspm.GSPM_FP64, gspm.GSPM_MIXED])
@pytest.mark.parametrize("op", [gspm.GSPM_OP_ELASTIC, gspm.GSPM_OP_MS])
@pytest.mark.parametrize("kind,n", [("cavity", 7), ("cavity", 20), ("slab", 10), ("body", 9)])
def test_solves_meet_their_residual(kind, n, op, precision):
    case = _open_case(kind, n)
    sim = gspm.Simulation(case.mesh, case.params, precision=precision)
    b = sim.apply(op, _field(case, np.random.default_rng(n)))
    x, it = sim.solve(op, b, tol=TOL)
    r = b - sim.apply(op, x)
    first = np.unique(case.mesh.site, return_index=True)[1]
    for c in ([slice(0, 3)] if op == gspm.GSPM_OP_ELASTIC else [0, 1, 2]):
        rel = np.linalg.norm(r[first, c]) / np.linalg.norm(b[first, c])
        print(f"{kind} n={n} op={op} precision={precision}: residual {rel:.2e}, {it} iterations", flush=True)
        assert rel <= (2.0 if precision == gspm.GSPM_FP64 else 1.01) * TOL
    sim.close()


@pytest.mark.parametrize("kind", ["cavity", "slab"])
def test_steps_match_the_oracle(kind):
    case = _open_case(kind, 8, sphere=0.3)
    p = dict(case.params, cg_tol=1e-12)
    hext = (2e5, 0.0, 0.0)
    sim = gspm.Simulation(case.mesh, p, hext=hext)
    sim.set_m(case.m0)
    sim.step(2e-12, 3)
    orc = O.Oracle.from_mesh(case.mesh)
    orc.set_params(p, hext=hext)
    orc.set_m(case.m0)
    orc.step(2e-12, 3)
    m, u, mr, ur = sim.get_m(), sim.get_u(), orc.get_m(), orc.get_u()
    em = np.linalg.norm(m - mr) / np.linalg.norm(mr)
    eu = np.linalg.norm(u - ur) / np.linalg.norm(ur)
    print(f"{kind}: m {em:.1e} u {eu:.1e}", flush=True)
    assert em < 1e-9 and eu < 1e-9
    sim.close()


def test_a_new_mesh_is_looked_at_anew():
    """Closed, open, closed on one context: each upload decides for itself."""
    closed = w.small_cube(9, seed=49, L=8 * H, jitter=0.15)
    opened = _open_case("cavity", 9)
    sim = gspm.Simulation(closed.mesh, closed.params)
    for case in (closed, opened, closed):
        gspm.gspm_upload_mesh(sim.ctx, case.mesh.xyz, case.mesh.tets, case.mesh.tags, case.mesh.lo, case.mesh.hi)
        sim.set_params(case.params)
        b = sim.apply(gspm.GSPM_OP_ELASTIC, _field(case, np.random.default_rng(3)))
        x, _ = sim.solve(gspm.GSPM_OP_ELASTIC, b, tol=TOL)
        assert np.linalg.norm(b - sim.apply(gspm.GSPM_OP_ELASTIC, x)) <= 2.0 * TOL * np.linalg.norm(b)
    sim.close()
