"""The elastic preconditioner on grids that the library transforms (with
k_pc_modes and the symbol by mode): planes that do not fit LDS, powers of 2, 3
or 5, and films and rods whose few planes or columns leave the own transforms
on few workgroups; and grids next to those that take the own transforms.

Films, rods and cubes on both sides of the choice: B x against the oracle's
plain DFTs at the 1e-12 of the preconditioner's other tests.

FP64, B x against the oracle on a 204 x 102 x 2 grid of cells of aspect 108:
the symbol of a mode along the long edges is that much stiffer across them, so
its inverse carries the rounding of the stencil times the aspect squared, 2^-53
x 108^2 = 1.3e-12 on each side; the bound is 3e-12.

FP32, on a 144 x 144 x 11 grid (167 kB a plane) over cells as compact as those
of the cubes, which take 15 to 20 iterations to 1e-8: FP64 must stay below 24,
and the mixed solve meet its solution in at most four iterations more (one an
inner solve and refinement), which a wrong mode would not.
"""
import numpy as np
import pytest

import oracle as O
import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

H = 200e-9 / 46


def _case(n, stretch):
    case = w.small_cube(n, seed=300 + n, L=(n - 1) * H, jitter=0.1)
    s = np.asarray(stretch, float)
    case.mesh.xyz = case.mesh.xyz * s
    case.mesh.hi = case.mesh.hi * s
    return case, dict(case.params, elastic_precond=gspm.GSPM_PRECOND_GREEN)


def test_fp64_against_the_oracle():
    case, p = _case(35, (6, 3, 1 / 18))
    orc = O.Oracle.from_mesh(case.mesh)
    orc.set_params(p)
    assert list(orc.precond_grid()) == [204, 102, 2]      # 166 kB a plane in FP32 already
    sim = gspm.Simulation(case.mesh, p)
    x = case.mesh.per_site(np.random.default_rng(35).standard_normal((case.mesh.n_sites, 3)))
    nmap = orc.node_map()
    xu = np.zeros((orc.n, 3))
    xu[nmap] = x
    y = sim.apply(gspm.GSPM_OP_PRECOND, x)
    ref = orc.precond_apply(xu)[nmap]
    err = np.abs(y - ref).max() / np.abs(ref).max()
    print(f"B x: max rel err {err:.2e}", flush=True)
    assert err < 3e-12
    sim.close()


def _slab(a, b, c):
    """Periodic a x b x c cells of side H, Kuhn-split, inner nodes jittered: coordinates, tets, site of every node."""
    d = np.array([a + 1, b + 1, c + 1])
    ijk = np.stack(np.meshgrid(*(np.arange(k) for k in d), indexing="ij"), -1)
    at = np.arange(d.prod()).reshape(d)
    unit = w.kuhn_cube(2, 1.0)
    cells = ijk[:-1, :-1, :-1].reshape(-1, 1, 1, 3) + unit.xyz.astype(int)[unit.tets][None]
    tets = at[cells[..., 0], cells[..., 1], cells[..., 2]].reshape(-1, 4).astype(np.int32)
    ijk = ijk.reshape(-1, 3)
    inner = np.all((ijk > 0) & (ijk < d - 1), axis=1)
    xyz = ijk * H
    xyz[inner] += np.random.default_rng(5).uniform(-0.1 * H, 0.1 * H, (int(inner.sum()), 3))
    wrapped = ijk % (d - 1)
    return xyz, tets, (wrapped[:, 0] * b + wrapped[:, 1]) * c + wrapped[:, 2], np.array([a, b, c]) * H


# pure powers (library), a rod of small factors at either side of the choice, rods and films with a prime at either side
GRIDS = [(8, 8, 64), (9, 9, 9), (64, 4, 4), (12, 12, 50), (6, 6, 100), (4, 4, 61), (5, 5, 127), (61, 46, 3), (101, 67, 3),
         (22, 22, 22)]


@pytest.mark.parametrize("grid", GRIDS)
def test_films_rods_and_cubes_against_the_oracle(grid):
    xyz, tets, site, hi = _slab(*grid)
    mesh = w.Mesh(xyz=xyz, tets=tets, tags=np.ones(len(tets), np.uint8), lo=np.zeros(3), hi=hi, n_axis=0, site=site)
    p = dict(w.MATERIAL_FEGA, elastic_precond=gspm.GSPM_PRECOND_GREEN)
    orc = O.Oracle.from_mesh(mesh)
    orc.set_params(p)
    assert tuple(orc.precond_grid()) == grid
    sim = gspm.Simulation(mesh, p)
    x = np.random.default_rng(3).standard_normal((int(np.prod(grid)), 3))[site]
    xu = np.zeros((orc.n, 3))
    nmap = orc.node_map()
    xu[nmap] = x
    y = sim.apply(gspm.GSPM_OP_PRECOND, x)
    ref = orc.precond_apply(xu)[nmap]
    err = np.abs(y - ref).max() / np.abs(ref).max()
    print(f"{grid}: max rel err {err:.2e}", flush=True)
    assert err < 1e-12
    assert np.array_equal(sim.apply(gspm.GSPM_OP_PRECOND, x), y)
    sim.close()


def test_fp32_preconditions_as_fp64():
    xyz, tets, site, hi = _slab(144, 144, 11)
    mesh = w.Mesh(xyz=xyz, tets=tets, tags=np.ones(len(tets), np.uint8), lo=np.zeros(3), hi=hi, n_axis=0, site=site)
    p = dict(w.MATERIAL_FEGA, elastic_precond=gspm.GSPM_PRECOND_GREEN)
    b = 1e8 * H ** 2 * np.random.default_rng(62).standard_normal((144 * 144 * 11, 3))
    b = np.ascontiguousarray((b - b.mean(0))[site])
    its = {}
    for prec in (gspm.GSPM_FP64, gspm.GSPM_MIXED):
        sim = gspm.Simulation(mesh, p, precision=prec)
        x, its[prec] = sim.solve(gspm.GSPM_OP_ELASTIC, b, tol=1e-8)
        if prec == gspm.GSPM_FP64:
            ref = x
        sim.close()
    err = np.linalg.norm(x - ref) / np.linalg.norm(ref)
    print(f"iterations FP64 {its[0]} mixed {its[1]}, difference {err:.1e}", flush=True)
    assert its[gspm.GSPM_FP64] <= 24
    assert its[gspm.GSPM_MIXED] <= its[gspm.GSPM_FP64] + 4
    assert err < 1e-6
