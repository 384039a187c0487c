"""Row forms are built only where a one-launch solve can use them.

An FP64 context has kernels for up to 2048 rows a workgroup, and a mesh whose
node order makes long halo lists may not fit LDS at any size: such contexts
solve by launches, and neither the upload nor set_params may take memory for
rows.  Counted through the caller's allocator."""
import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu

H = 4e-9


def _held(case, **kw):
    """Bytes held after the upload, and what set_params adds without and with the local magnetostatic solve."""
    import torch
    torch.cuda.synchronize()
    start = torch.cuda.memory_allocated(0)
    sim = gspm.Simulation(case.mesh, None, allocator=gspm.torch_allocator(0), **kw)
    out = [torch.cuda.memory_allocated(0) - start]
    for ld in (False, True):
        before = torch.cuda.memory_allocated(0)
        sim.set_params(case.params, local_demag=ld)
        out.append(torch.cuda.memory_allocated(0) - before)
    sim.close()
    return out


def test_fp64_meshes_beyond_its_rows():
    case = w.small_cube(82, seed=9, L=81 * H, jitter=0.1)          # 531,441 nodes: 2112 rows a workgroup
    n = 81 ** 3
    up, el, ms = _held(case, precision=gspm.GSPM_FP64)
    print(f"FP64: upload {up}, elastic {el}, magnetostatic {ms} bytes", flush=True)
    assert el == 0 and ms == 0
    up, el, ms = _held(case, precision=gspm.GSPM_MIXED)
    print(f"mixed: upload {up}, elastic {el}, magnetostatic {ms} bytes", flush=True)
    assert el == 0 and ms > 14 * n * (8 + 4)                       # K^ms in both types, 14 entries a row


def test_halos_beyond_lds():
    """Shuffled nodes in the caller's order: a workgroup's 576 rows have some 7000 halo nodes."""
    case = w.small_cube(53, seed=10, L=52 * H, jitter=0.1, shuffle=True)
    up, el, ms = _held(case, precision=gspm.GSPM_FP64, reorder=gspm.GSPM_REORDER_NONE)
    print(f"shuffled: upload {up}, elastic {el}, magnetostatic {ms} bytes", flush=True)
    assert el == 0
    _, el2, _ = _held(case, precision=gspm.GSPM_FP64)
    assert el2 > 6 * 14 * 8 * 52 ** 3                              # Morton order fits: six numbers an entry
    # and the solves serve
    sim = gspm.Simulation(case.mesh, case.params, reorder=gspm.GSPM_REORDER_NONE)
    x = case.mesh.per_site(np.random.default_rng(1).standard_normal((case.mesh.n_sites, 3)))
    for op in (gspm.GSPM_OP_ELASTIC, gspm.GSPM_OP_MS):
        b = np.ascontiguousarray(sim.apply(op, x))
        y, _ = sim.solve(op, b, tol=1e-8)
        assert np.linalg.norm(b - sim.apply(op, y)) <= 2e-8 * np.linalg.norm(b)
    sim.close()
