"""The network's set-up gives back what only its set-up reads: the neighbour
list, four bytes an edge, once the edges' vectors are formed."""
import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu


def test_the_neighbour_list_is_given_back():
    import torch
    case = w.small_cube(21, seed=77, L=8e-8, jitter=0.1)
    edges = 14 * 20 ** 3                      # directed, on a Kuhn mesh
    sim = gspm.Simulation(case.mesh, case.params, allocator=gspm.torch_allocator(0))
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats(0)
    before = torch.cuda.memory_allocated(0)
    sim.mpnn_set_params(np.random.default_rng(1).standard_normal(gspm.GSPM_MPNN_PARAMS).astype(np.float32) * 0.1)
    held, peak = torch.cuda.memory_allocated(0) - before, torch.cuda.max_memory_allocated(0) - before
    print(f"held {held}, at most {peak} bytes, {edges} edges", flush=True)
    assert peak - held >= 4 * edges
    y, s = sim.mpnn_forward(case.m0, np.roll(case.m0, 1, axis=1))
    assert np.all(np.isfinite(y)) and s > 0.0
    sim.close()
    assert torch.cuda.memory_allocated(0) <= before
