"""The network's gradient at the sizes where its kernels' partition can go wrong.

Nodes are dealt to workgroups in runs, to waves in groups of 16 (node GEMMs and
encoder) and 32 (weight gradients), edges in pairs and eights: meshes below one
group, with remainders of each, of one and of several workgroups, and the
five-tetrahedra split, whose degrees are not all 14.  Tolerances as derived in
test_gpu_mpnn: 5e-2 per parameter block (against the rms entry where a block
vanishes), 2e-2 on the loss.
"""
import numpy as np
import pytest

from oracle import mpnn_oracle as N
from paper_2510_09812_amd import gspm
from test_gpu_mpnn import _init_params, _oracle_inputs, _setup, _unique

pytestmark = pytest.mark.gpu


# unique nodes: 27, 64, 125, 216, 1000, 1331, 4913
@pytest.mark.parametrize("n,split", [(4, "kuhn"), (5, "five"), (6, "kuhn"), (7, "five"), (11, "five"), (12, "kuhn"),
                                     (18, "kuhn")])
def test_gradient_over_sizes(n, split):
    case, orc, g, m, mp = _setup(n=n, seed=420 + n, split=split)
    params = _init_params(30 + n, scale=0.8)
    sim = gspm.Simulation(case.mesh, case.params)
    sim.mpnn_set_params(params)
    mu, mpu, wts = _oracle_inputs(orc, m, mp)
    rng = np.random.default_rng(n)
    du = case.mesh.per_site(rng.standard_normal((case.mesh.n_sites, 3)) * 1e-12)
    args = mpu[orc.node_map()], mu[orc.node_map()], du
    loss_gpu, grad = sim.mpnn_train_step(*args, update=False, want_grad=True)
    x, sm = N.features(mu, mpu, wts)
    P = N.unpack(params)
    y, cache = N.forward(P, x, g, bf16=True)
    loss, gy = N.loss_and_grad_y(y, _unique(orc, du) / (case.params["lambda100"] * g.hbar * sm))
    G = N.pack(N.backward(P, cache, gy, g))
    assert abs(loss_gpu - loss) <= 2e-2 * loss
    o, gscale, worst = 0, np.linalg.norm(G) / np.sqrt(G.size), 0.0
    for name, shp in N.param_shapes():
        k = int(np.prod(shp))
        den = max(np.linalg.norm(G[o:o + k]), 1e-2 * gscale * np.sqrt(k))
        worst = max(worst, np.linalg.norm(grad[o:o + k] - G[o:o + k]) / den)
        assert worst < 5e-2, name
        o += k
    print(f"n={n} {split}: {orc.n} nodes, worst block {worst:.2e}", flush=True)
    sim.close()
