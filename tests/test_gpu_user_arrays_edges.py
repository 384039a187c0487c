"""Caller arrays at the sizes where their way changes: one workgroup checks and
writes up to 2048 nodes (12 and 13 nodes an axis: 1728, 2197), and three-vectors
up to 1 MB stay in the pinned buffer for the kernels (35 and 36: 42875, 46656;
the potential of 50, 125000 values, is exactly 1 MB).

Round trips are bit for bit; a failure in any array of a call is reported by
the first that fails, leaves every field as it was and does not touch the next
call."""
import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [12, 13, 35, 36, 50])
def test_round_trips_and_failures(n):
    case = w.small_cube(n, seed=540 + n, L=1e-7, jitter=0.1, shuffle=True)
    sim = gspm.Simulation(case.mesh, case.params)
    rng = np.random.default_rng(n)
    per = case.mesh.per_site
    u, ud = per(rng.standard_normal((case.mesh.n_sites, 3))), per(rng.standard_normal((case.mesh.n_sites, 1)))[:, 0].copy()
    sim.set_u(u)
    sim.set_ud(ud)
    sim.set_m(case.m0)
    m = sim.get_m()
    _, first, inv = np.unique(case.mesh.site, return_index=True, return_inverse=True)
    copies = np.flatnonzero(first[inv] != np.arange(len(u)))
    for at in (copies[0], copies[-1], len(u) - 1, 0):
        for text, value in (("non-finite", np.nan), ("periodic copies", None)):
            if value is None and at not in copies:
                continue
            bad = u.copy()
            bad[at, 2] = bad[at, 2] * (1 + 1e-9) if value is None else value
            with pytest.raises(gspm.GspmError, match=text):
                sim.set_u(bad)
            with pytest.raises(gspm.GspmError, match=text):      # in the second array of a call
                sim.solve(gspm.GSPM_OP_GS, u, x0=bad, eps=1e-17)
            assert np.array_equal(sim.get_u(), u) and np.array_equal(sim.get_ud(), ud)
    assert np.array_equal(sim.get_m(), m)
    x, _ = sim.solve(gspm.GSPM_OP_GS, u, eps=1e-17, tol=1e-9)
    y, _ = sim.solve(gspm.GSPM_OP_GS, u, x0=u, eps=1e-17, tol=1e-9)
    # two starts: each stops at 1e-9 of |b|
    assert np.linalg.norm(x - y) <= 1e-6 * np.linalg.norm(x)
    sim.close()


@pytest.mark.parametrize("n", [12, 13, 35, 36])
def test_three_arrays_of_one_call(n):
    """The training step's arrays are told apart: each one's failure is found, and the loss is that of a fresh context."""
    case = w.small_cube(n, seed=560 + n, L=n * 4e-9, jitter=0.1)
    weights = (np.random.default_rng(1).standard_normal(gspm.GSPM_MPNN_PARAMS) * 0.1).astype(np.float32)
    rng = np.random.default_rng(n)
    per = case.mesh.per_site
    arrays = [per(rng.standard_normal((case.mesh.n_sites, 3))) for _ in range(2)] + [
        per(rng.standard_normal((case.mesh.n_sites, 3))) * 1e-12]
    sims = [gspm.Simulation(case.mesh, case.params) for _ in range(2)]
    for s in sims:
        s.mpnn_set_params(weights)
    for which in range(3):
        bad = [a.copy() for a in arrays]
        bad[which][-1, 0] = np.inf
        with pytest.raises(gspm.GspmError, match="non-finite"):
            sims[0].mpnn_train_step(*bad, update=False)
    (loss, grad), (ref, gref) = (s.mpnn_train_step(*arrays, update=False, want_grad=True) for s in sims)
    assert abs(loss - ref) <= 1e-12 * abs(ref)      # sums of shards, in any order
    assert np.linalg.norm(grad - gref) <= 1e-3 * np.linalg.norm(gref)
    for s in sims:
        s.close()
