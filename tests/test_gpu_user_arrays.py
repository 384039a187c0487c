"""Caller arrays on their way to and from the device, against numpy.

Sizes from a part of one chunk of the staging buffer to several (1 MB, 43690
nodes' three-vectors): 27, 1000, 46656 and 226981 nodes.  A permutation and correctly rounded operations: results are equal
bit for bit.  Failures are reported as a check in caller order meets them, and
leave the state as it was.
"""
import numpy as np
import pytest

import workloads as w
from paper_2510_09812_amd import gspm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,shuffle", [(3, False), (10, True), (36, True), (61, False)])
def test_round_trip(n, shuffle):
    case = w.small_cube(n, seed=500 + n, L=1e-7, jitter=0.1, sphere=0.3, shuffle=shuffle)
    sim = gspm.Simulation(case.mesh, case.params)
    rng = np.random.default_rng(n)
    per = case.mesh.per_site
    u = per(rng.standard_normal((case.mesh.n_sites, 3)) * 1e-10)
    ud = per(rng.standard_normal((case.mesh.n_sites, 3)))[:, 0].copy()
    m = rng.standard_normal((case.mesh.n_sites, 3))
    m[::7] *= 1e150
    m = per(m)
    sim.set_u(u)
    sim.set_ud(ud)
    sim.set_m(m)
    assert np.array_equal(sim.get_u(), u)
    assert np.array_equal(sim.get_ud(), ud)
    got = sim.get_m()
    r = np.sqrt(m[:, 0] * m[:, 0] + m[:, 1] * m[:, 1] + m[:, 2] * m[:, 2])[:, None]
    mag = np.any(got != 0, axis=1)
    assert mag.any() and np.array_equal(got[mag], (m / r)[mag])
    sim.set_m(got)           # unit vectors to rounding come back as they were
    assert np.array_equal(sim.get_m(), got)
    sim.close()


def test_failures_in_caller_order():
    case = w.small_cube(12, seed=520, L=1e-7, jitter=0.1, shuffle=True)
    sim = gspm.Simulation(case.mesh, case.params)
    rng = np.random.default_rng(1)
    u = case.mesh.per_site(rng.standard_normal((case.mesh.n_sites, 3)))
    m = case.mesh.per_site(rng.standard_normal((case.mesh.n_sites, 3)))
    sim.set_u(u)
    sim.set_m(m)
    kept = sim.get_m()
    # a periodic copy: a node whose value another node shares
    _, first, inv = np.unique(u[:, 0], return_index=True, return_inverse=True)
    copy = int(np.flatnonzero(first[inv] != np.arange(len(u)))[3])
    sole = int(np.flatnonzero(np.bincount(inv)[inv] == 1)[5])
    lo, hi = min(copy, sole), max(copy, sole)

    def refused(setter, v, text):
        with pytest.raises(gspm.GspmError, match=text):
            setter(v)

    differs, bad, both = u.copy(), u.copy(), u.copy()
    differs[copy, 1] *= 1 + 1e-9
    bad[sole, 2] = np.inf
    both[copy, 1] *= 1 + 1e-9
    both[sole, 2] = np.nan
    refused(sim.set_u, differs, "periodic copies")
    refused(sim.set_u, bad, "non-finite")
    refused(sim.set_u, both, "periodic copies" if lo == copy else "non-finite")
    near = u.copy()
    near[copy, 1] *= 1 + 1e-14
    sim.set_u(near)                       # equal to rounding
    assert np.array_equal(sim.get_u(), u)
    zero = m.copy()
    zero[sole] = 0.0
    refused(sim.set_m, zero, "zero magnetisation")
    zero[sole] = 1e-200                   # its length underflows
    refused(sim.set_m, zero, "zero magnetisation")
    zero[hi, 0] = np.nan
    refused(sim.set_m, zero, "non-finite")
    assert np.array_equal(sim.get_m(), kept) and np.array_equal(sim.get_u(), u)
    sim.close()
