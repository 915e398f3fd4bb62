"""The search of the workgroups that keep their sources in LDS, at the edges of its variants: planes of the distances (levels up
to 7, 31 and beyond), nodes a thread has, links held or fetched, sources of a batch; and levels with more nodes than the
source has threads.  Against the oracle.  (Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen
from gpu_helpers import run_link_loads, run_distances, assert_loads_close, assert_sigma_equal

pytestmark = pytest.mark.gpu

CASES = {
    "7 levels": (lambda: gen.torus([4, 4, 6]), 0, 96),
    "8 levels": (lambda: gen.torus([4, 4, 8]), 3, 33),
    "31 levels": (lambda: gen.torus([30, 32]), 900, 32),
    "32 levels": (lambda: gen.torus([32, 32]), 0, 31),
    "31 levels, 8 nodes a thread": (lambda: gen.torus([16, 18, 28]), 8000, 64),
    "32 levels, 8 nodes a thread": (lambda: gen.torus([14, 18, 32]), 4095, 1),
    "4 nodes a thread, all in use": (lambda: gen.random_regular(4096, 7, 3), 1, 65),
    "links fetched for every level": (lambda: gen.random_regular(8191, 9, 3), 0, 40),
    "most links": (lambda: gen.random_regular(2048, 16, 3), 5, 300),
    "one level of 1023 nodes": (lambda: gen.random_regular(1024, 3, 3), 0, 600),
}


@pytest.mark.parametrize("name", CASES)
def test_search_matches_oracle(oracle, name):
    import paper_2309_13541_amd as a2a
    make, s0, cnt = CASES[name]
    print(name, flush=True)
    rp, col = make()
    topo = a2a.Topology(rp, col)
    o = oracle.run(rp, col, s0, cnt, threads=8, want_dist=True, want_sigma=True)
    dist, _, sums, _, _ = run_distances(topo, s0, cnt, want_sigma=False)
    assert np.array_equal(dist, o.dist) and np.array_equal(sums, o.dist_sum)
    dist, sigma, sums, _, _ = run_distances(topo, s0, cnt)
    assert np.array_equal(dist, o.dist) and np.array_equal(sums, o.dist_sum)
    assert_sigma_equal(sigma, o.sigma)
    load, dsum, flags = run_link_loads(topo, s0, cnt)
    assert_loads_close(load, o.load)
    assert dsum == int(o.dist_sum.sum()) and flags == o.flags
    topo.close()
