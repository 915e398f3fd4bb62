"""Levels of a search that go by the list of their new nodes (wide_list): a second level that just fits it and one that does not,
levels that all fit it with most pairs out of reach, 16 and 32 sources a word, ragged groups.  Distances and sums against the
oracle.  (Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen
from gpu_helpers import run_distances

pytestmark = pytest.mark.gpu


def rings(n, size):
    """Directed rings of that size, side by side."""
    return gen.csr_from_rows([[u - u % size + (u + 1) % size] for u in range(n)])


# 16392 nodes: at most 2049 entries, and 16 sources have 16 * 11 ** 2 or 16 * 12 ** 2 new nodes on their second level
CASES = {
    "second level fits": (lambda: gen.random_regular(16392, 11, 1), 7, 64),
    "second level is one too many": (lambda: gen.random_regular(16392, 12, 2), 7, 64),
    "all levels by the list": (lambda: rings(20000, 50), 19000, 1000),
    "32 sources a word": (lambda: gen.random_regular(20011, 5, 3), 100, 4200),
    "last group of one source": (lambda: gen.random_regular(65536, 3, 4), 65535 - 48, 49),
    "a node without links": (lambda: gen.remove_arcs(gen.random_regular(16400, 4, 5), np.arange(400)), 0, 200),
}


@pytest.mark.parametrize("name", CASES)
def test_distances(oracle, name):
    import paper_2309_13541_amd as a2a
    make, s0, cnt = CASES[name]
    rp, col = make()
    print(name, flush=True)
    topo = a2a.Topology(rp, col)
    o = oracle.run(rp, col, s0, cnt, threads=8, want_dist=True)
    dist, _, sums, _, _ = run_distances(topo, s0, cnt, want_sigma=False)
    assert np.array_equal(dist, o.dist) and np.array_equal(sums, o.dist_sum)
    topo.close()
