"""Single-path baseline with one source at a time in a workgroup's LDS, at the edges of where it is taken and of what it is cut up
by.  Bit for bit against the oracle (whole numbers).  (Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen
from test_sssp import run_sssp_gpu

pytestmark = pytest.mark.gpu

CASES = {  # topology, first source, sources, sources per iteration
    "4096 nodes: below": (lambda: gen.random_regular(4096, 4, 6), 0, 300, 128),
    "4097 nodes": (lambda: gen.random_regular(4097, 4, 6), 4000, 97, 64),
    "costs of many iterations": (lambda: gen.random_regular(4200, 6, 6), 0, 4200, 256),
    "8191 nodes, 2 words": (lambda: gen.random_regular(8191, 3, 6), 5, 700, 512),
    "8192 nodes, 3 words": (lambda: gen.random_regular(8192, 5, 6), 0, 513, 512),
    "13 levels of 2 links": (lambda: gen.imase_itoh(8000, 2), 100, 130, 64),
    "10007 nodes, 5 words": (lambda: gen.random_regular(10007, 9, 6), 1, 300, 256),
    "16383 nodes, 8 words": (lambda: gen.random_regular(16383, 16, 6), 16000, 200, 128),
    "16384 nodes, 4 words": (lambda: gen.random_regular(16384, 8, 6), 0, 257, 256),
    "16384 nodes, many levels": (lambda: gen.random_regular(16384, 3, 6), 777, 300, 256),
    "24 levels: too many": (lambda: gen.torus([16, 16, 17]), 0, 100, 64),
    "parts out of reach": (lambda: gen.remove_arcs(gen.random_regular(5000, 3, 6), range(0, 9000)), 0, 400, 256),
}


@pytest.mark.parametrize("name", CASES)
def test_matches_oracle(oracle, name):
    import paper_2309_13541_amd as a2a
    make, s0, cnt, k = CASES[name]
    print(name, flush=True)
    rp, col = make()
    topo = a2a.Topology(rp, col)
    want, dsum, unr = oracle.sssp(rp, col, s0, cnt, iter_sources=k)
    load, got_sum, flags = run_sssp_gpu(topo, s0, cnt, iter_sources=k)
    assert np.array_equal(load, want.astype(np.float64))
    assert got_sum == int(dsum.sum()) and flags == (a2a.FLAG_UNREACHABLE if unr else 0)
    topo.close()
