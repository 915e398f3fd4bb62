"""Link loads with a thread per node or two and two sources at a time, at the edges of its rule: against the oracle; the same bits in a
workspace for some of the rows.  (Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen

pytestmark = pytest.mark.gpu


def thinned(n, d, seed, gone):
    """Random out-lists, some links gone, and every link into the last 20 nodes: those are out of reach."""
    rp, col = gen.random_regular(n, d, seed)
    off = np.random.default_rng(seed).random(len(col)) < gone
    off |= col >= n - 20
    return gen.remove_arcs((rp, col), np.flatnonzero(off))


# sources a workgroup in front; an odd number of sources leaves the last workgroup one
CASES = {
    "2: 257 nodes": (lambda: gen.random_regular(257, 4, 1), 0, 257),
    "2: 1024 nodes, 10 links": (lambda: gen.random_regular(1024, 10, 2), 3, 511),
    "4: hypercube": (lambda: gen.hypercube(10), 0, 1023),
    "4: 16 levels": (lambda: gen.torus([16, 16, 4]), 0, 1024),
    "2: 1025 nodes, 8 links": (lambda: gen.random_regular(1025, 8, 3), 400, 512),
    "2: many levels": (lambda: gen.torus([20, 100]), 1, 509),
    "4: 2048 nodes": (lambda: gen.random_regular(2048, 6, 4), 7, 901),
    "5: 1537 nodes": (lambda: gen.random_regular(1537, 4, 5), 0, 1279),
    "6: 1536 nodes": (lambda: gen.random_regular(1536, 5, 6), 0, 1535),
    "8: 2048 nodes, 5 levels": (lambda: gen.random_regular(2048, 8, 7), 0, 2048),
    "2: out of reach": (lambda: thinned(700, 5, 8, 0.1), 200, 500),
    "4: out of reach": (lambda: thinned(1400, 6, 9, 0.1), 0, 1021),
}


@pytest.mark.parametrize("name", CASES)
def test_loads(oracle, name):
    import torch
    import paper_2309_13541_amd as a2a
    make, s0, cnt = CASES[name]
    csr = make()
    print(name, flush=True)
    topo = a2a.Topology(*csr)
    got = []
    for flags in (a2a.WS_LOADS, a2a.WS_LOADS | a2a.WS_MINIMAL):
        ws = torch.full((topo.workspace_bytes(cnt, flags),), 0xff, dtype=torch.uint8, device="cuda")
        load = torch.full((topo.E,), -7.0, dtype=torch.float64, device="cuda")
        words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
        topo.link_loads(s0, cnt, load=load, dist_sum_total=words[:1], flags=words[1:], workspace=ws)
        torch.cuda.synchronize()
        got.append((load.cpu(), words.cpu()))
    topo.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    o = oracle.run(*csr, s0, cnt, threads=8)
    # sums of up to 2048 x 2048 positive terms in double precision, in two orders
    assert np.allclose(got[0][0].numpy(), o.load, rtol=1e-11, atol=0)
    assert int(got[0][1][0]) == int(o.dist_sum.sum()) and int(got[0][1][1]) == o.flags
