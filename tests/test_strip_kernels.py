"""Link loads of topologies whose coefs of one source do not fit LDS (k_strip_sources), at the edges of what the kernels are chosen and
cut up by: strips, nodes per thread, words of the link table, levels of the sort and of a node's word, levels with few and with many
nodes, path counts that a word does not hold, one or two sources in the LDS of k_flow_links, pairs out of reach.  Against the
level kernels (which run while the profile counts links) and the oracle; the same bits for every workspace and from run
to run.  (Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen
from test_flow_kernels import call, kernels, thinned

pytestmark = pytest.mark.gpu


def blown_up(csr, copies):
    """Every node in so many copies, every link between all copies of its ends: path counts grow by that factor a level."""
    rp, col = csr
    rows = [[int(v) * copies + j for v in col[rp[u]:rp[u + 1]] for j in range(copies)] for u in range(len(rp) - 1)]
    return gen.csr_from_rows([row for row in rows for _ in range(copies)])


def layered_rings(rings, layers, width):
    """Rings of layers, every node linked to all of the next layer: width ** level shortest paths."""
    at = lambda r, l, i: (r * layers + l % layers) * width + i
    return gen.csr_from_rows([[at(r, l + 1, j) for j in range(width)] for r in range(rings) for l in range(layers) for _ in range(width)])


# topology, first source, sources
CASES = {
    "fewest nodes and sources": (lambda: gen.random_regular(20353, 6, 1), 5, 2048),
    "16 links": (lambda: gen.random_regular(24001, 16, 3), 1, 2049),
    "10 links": (lambda: gen.random_regular(30011, 10, 4), 20000, 2300),
    "12 levels of the sort": (lambda: gen.random_regular(30000, 4, 5), 100, 2050),
    "16 levels of the sort": (lambda: gen.random_regular(45000, 3, 6), 0, 2060),
    "two sources in LDS, two strips": (lambda: gen.random_regular(40320, 5, 7), 0, 2048),
    "one source in LDS, three strips": (lambda: gen.random_regular(40705, 5, 8), 38000, 2500),
    "most nodes, a level of few and one of many": (lambda: gen.random_regular(65536, 8, 9), 63488, 2048),
    "deepest level largest": (lambda: gen.imase_itoh(65535, 4), 30000, 2048),
    "out of reach": (lambda: thinned(33333, 6, 10, 0.1), 3, 2048),
    "path counts past a word": (lambda: blown_up(gen.random_regular(7000, 5, 11), 3), 0, 2048),
    "path counts past 16 bits": (lambda: layered_rings(190, 7, 16), 2000, 2048),
    "path counts past 12 bits, one source in LDS": (lambda: blown_up(gen.imase_itoh(14000, 3), 3), 39000, 2048),
    "path counts past 13 bits, one source in LDS": (lambda: layered_rings(370, 7, 16), 1, 2048),
    "sources without links": (lambda: gen.remove_arcs(gen.random_regular(24000, 5, 12), np.arange(100 * 5, 140 * 5)), 90, 2048),
}


def call_within(topo, s0, cnt, size):
    import torch
    ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")
    load = torch.full((topo.E,), -7.0, dtype=torch.float64, device="cuda")
    words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
    topo.link_loads(s0, cnt, load=load, dist_sum_total=words[:1], flags=words[1:], workspace=ws)
    torch.cuda.synchronize()
    return load, words


@pytest.mark.parametrize("name", CASES)
def test_loads(oracle, name):
    import torch
    import paper_2309_13541_amd as a2a
    make, s0, cnt = CASES[name]
    csr = make()
    print(name, flush=True)
    topo = a2a.Topology(*csr)
    assert "sources" in kernels(topo, a2a, s0, cnt, None)
    got, least, again = call(a2a, topo, s0, cnt, None), call(a2a, topo, s0, cnt, None, a2a.WS_MINIMAL), call(a2a, topo, s0, cnt, None)
    topo.profile_enable(2)
    ref = call(a2a, topo, s0, cnt, None)
    topo.profile_enable(0)
    for a, b, c in zip(got, least, again):
        assert torch.equal(a, b) and torch.equal(a, c)
    # a workspace of several groups but not all: a third of what the sources' rows take, behind a workgroup's records and the loads of groups
    some = max(topo.workspace_bytes(cnt, a2a.WS_LOADS | a2a.WS_MINIMAL),
               15 * topo.N * cnt // 3 + 256 * 6 * topo.N + cnt // 3 // 43 * topo.E * 8 + (8 << 20)) // 256 * 256
    topo.profile_enable(1)
    with_some = call_within(topo, s0, cnt, some)
    pieces = topo.profile_read()["reduce"]["launches"]
    topo.profile_enable(0)
    assert 2 <= pieces // 2 <= 6, pieces  # (a launch for the loads and one for the totals each)
    for a, b in zip(got, with_some):
        assert torch.equal(a, b)
    # (sums of at most 2^27 positive terms in double precision)
    assert bool(((got[0] - ref[0]).abs() <= 1e-12 * ref[0]).all())
    assert torch.equal(got[1], ref[1])
    o = oracle.run(*csr, s0, cnt, threads=8)
    assert np.allclose(got[0].cpu().numpy(), o.load, rtol=1e-11, atol=0)
    assert int(got[1][0]) == int(o.dist_sum.sum()) and int(got[1][1]) == o.flags
    topo.close()
