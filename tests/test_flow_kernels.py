"""Link loads of topologies whose path counts fit LDS and whose link loads do not fit registers, at the edges of what the
kernels are chosen and cut up by: nodes per thread and block, words of the link table, 8 x id or ids in it, one or two words of
level counters, ragged groups of sources, pairs out of reach.  Against the level kernels (which run while the profile counts
links) and the oracle; the same bits for every workspace and from run to run.  (Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen

pytestmark = pytest.mark.gpu


def thinned(n, d, seed, gone):
    """Random out-lists, some links gone, and every link into the last 40 nodes: those are out of reach."""
    rp, col = gen.random_regular(n, d, seed)
    rng = np.random.default_rng(seed)
    off = rng.random(len(col)) < gone
    off |= col >= n - 40
    return gen.remove_arcs((rp, col), np.flatnonzero(off))


# topology, first source, sources, whether demands come this way too
CASES = {
    "16 links, one node past a block": (lambda: gen.random_regular(2049, 16, 1), 0, 2049, True),
    "10 links": (lambda: gen.random_regular(4097, 10, 2), 5, 1030, True),
    "8 links, fewest nodes": (lambda: gen.random_regular(5121, 8, 3), 4097, 1024, True),
    "8 x id in the table": (lambda: gen.random_regular(8191, 7, 4), 100, 1537, True),
    "ids in the table": (lambda: gen.random_regular(8192, 5, 5), 7000, 1192, True),
    "most nodes with demands": (lambda: gen.random_regular(10176, 6, 6), 0, 1500, True),
    "more nodes than with demands": (lambda: gen.random_regular(10177, 6, 7), 0, 1100, False),
    "ten levels": (lambda: gen.random_regular(16383, 4, 8), 1, 1031, False),
    "64 sources a word, four words of levels": (lambda: gen.imase_itoh(16384, 4), 3, 2000, False),
    "five words of levels": (lambda: gen.random_regular(16385, 5, 9), 0, 1025, False),
    "most nodes": (lambda: gen.random_regular(20352, 6, 10), 19200, 1152, False),
    "16 links, most nodes": (lambda: gen.random_regular(20351, 16, 11), 0, 1024, False),
    "out of reach": (lambda: thinned(9001, 6, 12, 0.05), 7977, 1024, True),
}
# calls that stay with the level kernels
OTHERS = {
    "too few sources": (lambda: gen.random_regular(8192, 5, 5), 0, 1023),
    "too many nodes": (lambda: gen.random_regular(20353, 6, 10), 0, 1024),
    "12 levels": (lambda: gen.random_regular(20011, 3, 6), 0, 1024),
    "path counts past 2^24": (lambda: gen.torus([64, 64, 3]), 0, 1024),
}


def call(a2a, topo, s0, cnt, demand, flags=0):
    import torch
    ws = torch.full((topo.workspace_bytes(cnt, a2a.WS_LOADS | flags),), 0xff, dtype=torch.uint8, device="cuda")
    load = torch.full((topo.E,), -7.0, dtype=torch.float64, device="cuda")
    words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
    weighted = torch.full((1,), -7.0, dtype=torch.float64, device="cuda")
    if demand is None:
        topo.link_loads(s0, cnt, load=load, dist_sum_total=words[:1], flags=words[1:], workspace=ws)
    else:
        topo.link_loads_demand(s0, cnt, demand=demand, load=load, weighted_dist=weighted, dist_sum_total=words[:1],
                               flags=words[1:], workspace=ws)
    torch.cuda.synchronize()
    return load, words, weighted


def kernels(topo, a2a, s0, cnt, demand):
    topo.profile_enable(1)
    call(a2a, topo, s0, cnt, demand)
    p = topo.profile_read()
    topo.profile_enable(0)
    return {k for k, v in p.items() if isinstance(v, dict) and v["launches"] > 0}


@pytest.mark.parametrize("name", CASES)
def test_loads(oracle, name):
    import torch
    import paper_2309_13541_amd as a2a
    make, s0, cnt, with_demand = CASES[name]
    csr = make()
    print(name, flush=True)
    topo = a2a.Topology(*csr)
    # demands of any sign and size, none from some sources
    demand = torch.randn((topo.N, cnt), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    demand[:, ::17] = 0.0
    for dem in (None, demand):
        assert kernels(topo, a2a, s0, cnt, dem) & {"sources", "bwd_rows"} == {"sources" if dem is None or with_demand else "bwd_rows"}
        got, least, again = call(a2a, topo, s0, cnt, dem), call(a2a, topo, s0, cnt, dem, a2a.WS_MINIMAL), call(a2a, topo, s0, cnt, dem)
        topo.profile_enable(2)
        ref = call(a2a, topo, s0, cnt, dem)
        topo.profile_enable(0)
        for a, b, c in zip(got, least, again):
            assert torch.equal(a, b) and torch.equal(a, c)
        assert torch.equal(got[1], ref[1])
        # Loads are sums of up to cnt * N terms of either sign with demands: error against the sum of their magnitudes.
        if dem is None:
            size = ref[0]
        else:
            size = call(a2a, topo, s0, cnt, dem.abs())[0]
            assert abs(float(got[2] - ref[2])) <= 1e-12 * float(call(a2a, topo, s0, cnt, dem.abs())[2])
        assert bool(((got[0] - ref[0]).abs() <= 1e-12 * size).all())
        if dem is None:
            o = oracle.run(*csr, s0, cnt, threads=8)
            assert np.allclose(got[0].cpu().numpy(), o.load, rtol=1e-11, atol=0)
            assert int(got[1][0]) == int(o.dist_sum.sum()) and int(got[1][1]) == o.flags
    topo.close()


@pytest.mark.parametrize("name", OTHERS)
def test_calls_that_stay_with_the_level_kernels(name):
    import paper_2309_13541_amd as a2a
    make, s0, cnt = OTHERS[name]
    topo = a2a.Topology(*make())
    print(name, flush=True)
    assert "sources" not in kernels(topo, a2a, s0, cnt, None)
    topo.close()


def test_infinite_demand_stays_on_its_paths():
    """An infinite demand makes the loads on its own shortest paths infinite and leaves all others alone."""
    import torch
    import paper_2309_13541_amd as a2a
    topo = a2a.Topology(*gen.random_regular(8200, 6, 3))
    cnt = 1100
    demand = torch.rand((topo.N, cnt), dtype=torch.float64, device="cuda")
    demand[4000, 5] = float("inf")
    assert "sources" in kernels(topo, a2a, 0, cnt, demand)
    got = call(a2a, topo, 0, cnt, demand)[0]
    topo.profile_enable(2)
    ref = call(a2a, topo, 0, cnt, demand)[0]
    topo.profile_enable(0)
    assert torch.equal(torch.isfinite(got), torch.isfinite(ref)) and not bool(torch.isnan(got).any())
    assert not bool(torch.isfinite(got).all())
    topo.close()
