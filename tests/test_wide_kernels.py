"""Distances of 8192 to 65536 nodes (search with the frontier in LDS) at the edges of what the kernel is chosen and cut
up by: nodes per thread, sources per word (16, 32, 64), words of the link table, levels, ragged last workgroups, pairs
out of reach.  All rows against the level kernels (which run while the profile counts links), some against the oracle.
(Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen

pytestmark = pytest.mark.gpu


def thinned(n, d, seed, gone):
    """Random out-lists, a share of the links gone: some nodes are out of reach."""
    csr = gen.random_regular(n, d, seed)
    rng = np.random.default_rng(seed)
    return gen.remove_arcs(csr, rng.choice(len(csr[1]), int(gone * len(csr[1])), replace=False))


CASES = {
    "smallest, 16 sources a word": (lambda: gen.random_regular(8192, 4, 1), 100, 777),
    "one source": (lambda: gen.random_regular(9001, 3, 2), 9000, 1),
    "32 sources a word, ragged": (lambda: gen.random_regular(12345, 5, 3), 100, 4101),
    "64 sources a word, most nodes": (lambda: gen.random_regular(16384, 8, 4), 7000, 8200),
    "past 64 sources a word": (lambda: gen.random_regular(16385, 6, 5), 0, 8200),
    "past 32 sources a word": (lambda: gen.random_regular(32769, 3, 6), 5, 4100),
    "most nodes, three rounds": (lambda: gen.random_regular(65536, 3, 7), 56000, 9500),
    "16 links a node": (lambda: gen.random_regular(10000, 16, 8), 0, 100),
    "17 links a node: level kernels": (lambda: gen.random_regular(10000, 17, 8), 0, 100),
    "out of reach": (lambda: thinned(10240, 3, 9, 0.5), 3, 4200),
    "out of reach, more than 64 sources a word holds": (lambda: thinned(20011, 5, 10, 0.6), 1, 300),
    "deepest": (lambda: gen.torus([60, 64, 3]), 0, 9000),
    "one level too deep": (lambda: gen.torus([60, 66, 3]), 0, 100),
}


@pytest.mark.parametrize("name", CASES)
def test_wide_distances(oracle, name):
    import torch
    import paper_2309_13541_amd as a2a
    make, s0, cnt = CASES[name]
    csr = make()
    print(name, flush=True)
    topo = a2a.Topology(*csr)

    def run(ws_bytes=None, want=True):
        ws = torch.empty(ws_bytes or topo.workspace_bytes(cnt, a2a.WS_DISTANCES), dtype=torch.uint8, device="cuda")
        dist = torch.full((cnt, topo.N), -7, dtype=torch.int32, device="cuda") if want else None
        sums = torch.full((cnt,), -7, dtype=torch.int64, device="cuda")
        words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
        topo.distances(s0, cnt, dist=dist, dist_sum=sums, unreachable=words[:1], flags=words[1:], workspace=ws)
        torch.cuda.synchronize()
        return dist, sums, words

    dist, sums, words = run()
    topo.profile_enable(2)
    ref = run()
    topo.profile_enable(0)
    assert torch.equal(dist, ref[0]) and torch.equal(sums, ref[1]) and torch.equal(words, ref[2])
    only = run(topo.workspace_bytes(cnt, a2a.WS_DISTANCES | a2a.WS_MINIMAL), False)
    assert torch.equal(sums, only[1]) and torch.equal(words, only[2])
    rows = min(cnt, 32)
    o = oracle.run(*csr, s0, rows, want_dist=True, threads=8)
    assert np.array_equal(dist[:rows].cpu().numpy(), o.dist)
    topo.close()


SIGMA = {
    "smallest": (lambda: gen.random_regular(8192, 4, 1), 100, 777),
    "one source": (lambda: gen.random_regular(9001, 3, 2), 9000, 1),
    "most nodes, whole LDS": (lambda: gen.random_regular(16384, 8, 3), 7000, 4200),
    "too many nodes: level kernels": (lambda: gen.random_regular(16385, 5, 3), 0, 70),
    "odd rows, out of reach": (lambda: thinned(10241, 3, 9, 0.5), 3, 300),
    "16 links a node": (lambda: gen.random_regular(12000, 16, 5), 0, 64),
    "deepest": (lambda: gen.torus([56, 62, 3]), 10, 300),
    "one level too deep": (lambda: gen.torus([56, 64, 3]), 10, 70),
}


@pytest.mark.parametrize("name", SIGMA)
def test_wide_path_counts(oracle, name):
    import torch
    import paper_2309_13541_amd as a2a
    make, s0, cnt = SIGMA[name]
    csr = make()
    print(name, flush=True)
    topo = a2a.Topology(*csr)

    def run(flags):
        ws = torch.empty(topo.workspace_bytes(cnt, a2a.WS_SIGMA | flags), dtype=torch.uint8, device="cuda")
        dist = torch.full((cnt, topo.N), -7, dtype=torch.int32, device="cuda")
        sigma = torch.full((cnt, topo.N), -7.0, dtype=torch.float64, device="cuda")
        sums = torch.full((cnt,), -7, dtype=torch.int64, device="cuda")
        words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
        topo.distances(s0, cnt, dist=dist, sigma=sigma, dist_sum=sums, unreachable=words[:1], flags=words[1:], workspace=ws)
        torch.cuda.synchronize()
        return sigma, dist, sums, words

    got, least = run(0), run(a2a.WS_MINIMAL)
    topo.profile_enable(2)
    ref = run(0)
    topo.profile_enable(0)
    for a, b in zip(got, least):
        assert torch.equal(a, b)
    for a, b in zip(got[1:], ref[1:]):
        assert torch.equal(a, b)
    whole = ref[0] < 2.0 ** 53
    assert torch.equal(got[0][whole], ref[0][whole])
    assert bool(((got[0] - ref[0]).abs() <= 1e-13 * ref[0]).all())
    if bool(whole.all()):
        o = oracle.run(*csr, s0, min(cnt, 16), want_sigma=True, threads=8)
        assert np.array_equal(got[0][:min(cnt, 16)].cpu().numpy(), o.sigma.astype(np.float64))
    topo.close()


LOADS = {
    "8 x id in the table": (lambda: gen.random_regular(8191, 8, 1), 0, 700),
    "fewest nodes with padded rows": (lambda: gen.random_regular(4097, 10, 2), 4000, 97),
    "64 sources a word": (lambda: gen.random_regular(8192, 5, 3), 1000, 777),
    "64 sources a word, most nodes": (lambda: gen.random_regular(16384, 4, 4), 16000, 384),
    "16 sources a word, ragged batch": (lambda: gen.random_regular(16385, 4, 5), 3, 213),
    "more groups than workgroups": (lambda: gen.random_regular(20011, 3, 6), 0, 4200),
    "out of reach": (lambda: thinned(17000, 3, 7, 0.5), 10, 300),
    "out of reach, 64 sources a word": (lambda: thinned(9000, 3, 8, 0.5), 10, 300),
    "deep": (lambda: gen.torus([90, 95]), 0, 130),
    "2500 levels": (lambda: gen.bidirectional_ring(5000), 4900, 100),
    # a source's levels end with the chain: batches of 2200 to 2400 levels, most of a topology's 4999 empty
    "4999 levels, batches that end early": (lambda: gen.csr_from_rows([[u + 1] for u in range(4999)] + [[]]), 2600, 200),
}


@pytest.mark.parametrize("name", LOADS)
def test_index_entries_from_wide_search(oracle, name):
    """Loads: the index entries are those of the level search (which runs while the profile counts links), so the bits
    are too."""
    import torch
    import paper_2309_13541_amd as a2a
    make, s0, cnt = LOADS[name]
    csr = make()
    print(name, flush=True)
    topo = a2a.Topology(*csr)
    demand = torch.rand((topo.N, cnt), dtype=torch.float64, device="cuda") + 0.5

    def run(flags, dem):
        ws = torch.empty(topo.workspace_bytes(cnt, a2a.WS_LOADS | flags), dtype=torch.uint8, device="cuda")
        load = torch.full((topo.E,), -7.0, dtype=torch.float64, device="cuda")
        words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
        weighted = torch.full((1,), -7.0, dtype=torch.float64, device="cuda")
        if dem:
            topo.link_loads_demand(s0, cnt, demand=demand, load=load, weighted_dist=weighted, dist_sum_total=words[:1],
                                   flags=words[1:], workspace=ws)
        else:
            topo.link_loads(s0, cnt, load=load, dist_sum_total=words[:1], flags=words[1:], workspace=ws)
        torch.cuda.synchronize()
        return load, words, weighted

    for dem in (False, True):
        got, least = run(0, dem), run(a2a.WS_MINIMAL, dem)
        topo.profile_enable(2)
        ref = run(0, dem)
        topo.profile_enable(0)
        for a, b, c in zip(got, least, ref):
            assert torch.equal(a, b) and torch.equal(a, c)
        if not dem:
            o = oracle.run(*csr, s0, cnt, threads=8)
            # (with path counts beyond 2^53 the level kernels are the only reference)
            assert o.flags & 1 or np.allclose(got[0].cpu().numpy(), o.load, rtol=1e-11, atol=0)
            assert int(got[1][0]) == int(o.dist_sum.sum())
    topo.close()
