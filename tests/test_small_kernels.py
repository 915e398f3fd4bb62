"""The kernel that takes a source from its search to its link loads inside one workgroup, at the edges of what it is
chosen and cut up by: nodes per workgroup and per thread, words of the link table, deepest level, sources per
workgroup.  And the level kernels on the small graphs, which they do not serve by themselves.  Against the oracle.
(Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen
from gpu_helpers import run_link_loads, run_distances, assert_loads_close, assert_sigma_equal, beside_a_hub
from test_demands import run_demand_gpu, seeded_demand
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def a2a():
    import torch
    assert torch.cuda.is_available()
    import paper_2309_13541_amd as lib
    lib.load_library()
    return lib


EDGES = [(f"{n} nodes, degree {d}, {cnt} sources", (n, d), s0, cnt) for n, d, s0, cnt in (
    # nodes at which the threads per source change, and one over
    (96, 3, 0, 96), (97, 3, 0, 97), (384, 4, 0, 384), (385, 4, 0, 385), (1536, 4, 0, 1536), (1537, 4, 1000, 537),
    # words per node of the link table: 2, 3, 4, 5, 8; beyond 16 links the level kernels
    (200, 2, 0, 200), (201, 5, 0, 201), (202, 6, 0, 202), (203, 7, 0, 203), (204, 9, 0, 204), (205, 10, 0, 205),
    (206, 11, 0, 206), (207, 16, 0, 207), (208, 17, 0, 208),
    # most nodes per thread for each width, and one node over; most nodes that LDS and 16-bit places allow
    (5120, 8, 0, 40), (5121, 8, 0, 40), (6144, 6, 100, 520), (4096, 10, 0, 33), (2048, 16, 0, 70), (2049, 16, 0, 70),
    (8191, 4, 0, 270), (8192, 4, 0, 70),
    # one source; two sources at a time with one left over; a ragged last workgroup
    (1000, 5, 999, 1), (600, 5, 0, 513), (1300, 5, 7, 1037))]


@pytest.mark.parametrize("name,shape,s0,cnt", EDGES, ids=[e[0] for e in EDGES])
def test_edges_match_oracle(a2a, oracle, name, shape, s0, cnt):
    rp, col = gen.random_regular(*shape, 3)
    print(name, flush=True)
    topo = a2a.Topology(rp, col)
    o = oracle.run(rp, col, s0, cnt, threads=8)
    load, dsum, flags = run_link_loads(topo, s0, cnt)
    assert_loads_close(load, o.load)
    assert dsum == int(o.dist_sum.sum()) and flags == o.flags
    least = topo.workspace_bytes(cnt, a2a.WS_LOADS | a2a.WS_MINIMAL)
    assert np.array_equal(run_link_loads(topo, s0, cnt, least)[0], load)
    topo.close()


def circulant(nodes, offsets):
    return gen.csr_from_rows([[(u + o) % nodes for o in offsets] for u in range(nodes)])


# Three sources of a workgroup leave too few threads for 1921 to 2048 nodes with 11 to 16 links each: two are taken then.
# The second shape is so deep that LDS allows no fourth source.
THREES = {
    "2000 nodes, 12 links, 800 sources": (2000, [1, -1, 2, -2, 3, -3, 4, -4, 5, -5, 6, -6], 5, 800),
    "2048 nodes, 12 links, all sources": (2048, [1, 2, 3, 4, 5, -1, -2, -3, -4, 1, 2, -1], 0, 2048),
}


@pytest.mark.parametrize("name", THREES)
def test_too_many_nodes_for_three_sources(a2a, oracle, name):
    nodes, offsets, s0, cnt = THREES[name]
    rp, col = circulant(nodes, offsets)
    print(name, flush=True)
    topo = a2a.Topology(rp, col)
    o = oracle.run(rp, col, s0, cnt, threads=8)
    load, dsum, flags = run_link_loads(topo, s0, cnt)
    assert_loads_close(load, o.load)
    assert dsum == int(o.dist_sum.sum()) and flags == o.flags
    topo.close()


# A thread per node or two (k_node_loads), at the edges of its rule: a wave and one node over; a node a thread and one over, one
# source each and two; most nodes; three sources with few and with too many levels; and links out of service, so that some
# nodes are out of reach.
NODES = [(name, csr, s0, cnt) for name, csr, s0, cnt in (
    ("1 node", lambda: gen.csr_from_rows([[]]), 0, 1),
    ("64 nodes", lambda: gen.random_regular(64, 4, 3), 0, 64),
    ("65 nodes, one source", lambda: gen.random_regular(65, 9, 3), 64, 1),
    ("1024 nodes, 3 sources each", lambda: gen.random_regular(1024, 3, 3), 100, 700),
    ("1025 nodes, a source each", lambda: gen.random_regular(1025, 5, 3), 700, 256),
    ("2048 nodes, 2 sources each", lambda: gen.random_regular(2048, 8, 3), 1, 511),
    ("1536 nodes, 6 sources each", lambda: gen.random_regular(1536, 4, 3), 0, 1536),
    ("2047 nodes, 3 sources each", lambda: gen.random_regular(2047, 4, 3), 1300, 640),
    ("1080 nodes, 5 sources each, 11 levels", lambda: gen.torus([5, 6, 6, 6]), 0, 1080),
    ("40x40 torus, 2 sources each", lambda: gen.torus([40, 40]), 1000, 400),
    ("22x23 torus", lambda: gen.torus([22, 23]), 0, 506),
    ("26x27 torus, 3 sources each", lambda: gen.torus([26, 27]), 0, 702),
    ("8x9 torus with 90 links left", lambda: gen.remove_arcs(gen.torus([8, 9]), np.random.default_rng(5).permutation(288)[90:]), 0, 72))]


@pytest.mark.parametrize("name,csr,s0,cnt", NODES, ids=[e[0] for e in NODES])
def test_a_thread_per_node(a2a, oracle, name, csr, s0, cnt):
    rp, col = csr()
    print(name, flush=True)
    topo = a2a.Topology(rp, col)
    o = oracle.run(rp, col, s0, cnt, threads=8)
    load, dsum, flags = run_link_loads(topo, s0, cnt)
    assert_loads_close(load, o.load)
    assert dsum == int(o.dist_sum.sum()) and flags == o.flags
    least = topo.workspace_bytes(cnt, a2a.WS_LOADS | a2a.WS_MINIMAL)
    assert np.array_equal(run_link_loads(topo, s0, cnt, least)[0], load)
    dem = np.random.default_rng(78).integers(0, 7, (cnt, topo.N)).astype(np.float64)
    want, want_wd = oracle.run_demand(rp, col, dem, s0)
    load, wd, dsum, flags = run_demand_gpu(topo, dem, s0)
    assert_loads_close(load, want)
    assert wd == pytest.approx(want_wd, rel=1e-12) and dsum == int(o.dist_sum.sum())
    topo.close()


@pytest.mark.parametrize("nodes", [600, 1100])
def test_a_thread_per_node_demands_of_any_kind(a2a, oracle, nodes):
    """Demands of both signs; and an infinite one and one that is no number, which change the loads on their own shortest paths
    only: those of the source's other demands."""
    topo = a2a.Topology(*gen.random_regular(nodes, 6, 5))
    rp, col = gen.random_regular(nodes, 6, 5)
    s0, cnt = 40, 500
    assert int(topo.N) == nodes
    dem = np.random.default_rng(3).standard_normal((cnt, nodes))
    size = oracle.run_demand(rp, col, np.abs(dem), s0)
    want = oracle.run_demand(rp, col, dem, s0)
    load, wd, _, _ = run_demand_gpu(topo, dem, s0)
    # (sums of up to cnt * nodes terms of either sign: error against the sum of their magnitudes)
    assert np.all(np.abs(load - want[0]) <= 1e-12 * size[0]) and abs(wd - want[1]) <= 1e-12 * size[1]
    on_path = []  # links on a shortest path from the source to the target
    for s, t, value in ((7, 300, np.inf), (333, 5, np.nan)):
        one = np.zeros((cnt, nodes))
        one[s, t] = 1.0
        on_path.append(oracle.run_demand(rp, col, one, s0)[0] > 0)
        dem[s, t] = value
    got, got_wd, _, _ = run_demand_gpu(topo, dem, s0)
    assert on_path[0].any() and on_path[1].any() and np.isnan(got_wd)
    assert np.array_equal(np.isnan(got), on_path[1])
    assert np.array_equal(np.isposinf(got), on_path[0] & ~on_path[1])
    rest = ~(on_path[0] | on_path[1])
    assert np.array_equal(got[rest], load[rest])
    topo.close()


@pytest.mark.parametrize("nodes", [32, 33, 254, 255, 256])
def test_deepest_levels(a2a, oracle, nodes):
    """Directed rings: as many levels as nodes.  Levels fit a byte, with one value for nodes not reached, up to 253."""
    rp, col = gen.ring(nodes)
    topo = a2a.Topology(rp, col)
    load, dsum, flags = run_link_loads(topo)
    assert np.array_equal(load, np.full(nodes, nodes * (nodes - 1) / 2.0))
    assert dsum == nodes * nodes * (nodes - 1) // 2 and flags == 0
    topo.close()


@pytest.mark.parametrize("name", sorted(n for n in SMALL if len(SMALL[n][1])))
@pytest.mark.parametrize("how", ["beside a hub", "counting"])
def test_level_kernels_on_small_graphs(a2a, oracle, name, how):
    from test_sssp import run_sssp_gpu
    rp, col = beside_a_hub(SMALL[name]) if how == "beside a hub" else SMALL[name]
    print(name, flush=True)
    topo = a2a.Topology(rp, col)
    topo.profile_enable(2 if how == "counting" else 0)
    o = oracle.run(rp, col, want_dist=True, want_sigma=True)
    load, dsum, flags = run_link_loads(topo)
    assert_loads_close(load, o.load)
    assert dsum == int(o.dist_sum.sum()) and flags == o.flags
    for want_sigma in (True, False):
        dist, sigma, sums, unr, flags = run_distances(topo, want_sigma=want_sigma)
        assert np.array_equal(dist, o.dist) and np.array_equal(sums, o.dist_sum) and unr == o.unreachable
        if want_sigma and not o.flags & 1:
            assert_sigma_equal(sigma, o.sigma)
    if how == "beside a hub":
        want, _, _ = oracle.sssp(rp, col, iter_sources=64)
        assert np.array_equal(run_sssp_gpu(topo)[0], want.astype(np.float64))
    if name != "chain_2pow54":
        dem = seeded_demand(topo.N, topo.N, 77)
        want, want_wd = oracle.run_demand(rp, col, dem)
        load, wd, dsum, flags = run_demand_gpu(topo, dem)
        assert_loads_close(load, want)
        assert wd == pytest.approx(want_wd, rel=1e-12) and dsum == int(o.dist_sum.sum())
    topo.profile_enable(0)
    topo.close()


OUTPUTS = [(f"{n} nodes, degree {d}, {cnt} sources", (n, d), s0, cnt) for n, d, s0, cnt in (
    (64, 3, 0, 64), (65, 5, 3, 60), (1024, 10, 0, 1024), (1025, 6, 0, 1025), (2049, 4, 1, 2048), (4097, 8, 0, 700),
    (4900, 6, 0, 1100), (8191, 3, 5, 800), (8192, 3, 0, 70), (700, 16, 0, 513), (700, 17, 0, 100))]


@pytest.mark.parametrize("name,shape,s0,cnt", OUTPUTS, ids=[e[0] for e in OUTPUTS])
def test_distances_and_path_counts(a2a, oracle, name, shape, s0, cnt):
    rp, col = gen.random_regular(*shape, 4)
    print(name, flush=True)
    topo = a2a.Topology(rp, col)
    o = oracle.run(rp, col, s0, cnt, threads=8, want_dist=True, want_sigma=True, want_load=False)
    for flags_of in (a2a.WS_SIGMA, a2a.WS_DISTANCES):
        least = topo.workspace_bytes(cnt, flags_of | a2a.WS_MINIMAL)
        for max_ws in (None, least):
            want_sigma = flags_of == a2a.WS_SIGMA
            dist, sigma, dsum, unr, flags = run_distances(topo, s0, cnt, want_sigma=want_sigma, max_ws=max_ws)
            assert np.array_equal(dist, o.dist) and np.array_equal(dsum, o.dist_sum)
            assert unr == o.unreachable and flags == (o.flags if want_sigma else o.flags & ~1)
            if want_sigma:
                assert_sigma_equal(sigma, o.sigma)
    _, _, dsum, unr, _ = run_distances(topo, s0, cnt, want_sigma=False, want_dist=False)
    assert np.array_equal(dsum, o.dist_sum) and unr == o.unreachable
    topo.close()


SSSP = [(f"{n} nodes, degree {d}, {cnt} sources, {k} per iteration", (n, d), s0, cnt, k) for n, d, s0, cnt, k in (
    (64, 3, 0, 64, 64), (700, 5, 3, 690, 256), (1024, 10, 0, 1024, 512), (2050, 8, 0, 2050, 1024), (3000, 16, 5, 600, 64),
    # ids instead of scaled places; most nodes whose state fits; one node over; too many links
    (8191, 3, 0, 200, 128), (8192, 3, 0, 200, 128), (16384, 4, 100, 300, 128), (16384, 10, 0, 70, 64), (16385, 3, 0, 70, 64),
    (900, 17, 0, 130, 64))]


@pytest.mark.parametrize("name,shape,s0,cnt,k", SSSP, ids=[e[0] for e in SSSP])
def test_single_path_baseline(a2a, oracle, name, shape, s0, cnt, k):
    from test_sssp import run_sssp_gpu
    rp, col = gen.random_regular(*shape, 6)
    print(name, flush=True)
    topo = a2a.Topology(rp, col)
    want, dsum, unr = oracle.sssp(rp, col, s0, cnt, iter_sources=k)
    for extra in (0, 1 << 20):
        load, got_sum, flags = run_sssp_gpu(topo, s0, cnt, iter_sources=k, extra_ws=extra)
        assert np.array_equal(load, want.astype(np.float64))
        assert got_sum == int(dsum.sum()) and flags == (a2a.FLAG_UNREACHABLE if unr else 0)
    topo.close()
