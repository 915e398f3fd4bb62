"""The per-launch profile: it describes the kernels that a call runs without it, and changes no bit of the results.
(Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen

pytestmark = pytest.mark.gpu

FWD, BWD = "fwd", "bwd"  # whichever lane layouts the levels stand for
SOURCES, LEVELS = {"sources", "reduce"}, {"init", "bfs", "offsets", FWD, BWD, "reduce"}
SSSP = {"search", "sources", "reduce"}
# topology, its sources, and what each call launches
CASES = {
    "state of a source in LDS": ((1024, 6), 5, 1000, {"loads": SOURCES, "demand": SOURCES, "dist": SOURCES, "sigma": SOURCES,
                                                      "sssp": SSSP}),
    "search in LDS": ((9000, 5), 100, 300, {"loads": {"search", "offsets", FWD, BWD, "reduce"},
                                            "demand": {"search", "offsets", FWD, BWD, "reduce"},
                                            "dist": {"search", "reduce"}, "sigma": {"search", "sources", "reduce"}, "sssp": SSSP}),
    "more than 16 links a node": ((400, 17), 0, 400, {"loads": LEVELS, "demand": LEVELS, "dist": {"init", "bfs", "extract"},
                                                      "sigma": {"init", "bfs", "offsets", FWD, "extract"},
                                                      "sssp": {"init", "bfs", FWD, BWD}}),
}


def classes(profile):
    return {k[:3] if k[:3] in (FWD, BWD) else k for k, v in profile.items() if isinstance(v, dict) and v["launches"] > 0}


@pytest.mark.parametrize("name", CASES)
def test_profile_describes_what_runs(oracle, name):
    import torch
    import paper_2309_13541_amd as a2a
    shape, s0, cnt, want = CASES[name]
    rp, col = gen.random_regular(*shape, 9)
    print(name, flush=True)
    topo = a2a.Topology(rp, col)
    n = topo.N
    o = oracle.run(rp, col, s0, cnt, want_dist=True, want_load=False)
    pairs = np.bincount(o.dist[o.dist >= 0], minlength=64).tolist()
    tails = np.repeat(np.arange(n), np.diff(rp))
    links = int(((o.dist[:, col] == o.dist[:, tails] + 1) & (o.dist[:, tails] >= 0)).sum())
    demand = torch.rand((n, cnt), dtype=torch.float64, device="cuda")

    def call(what):
        ws_of = {"loads": a2a.WS_LOADS, "demand": a2a.WS_LOADS, "dist": a2a.WS_DISTANCES, "sigma": a2a.WS_SIGMA, "sssp": a2a.WS_SSSP}
        ws = torch.empty(topo.workspace_bytes(128 if what == "sssp" else cnt, ws_of[what]), dtype=torch.uint8, device="cuda")
        words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
        if what in ("dist", "sigma"):
            dist = torch.full((cnt, n), -7, dtype=torch.int32, device="cuda")
            sigma = torch.full((cnt, n), -7.0, dtype=torch.float64, device="cuda") if what == "sigma" else None
            topo.distances(s0, cnt, dist=dist, sigma=sigma, unreachable=words[:1], flags=words[1:], workspace=ws)
            out = [dist, words] + ([sigma] if what == "sigma" else [])
        else:
            load = torch.full((topo.E,), -7.0, dtype=torch.float64, device="cuda")
            kw = dict(load=load, dist_sum_total=words[:1], flags=words[1:], workspace=ws)
            if what == "loads":
                topo.link_loads(s0, cnt, **kw)
            elif what == "demand":
                topo.link_loads_demand(s0, cnt, demand=demand, **kw)
            else:
                topo.sssp_loads(s0, cnt, 128, **kw)
            out = [load, words]
        torch.cuda.synchronize()
        return out

    for what in want:
        plain = call(what)
        topo.profile_enable(1)
        timed = call(what)
        p = topo.profile_read()
        assert all(torch.equal(a, b) for a, b in zip(plain, timed)), what
        assert classes(p) == want[what], what
        assert all(v["ms"] > 0 for v in p.values() if isinstance(v, dict) and v["launches"] > 0)
        if what != "sssp":
            assert p["pairs_level"] == pairs and p["depth"] == int(o.dist.max()) and p["calls"] == 1 and p["groups"] >= 1
            topo.profile_enable(2)
            call(what)
            p = topo.profile_read()
            assert {"init", "bfs"} <= classes(p) and not {"search", "sources"} & classes(p) and p["pairs_level"] == pairs
            if what != "dist":
                assert p["dag_links"] == links
        topo.profile_enable(0)
    topo.close()
