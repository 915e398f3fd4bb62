"""Link loads with a thread per node or two and two sources at a time, at the edges of its rule: that the rule takes them; against the
oracle; the same bits in a workspace for some of the rows.  (Loads need an MI355X.)"""
import os
import subprocess

import numpy as np
import pytest

import a2a_inputs as gen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def thinned(n, d, seed, gone):
    """Random out-lists, some links gone, and every link into the last 20 nodes: those are out of reach."""
    rp, col = gen.random_regular(n, d, seed)
    off = np.random.default_rng(seed).random(len(col)) < gone
    off |= col >= n - 20
    return gen.remove_arcs((rp, col), np.flatnonzero(off))


# in front: sources a workgroup, 0 where another kernel takes them; an odd number of sources leaves the last workgroup one
CASES = {
    "2: 257 nodes": (lambda: gen.random_regular(257, 4, 1), 0, 257),
    "2: 1024 nodes, 10 links": (lambda: gen.hypercube(10), 3, 511),
    "4: hypercube": (lambda: gen.hypercube(10), 0, 1023),
    "4: 16 levels": (lambda: gen.torus([16, 8, 8]), 0, 1024),
    "0: 18 levels": (lambda: gen.torus([16, 16, 4]), 0, 1024),
    # 7 and 8 links: a node's place is not its number; the last block of 16 whole, and of one node
    "4: 8 links": (lambda: gen.imase_itoh(1024, 8), 0, 1024),
    "4: 8 links, a block of one": (lambda: gen.imase_itoh(1009, 8), 5, 901),
    "2: 7 links, out of reach": (lambda: thinned(913, 7, 11, 0.1), 0, 511),
    "0: 1025 nodes, 8 links": (lambda: gen.random_regular(1025, 8, 3), 400, 512),
    "2: 1025 nodes, 6 links": (lambda: gen.random_regular(1025, 6, 3), 400, 512),
    "2: many levels": (lambda: gen.torus([20, 100]), 1, 509),
    "4: 2048 nodes": (lambda: gen.random_regular(2048, 6, 4), 7, 901),
    "5: 1537 nodes": (lambda: gen.random_regular(1537, 4, 5), 0, 1279),
    "5: 1553 nodes, 8 links": (lambda: gen.imase_itoh(1553, 8), 0, 1279),
    "6: 1536 nodes": (lambda: gen.random_regular(1536, 5, 6), 0, 1535),
    "8: 2048 nodes, 5 levels": (lambda: gen.random_regular(2048, 8, 7), 0, 2048),
    "2: out of reach": (lambda: thinned(700, 5, 8, 0.1), 200, 500),
    "4: out of reach": (lambda: thinned(1400, 6, 9, 0.1), 0, 1021),
}

RULE = r"""
#include <cstdio>
#include <cstdlib>
#include "a2a_plan.h"
using namespace a2a_dev;

int main(int argc, char** argv) {  // nodes, words of the link table, deepest level, sources
  const int N = std::atoi(argv[1]), n = std::atoi(argv[4]);
  std::printf("%d", node_pairs(N, std::atoi(argv[2]), std::atoi(argv[3]), n) ? node_cut(N, n).per_wg : 0);
}
"""


def test_cases_are_what_they_say(oracle, tmp_path):
    (tmp_path / "rule.cpp").write_text(RULE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2309_13541_amd", "csrc"), str(tmp_path / "rule.cpp"),
                    "-o", str(tmp_path / "rule")], check=True, timeout=120)
    for name, (make, _, cnt) in CASES.items():
        rp, col = make()
        degree = max(np.diff(rp).max(), np.bincount(col).max())  # the tables of both directions are equally wide
        words = next(w for w in (2, 3, 4, 5, 8) if degree <= 2 * w)
        depth = oracle.run(rp, col, want_dist=True, threads=8).dist.max()
        got = subprocess.run([str(tmp_path / "rule")] + [str(k) for k in (len(rp) - 1, words, depth, cnt)], check=True, capture_output=True,
                             text=True, timeout=60).stdout
        assert got == name.split(":")[0], (name, words, depth)


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_loads(oracle, name):
    import torch
    import paper_2309_13541_amd as a2a
    make, s0, cnt = CASES[name]
    csr = make()
    print(name, flush=True)
    topo = a2a.Topology(*csr)
    topo.profile_enable(1)
    got = []
    for flags in (a2a.WS_LOADS, a2a.WS_LOADS | a2a.WS_MINIMAL):
        ws = torch.full((topo.workspace_bytes(cnt, flags),), 0xff, dtype=torch.uint8, device="cuda")
        load = torch.full((topo.E,), -7.0, dtype=torch.float64, device="cuda")
        words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
        topo.link_loads(s0, cnt, load=load, dist_sum_total=words[:1], flags=words[1:], workspace=ws)
        torch.cuda.synchronize()
        got.append((load.cpu(), words.cpu()))
    # a source at a time in LDS, whatever the kernel: not the level kernels
    assert topo.profile_read()["sources"]["launches"] > 0
    topo.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    o = oracle.run(*csr, s0, cnt, threads=8)
    # sums of up to 2048 x 2048 positive terms in double precision, in two orders
    assert np.allclose(got[0][0].numpy(), o.load, rtol=1e-11, atol=0)
    assert int(got[0][1][0]) == int(o.dist_sum.sum()) and int(got[0][1][1]) == o.flags
