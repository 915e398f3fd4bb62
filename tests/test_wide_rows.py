"""Distances of a workgroup whose waves store the same row at a time, and of one whose waves store by themselves: that the rule takes the
cases one way or the other, and the same matrix as in calls of few sources, which never store together.  (Matrices need an MI355X.)"""
import os
import subprocess

import numpy as np
import pytest

import a2a_inputs as gen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def thinned(n, d, seed):
    """Random out-lists, a tenth of the links gone, and every link into the last 20 nodes: those are out of reach."""
    rp, col = gen.random_regular(n, d, seed)
    off = np.random.default_rng(seed).random(len(col)) < 0.1
    off |= col >= n - 20
    return gen.remove_arcs((rp, col), np.flatnonzero(off))


# topology, first source and sources; sources a word and a bound on the levels; whether rows are stored together
CASES = {
    "odd rows, 64 a word": (lambda: gen.random_regular(8501, 4, 1), 0, 8501, 64, 12, True),
    "odd rows, 32 a word, last group of one": (lambda: gen.random_regular(12301, 5, 2), 3, 32 * 178 + 1, 32, 9, True),
    "odd rows, 16 a word": (lambda: gen.random_regular(20011, 5, 3), 7, 3501, 16, 9, True),
    "odd rows, out of reach": (lambda: thinned(33001, 6, 4), 0, 16 * 133 + 2, 16, 12, True),
    "odd rows, few": (lambda: gen.random_regular(33001, 6, 5), 0, 1199, 16, 9, False),
    "odd rows, fewest": (lambda: gen.random_regular(40004, 6, 5), 30, 1200, 16, 9, True),
    "half lines, most nodes": (lambda: gen.random_regular(65528, 3, 6), 60000, 1203, 16, 17, True),
    "whole lines, 64 a word": (lambda: gen.random_regular(16384, 3, 7), 0, 16384, 64, 15, False),
    "whole lines, 3 bits": (lambda: gen.random_regular(50000, 12, 8), 11, 45001, 16, 6, True),
    "whole lines, most nodes": (lambda: gen.random_regular(65536, 3, 9), 63000, 2000, 16, 17, True),
    "whole lines, fewer nodes": (lambda: gen.random_regular(61984, 3, 9), 59000, 2100, 16, 17, False),
    "whole lines, many levels": (lambda: gen.torus([40, 40, 40]), 0, 5470, 16, 60, True),
}

RULE = r"""
#include <cstdio>
#include <cstdlib>
#include "a2a_plan.h"

int main(int argc, char** argv) {  // nodes, sources, sources a word, deepest level
  std::printf("%d", a2a_dev::wide_together(std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4])) ? 1 : 0);
}
"""


def test_rule(tmp_path):
    (tmp_path / "rule.cpp").write_text(RULE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2309_13541_amd", "csrc"), str(tmp_path / "rule.cpp"),
                    "-o", str(tmp_path / "rule")], check=True, timeout=120)

    def rule(*args):
        return subprocess.run([str(tmp_path / "rule")] + [str(x) for x in args], check=True, capture_output=True, text=True, timeout=60).stdout == "1"

    for name, (make, _, cnt, W, depth, together) in CASES.items():
        n = len(make()[0]) - 1
        assert rule(n, cnt, W, depth) == together, name
        assert not rule(n, 512, W, depth), name  # the calls that the matrices are compared with
    # nodes, sources, sources a word, levels, whether together was the faster one when both were timed
    for n, cnt, W, depth, faster in ((40001, 40001, 16, 7, 1), (20011, 300, 16, 9, 0), (9000, 9000, 64, 6, 1), (44444, 900, 16, 14, 0),
                                     (8260, 8260, 64, 6, 0), (36000, 36000, 16, 7, 0), (60000, 60000, 16, 15, 0), (65536, 4096, 16, 13, 1), (53248, 53248, 16, 7, 1),
                                     (52000, 20800, 16, 7, 0), (16384, 16384, 64, 7, 0), (46656, 46656, 16, 54, 1), (46656, 4665, 16, 54, 0),
                                     (13824, 13824, 64, 36, 0), (32768, 10922, 32, 48, 1)):
        assert rule(n, cnt, W, depth) == bool(faster), (n, cnt, W, depth)


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_matrix(oracle, name):
    import torch
    import paper_2309_13541_amd as a2a
    make, s0, cnt = CASES[name][:3]
    csr = make()
    print(name, flush=True)
    topo = a2a.Topology(*csr)

    def run(first, count):
        ws = torch.full((topo.workspace_bytes(count, a2a.WS_DISTANCES),), 0xff, dtype=torch.uint8, device="cuda")
        dist = torch.full((count, topo.N), -7, dtype=torch.int32, device="cuda")
        sums = torch.full((count,), -7, dtype=torch.int64, device="cuda")
        words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
        topo.distances(first, count, dist=dist, dist_sum=sums, unreachable=words[:1], flags=words[1:], workspace=ws)
        return dist, sums, words

    dist, sums, words = run(s0, cnt)
    gone, flags = 0, 0
    for first in range(0, cnt, 512):
        n = min(512, cnt - first)
        part = run(s0 + first, n)
        assert torch.equal(dist[first:first + n], part[0]) and torch.equal(sums[first:first + n], part[1]), first
        gone, flags = gone + int(part[2][0]), flags | int(part[2][1])
    assert int(words[0]) == gone and int(words[1]) == flags
    topo.close()
    for first in (0, cnt - 8):  # both ends against the oracle
        o = oracle.run(*csr, s0 + first, 8, want_dist=True, threads=8)
        assert np.array_equal(dist[first:first + 8].cpu().numpy(), o.dist)
        assert np.array_equal(sums[first:first + 8].cpu().numpy(), o.dist_sum)
