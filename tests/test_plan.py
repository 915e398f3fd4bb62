"""How calls are cut into workgroups (csrc/a2a_plan.h, plain host arithmetic), checked over the range of nodes, link table
widths, depths and source counts that the kernels take: no device needed, but for the call that shows the result."""
import os
import subprocess

import numpy as np
import pytest

import a2a_inputs as gen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include <cstdio>
#include "a2a_plan.h"
using namespace a2a_dev;

static long long bad = 0, seen = 0;
static void check(int N, int depth, int words, int n, SmallWhat what, int state) {
  const SmallCut c = small_cut(N, depth, words, n, what);
  ++seen;
  const bool sorts = what != SmallWhat::kDist;
  const bool ok = c.per >= 1 && c.tg >= kSmallWave && c.tg % kSmallWave == 0 && c.threads == c.per * c.tg &&
                  c.threads <= kSmallThreads &&                                     // what a launch may ask for
                  c.lds <= kSmallLds && (!sorts || c.lds >= small_lds_bytes(N, c.per, depth, state)) &&
                  c.nodes >= 1 && c.nodes <= small_most_nodes(what, words) && (long long)c.nodes * c.threads >= N &&
                  (what != SmallWhat::kSssp || N <= kSmallStripes * c.tg) &&
                  c.ts >= kSmallWave && c.ts <= c.tg && c.ts % kSmallWave == 0 &&
                  c.per_wg >= c.per && c.per_wg % c.per == 0 && c.per_wg <= kSmallBatch &&
                  c.workgroups >= 1 && (long long)c.workgroups * c.per_wg >= n && (long long)(c.workgroups - 1) * c.per_wg < n;
  if (!ok && ++bad <= 10)
    std::printf("N %d depth %d words %d sources %d what %d: %d sources x %d threads, %d nodes, %zu bytes, %d per workgroup, %d workgroups\n",
                N, depth, words, n, (int)what, c.per, c.tg, c.nodes, c.lds, c.per_wg, c.workgroups);
}

int main() {
  const int depths[] = {1, 2, 5, 12, 15, 16, 24, 60, 100, 167, 225, 253};
  const int words[] = {2, 3, 4, 5, 8};
  for (int N = 2; N <= kBothTables; N += N < 8300 ? 1 : 13)
    for (int depth : depths) {
      if (depth >= N) continue;
      const int sources[] = {1, 64, 255, 256, 511, 512, 700, 767, 768, 900, 1023, 1024, 1280, 1536, 2048, 4096, N - 1, N};
      for (int n : sources) {
        if (n < 1 || n > N) continue;
        if (N <= kScaledNodes) {
          for (int w : words)  // what link loads take: registers and LDS
            if (N <= small_max_nodes(w) * kSmallThreads && small_lds_bytes(N, 1, depth, kStateLoads) <= kSmallLds)
              check(N, depth, w, n, SmallWhat::kLoads, kStateLoads);
          if (small_lds_bytes(N, 1, depth, kStateSigma) <= kSmallLds) {
            check(N, depth, 2, n, SmallWhat::kSigma, kStateSigma);
            check(N, depth, 2, n, SmallWhat::kDist, 0);
          }
        }
        if (small_lds_bytes(N, 1, depth, kStateSssp) <= kSmallLds) check(N, depth, 2, n, SmallWhat::kSssp, kStateSssp);
      }
    }
  std::printf("%lld cuts, %lld bad\n", seen, bad);
  return bad != 0;
}
"""


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    def build(name, source):
        at = tmp_path_factory.mktemp(name)
        (at / "check.cpp").write_text(source)
        subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I" + os.path.join(ROOT, "paper_2309_13541_amd", "csrc"),
                        "-o", str(at / "check"), str(at / "check.cpp")], check=True)
        res = subprocess.run([str(at / "check")], stdout=subprocess.PIPE, text=True, timeout=300)
        print(res.stdout)
        return res
    return build


def test_cuts_fit_a_workgroup(compiled):
    """At most 1024 threads (three sources of a topology of 1921 to 2048 nodes once got 1152), within LDS, every node and
    every source with a place."""
    assert compiled("cuts", CHECK).returncode == 0


PIECES = r"""
#include <cstdio>
#include "a2a_plan.h"
using namespace a2a_dev;

int main() {
  long long bad = 0, seen = 0;
  for (long long nb64 = 4; nb64 <= 65536; nb64 += nb64 < 2100 ? 4 : 1024)  // up to 4 Mi nodes, a multiple of 256
    for (long long SB = 1; SB <= 2048; SB *= 2)
      for (long long levels = 1; levels <= nb64 * 64; levels = levels * 3 / 2 + 1) {
        const long long blocks = (SB + 7) / 8 * 8 * nb64;
        if (blocks * 512 > kMostThreads) continue;  // (more than 60 TB of masks)
        const long long each = offset_levels(SB * nb64, blocks, 512, (int)levels), pieces = (levels - 1 + each) / each;
        ++seen;
        if (each < 1 || each > levels || pieces * each < levels || pieces * blocks * 512 > kMostThreads)
          if (++bad <= 10) std::printf("%lld blocks of nodes, %lld super-batches, %lld levels: %lld a workgroup\n", nb64, SB, levels, each);
      }
  std::printf("%lld shapes, %lld bad\n", seen, bad);
  return bad != 0;
}
"""


def test_index_launches_stay_below_2_32_threads(compiled):
    assert compiled("pieces", PIECES).returncode == 0


BLOCKS = r"""
#include <cstdio>
#include "a2a_plan.h"
using namespace a2a_dev;

int main() {
  long long bad = 0, seen = 0;
  for (long long N = 1; N <= 4 << 20; N = N * 9 / 8 + 1)
    for (long long d = 0; d <= 64; d = d * 2 + 1) {
      const size_t ell = N <= 65536 && d <= 16 ? (size_t)N * 32 : 0;
      const HandleBlocks b = handle_blocks(N, N * d, ell, ell, 256, 1 << 17, 4096, 1024);
      bool ok = b.device >= b.upload + (1 << 17) && b.host >= 5120;
      for (int i = 0; i < kHandleParts; ++i)
        ok &= b.at[i] % 256 == 0 && b.at[i] + b.bytes[i] <= (i + 1 < kHandleParts ? b.at[i + 1] : b.upload);
      ok &= b.bytes[kOutCol] >= 4 && b.bytes[kInPtr] == ((size_t)N + 1) * 4 && b.bytes[kInLink] >= (size_t)(N * d) * 4;
      // pinned memory: a copy of the upload only where it is small
      ok &= b.staged ? b.slots >= b.upload && b.host <= kStagedBytes + 5120 : b.slots == 0 && b.host <= 5120;
      ++seen;
      if (!ok && ++bad <= 10) std::printf("N %lld degree %lld: upload %zu host %zu\n", N, d, b.upload, b.host);
    }
  std::printf("%lld handles, %lld bad\n", seen, bad);
  return bad != 0;
}
"""


def test_pinned_memory_of_a_handle(compiled):
    """A handle holds no pinned copy of a large upload."""
    assert compiled("blocks", BLOCKS).returncode == 0


def bottleneck(n, sources, chain):
    """`sources` nodes in a tree of eight links a node to its root, a chain from there, two equal ways at its end, and a
    tree of eight links a node to all the others: every commodity of the first nodes to the last ones takes the chain."""
    rows = [[(i - 1) // 8] if i > 0 else [sources] for i in range(sources)]
    rows += [[sources + i + 1] for i in range(chain - 1)] + [[sources + chain, sources + chain + 1]]
    rows += [[sources + chain + 2]] * 2
    first, last = sources + chain + 2, n
    rows += [[w for w in range(first + 8 * (v - first) + 1, first + 8 * (v - first) + 9) if w < last] for v in range(first, last)]
    return gen.csr_from_rows(rows)


@pytest.mark.gpu
@pytest.mark.parametrize("over", [0, 1])
def test_single_path_costs_near_2_32(oracle, over):
    """The most sources whose costs are kept in 32 bits, and one more: costs come to 3.05e9, and the choice between the
    two ways behind the chain is made on sums of that size."""
    import paper_2309_13541_amd as a2a
    from test_sssp import run_sssp_gpu
    rp, col = bottleneck(8191, 2100, 242)
    topo = a2a.Topology(rp, col)
    assert topo.level_bound == 253  # as deep as the kernels with 32-bit costs take
    sources = (2 ** 32 - 2) // (topo.level_bound * (topo.N - 1)) + over
    assert sources <= 2100
    want, dsum, unr = oracle.sssp(rp, col, 0, sources, iter_sources=64)
    assert 2 ** 31 < 242 * int(want[2100]) < 2 ** 32  # the chain's first link
    load, got_sum, flags = run_sssp_gpu(topo, 0, sources, iter_sources=64)
    assert np.array_equal(load, want.astype(np.float64))
    assert got_sum == int(dsum.sum()) and flags == (a2a.FLAG_UNREACHABLE if unr else 0)
    topo.close()


@pytest.mark.gpu
def test_path_counts_of_ten_thousand_levels():
    """A bidirectional ring of 20000 nodes: the index entries of its levels take more than one level a workgroup."""
    import paper_2309_13541_amd as a2a
    from gpu_helpers import run_distances
    n, s0, cnt = 20000, 77, 3
    topo = a2a.Topology(*gen.bidirectional_ring(n))
    dist, sigma, dsum, unr, flags = run_distances(topo, s0, cnt)
    for i in range(cnt):
        away = (np.arange(n) - (s0 + i)) % n
        want = np.minimum(away, n - away)
        assert np.array_equal(dist[i], want) and np.array_equal(sigma[i], np.where(want == n // 2, 2.0, 1.0))
        assert dsum[i] == want.sum()
    assert unr == 0 and flags == 0
    topo.close()


NODES = r"""
#include <cstdio>
#include "a2a_plan.h"
using namespace a2a_dev;

int main() {
  long long bad = 0, seen[2] = {};
  for (int N = 1; N <= kScaledNodes; ++N)
    for (int words : {2, 3, 4, 5, 8})
      for (int depth : {0, 1, 10, 11, 253})
        for (int n : {1, 2, 255, 256, 257, 511, 512, 513, 1024, 1280, 1536, N - 1, N}) {
          for (int sources = 1; sources <= 2; ++sources) {  // at a time
            if (n < 1 || n > N || !(sources == 2 ? node_pairs(N, words, depth, n) : node_fits(N, words, depth, n))) continue;
            const NodeCut c = node_cut(N, n);
            ++seen[sources - 1];
            const int most = sources == 2 ? (words <= 4 ? kNodeMost : words <= 5 ? 1 : 0) : words <= 5 ? kNodeMost : 1;  // nodes that are built for
            const size_t lds = node_lds_bytes(N, c.nodes, sources, words), each = (size_t)node_places(N) * 8 * sources;  // of an array
            const bool ok = c.threads >= kSmallWave && c.threads % kSmallWave == 0 && c.threads <= kSmallThreads &&
                            c.nodes >= 1 && c.nodes <= most && c.nodes * c.threads >= N &&
                            node_places(N) >= N && each <= (size_t)node_apart(c.nodes, sources, words) && each <= 0x10000 &&  // places have 16 bits
                            node_apart(c.nodes, sources, words) % (8 * sources) == 0 &&
                            lds >= 3 * (size_t)node_apart(c.nodes, sources, words) + each + c.threads / kSmallWave * 32 &&
                            lds <= kSmallLds && c.per_wg >= sources && c.workgroups <= kComputeUnits &&
                            (long long)c.workgroups * c.per_wg >= n && (long long)(c.workgroups - 1) * c.per_wg < n;
            if (!ok && ++bad <= 10) std::printf("N %d words %d depth %d sources %d, %d at a time\n", N, words, depth, n, sources);
          }
        }
  std::printf("%lld and %lld cuts, %lld bad\n", seen[0], seen[1], bad);
  return bad != 0 || seen[0] == 0 || seen[1] == 0;
}
"""


def test_a_thread_per_node_fits_a_workgroup(compiled):
    assert compiled("nodes", NODES).returncode == 0


EDGES = r"""
#include <cstdio>
#include "a2a_plan.h"
using namespace a2a_dev;

int main() {
  // nodes, words of the link table, levels, sources, whether k_node_loads was the faster one when both were timed, a source at a time
  const int measured[][5] = {
      {256, 4, 4, 256, 1},   {1024, 2, 68, 512, 1},  {500, 2, 250, 500, 1},  {1000, 3, 15, 768, 1},  {576, 2, 24, 576, 0},
      {702, 2, 26, 702, 0},  {729, 3, 12, 729, 1},   {1024, 5, 10, 1024, 1}, {1024, 4, 12, 1024, 0}, {1000, 3, 15, 1000, 0},
      {2000, 4, 5, 256, 1},  {2024, 2, 45, 256, 1},  {1520, 2, 39, 512, 1},  {1500, 2, 152, 512, 1}, {2048, 3, 24, 512, 1},
      {2040, 2, 61, 512, 1}, {2048, 2, 132, 512, 1}, {1600, 2, 40, 512, 0},  {2025, 2, 44, 400, 0},  {1776, 2, 49, 400, 0},
      {2048, 2, 9, 768, 1},  {1536, 5, 11, 768, 1},  {1296, 4, 12, 768, 0},  {1331, 3, 15, 768, 0},  {1300, 3, 6, 1024, 1},
      {2048, 4, 5, 1024, 1}, {1536, 2, 8, 1024, 0},  {1100, 2, 9, 1024, 0},  {1050, 4, 10, 896, 0},  {1080, 4, 11, 1080, 1},
      {1536, 2, 9, 1536, 1}, {1296, 4, 12, 1296, 0}, {1600, 2, 10, 1600, 0}, {2048, 2, 8, 2048, 0}};
  int bad = 0;
  for (const auto& m : measured)
    if (node_fits(m[0], m[1], m[2], m[3]) != (m[4] != 0)) {
      std::printf("%d nodes, %d words, %d levels, %d sources: not %d\n", m[0], m[1], m[2], m[3], m[4]);
      ++bad;
    }
  const int pairs[][5] = {  // two at a time against the faster of the others
      {1024, 2, 32, 512, 1}, {1000, 3, 15, 512, 1},  {1000, 4, 5, 512, 1},   {1024, 5, 10, 512, 1},  {1000, 2, 9, 768, 0},
      {1000, 3, 15, 768, 0}, {1024, 3, 16, 1000, 1}, {1024, 5, 10, 1024, 1}, {1024, 4, 4, 1024, 1},  {1024, 2, 32, 1024, 0},
      {1520, 2, 39, 512, 1}, {2028, 3, 18, 512, 1},  {1300, 4, 5, 512, 0},   {1800, 4, 5, 512, 0},   {2000, 2, 8, 1024, 1},
      {1300, 3, 6, 1024, 1}, {1296, 4, 12, 1024, 0}, {1800, 4, 5, 1024, 0},  {1300, 3, 6, 1280, 0},  {2000, 2, 8, 1280, 1},
      {2000, 4, 5, 1280, 1}, {2000, 2, 8, 1500, 1},  {1368, 4, 4, 1368, 1},  {1331, 3, 15, 1331, 0}, {2000, 4, 5, 1700, 1},
      {1800, 4, 4, 1800, 1}, {2000, 4, 5, 2000, 1},  {2000, 2, 8, 2000, 0}};
  for (const auto& m : pairs)
    if (node_pairs(m[0], m[1], m[2], m[3]) != (m[4] != 0)) {
      std::printf("%d nodes, %d words, %d levels, %d sources: not %d, two at a time\n", m[0], m[1], m[2], m[3], m[4]);
      ++bad;
    }
  return bad != 0;
}
"""


def test_a_thread_per_node_where_it_was_faster(compiled):
    out = compiled("edges", EDGES)
    assert out.returncode == 0, out.stdout
