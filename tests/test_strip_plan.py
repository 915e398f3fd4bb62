"""Where k_strip_sources and k_flow_links after it lay things out (csrc/a2a_plan.h, plain host arithmetic), over all nodes and
depths and over workspaces: no device needed."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include <cstdio>
#include "a2a_plan.h"
using namespace a2a_dev;

int main() {
  long long bad = 0, seen = 0;
  const auto check = [&](bool ok, const char* what, int N, int x, int y) {
    ++seen;
    if (!ok && ++bad <= 10) std::printf("%s: N %d, %d, %d\n", what, N, x, y);
  };
  for (int N = 8192; N <= 65536; ++N) {
    const long long S = flow_stride(N), state = (long long)kStripState;
    const int words = (N + 4095) / 4096;
    const StripCut c = strip_cut(N);
    check(words <= kStripWords && c.count >= 1 && c.count <= kStripMost && c.nodes == c.threads * 4 * words &&
          (long long)c.nodes * c.count >= N && (c.count - 1) * c.threads < 1024 && (long long)c.nodes * (c.count - 1) < N,
          "strips", N, c.count, c.nodes);
    check(8ll * c.nodes + 16 <= c.bits && c.bits % 16 == 0 && c.before - c.bits >= (N + 31) / 32 * 4 && (c.before - c.bits) % 16 == 0 &&
          c.few - c.before >= (N + 31) / 32 * 2 && c.few % 8 == 0 && c.few + 8ll * c.most <= state && c.most >= kStripFewLeast &&
          c.most <= kStripFew, "few", N, c.most, c.few);
    check((long long)strip_link_lds(N) >= 2 * S * (strip_links_single(N) ? 1 : 2) && strip_link_lds(N) <= kSmallLds, "links", N, 0, 0);
    for (int depth = 1; depth <= kStripDeepest + 1; ++depth) {
      if (!strip_lds_fits(N, depth)) continue;
      const int levels = strip_levels(depth), bits = strip_count_bits(depth);
      check(levels >= depth && levels <= 16 && 2 * S + (levels + 1) * 2048 <= state, "sort", N, depth, levels);
      check((depth << bits | ((1 << bits) - 1)) < 65536, "a node's word", N, depth, bits);
    }
  }
  check(strip_lds_fits(65536, 12) && strip_lds_fits(60000, 15) && !strip_lds_fits(60000, 16) && !strip_lds_fits(65537, 5), "range", 0, 0, 0);
  const int nodes[] = {10177, 20353, 40704, 40705, 65536}, words[] = {2, 3, 4, 5, 8};
  for (int N : nodes)
    for (int w : words)
      for (int n : {kStripFewestSources, 2501, 10000, N}) {
        if (n > N) continue;
        const FlowGroups g = flow_groups(N, w, n, true);
        check(g.group >= 1 && g.group <= 256 && (long long)g.group * g.groups >= n && (long long)g.group * (g.groups - 1) < n, "groups", N, w, n);
        const FlowLayout whole = flow_layout(N, w, n, true, ~(size_t)0, true);
        const size_t S = (size_t)flow_stride(N);
        check(whole.rows == n && whole.part - whole.record >= 256 * strip_record_bytes((int)S) && whole.exact - whole.escaped >= 4 * (size_t)n &&
              whole.count - whole.exact >= 4 * S * n && whole.coef - whole.count >= 2 * S * n && whole.total - whole.coef >= 8 * S * n,
              "whole layout", N, w, n);
        for (int part = 0; part < 64; ++part) {
          const size_t bytes = whole.total / 64 * part;
          const FlowLayout l = flow_layout(N, w, n, true, bytes, true);
          check((l.rows == 0 || l.total <= bytes) && (l.rows % g.group == 0 || l.rows < g.group), "layout", N, n, part);
        }
      }
  // nodes, words, groups, whether two nodes a thread were the faster ones when both were timed
  const int narrow[][4] = {{65536, 4, 1, 1}, {65536, 4, 7, 1},  {65536, 4, 11, 0}, {45000, 2, 8, 1},  {45000, 2, 10, 0}, {45000, 2, 11, 0},
                           {24000, 4, 16, 1}, {24000, 4, 19, 0}, {33000, 4, 7, 1},  {33000, 4, 10, 0}, {33000, 4, 11, 0}, {50000, 3, 7, 1},
                           {50000, 3, 10, 0}, {30000, 2, 12, 1}, {30000, 2, 17, 0}, {20353, 2, 24, 1}, {40000, 8, 1, 0}};
  for (const auto& m : narrow) check(strip_links_narrow(m[0], m[1], m[2]) == (m[3] != 0), "two nodes a thread", m[0], m[1], m[2]);
  std::printf("%lld checks, %lld bad\n", seen, bad);
  return bad != 0;
}
"""


def test_layouts_over_their_range(tmp_path):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(CHECK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2309_13541_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(out.stdout)
    assert out.returncode == 0, out.stdout


ROWS = r"""
#include <cstdio>
#include <cstdlib>
#include "a2a_plan.h"
using namespace a2a_dev;

int main(int argc, char** argv) {  // nodes, words of the link table, deepest level; 1: after a search
  const int N = std::atoi(argv[1]), words = std::atoi(argv[2]), depth = std::atoi(argv[3]);
  if (std::atoi(argv[4]) != 0)
    std::printf("%d", flow_groups(N, words, N, N > kFlowNodes).groups);
  else
    std::printf("%d", node_pairs(N, words, depth, N) || node_fits(N, words, depth, N) ? node_cut(N, N).workgroups
                                                                                    : small_cut(N, depth, words, N, SmallWhat::kLoads).workgroups);
}
"""


def test_rows_of_partial_loads_that_the_benchmark_counts(tmp_path):
    sys.path.insert(0, ROOT)
    import bench
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(ROWS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2309_13541_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    for nodes, degree, words, depth, search in ((64, 4, 2, 8, 0), (1024, 10, 5, 10, 0), (4096, 6, 3, 24, 0), (16384, 4, 2, 7, 1), (20352, 6, 3, 7, 1),
                                                (20353, 6, 3, 7, 1), (40000, 16, 8, 5, 1), (65536, 8, 4, 7, 1)):
        rows = subprocess.run([str(exe), str(nodes), str(words), str(depth), str(search)], check=True, capture_output=True, text=True, timeout=60).stdout
        assert bench.partial_rows(nodes, degree, bool(search)) == int(rows), (nodes, degree)
