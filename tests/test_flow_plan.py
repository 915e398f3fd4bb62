"""Where the kernels that take one source at a time through a workgroup's LDS lay things out (csrc/a2a_plan.h, plain host
arithmetic), over the nodes, depths and workspaces they are given: no device needed."""
import os
import subprocess

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
  for (int N = 2; N <= kFlowNodes + 5; ++N) {
    const size_t S = (size_t)flow_stride(N);
    for (int depth = 1; depth <= 16; ++depth) {
      const size_t places = (size_t)(8 * (depth <= 8 ? 1 : 2) + 1) * 2 * 1024;  // positions of the sort
      if (flow_sssp_fits(N, depth, 64)) {
        const size_t q = flow_sssp_queue(N, depth), end = q + (S + 32) * 4 + 512, lds = flow_sssp_lds(N, depth);
        const bool apart = flow_sssp_apart(N, depth);
        check(lds <= kSmallLds && q % 16 == 0 && q >= S * 4 && lds >= (apart ? end + places : end) && (apart || q >= places),
              "single path", N, depth, apart);
        check(depth <= 16 && N <= 4 * kFlowWords * 1024 && N <= 1 << 14, "single path, sort and entries", N, depth, 0);
      }
      for (int demand = 0; demand < 2; ++demand)
        if (N <= kFlowNodes && depth <= kFlowDeepest && flow_lds_fits(N, depth, demand)) {
          // [from, to) of what is in LDS at a time: sort and forward sweep (positions only in the first), backward sweep
          const FlowKeep keep = flow_keep(N, depth, demand);
          const bool memory = keep == FlowKeep::kMemory, records = keep == FlowKeep::kRecords;
          const size_t lds = flow_source_lds(N, depth, demand), tail = flow_tail_at(N, depth, keep, demand);
          const size_t queue = (memory ? 4 : 8) * S, paths = queue + (S + 32) * 2;
          const size_t behind = paths + (records ? 4 * S : 0), base = !memory && flow_gap(N, depth) ? 4 * S : behind;
          const size_t dem = flow_demand_at(N, depth);
          check(memory || !demand, "demands go through memory", N, depth, demand);
          check(base >= 4 * S && (base + places <= queue || base >= behind) && base + places <= (demand ? dem : tail), "positions", N, depth, (int)keep);
          check(behind <= (demand ? dem : tail) && (memory || queue >= 8 * S) && 8 * S <= (demand ? dem : tail), "queue, path counts, doubles", N, depth, (int)keep);
          check(!demand || (dem % 16 == 0 && dem >= 8 * S && dem + 8 * S <= tail && 16 * S <= tail), "demands", N, depth, demand);
          check(tail % 8 == 0 && queue % 16 == 0 && paths % 4 == 0 && base % 2 == 0 && lds >= tail + 16 * (8 + 32) && lds <= 160 * 1024 &&
                flow_link_lds(N) <= kSmallLds, "sources", N, depth, demand);
          check(N > kScaledNodes || demand || records, "with 8 x id in the tables all of it stays", N, depth, 0);
        }
    }
  }
  check(flow_keep(11584, 11, false) == FlowKeep::kRecords && flow_keep(11585, 5, false) == FlowKeep::kQueue &&
        flow_keep(16256, 11, false) == FlowKeep::kQueue && flow_keep(16257, 5, false) == FlowKeep::kMemory, "where the forms change", 0, 0, 0);
  const int nodes[] = {5121, 8191, 8192, 10176, 16384, 20000, kFlowNodes}, words[] = {2, 3, 4, 5, 8};
  for (int N : nodes)
    for (int w : words)
      for (int n : {kFlowFewestSources, 1025, 2501, 5000, N})
        for (int demand = 0; demand < 2; ++demand) {
          if (n > N) continue;
          const FlowGroups g = flow_groups(N, w, n);
          check(g.group >= 1 && (long long)g.group * g.groups >= n && (long long)g.group * (g.groups - 1) < n &&
                (long long)g.blocks * flow_nodes(w) * 1024 >= N, "groups", N, w, n);
          const size_t all = flow_layout(N, w, n, demand, ~(size_t)0).total;
          for (int part = 0; part <= 64; ++part) {
            const size_t bytes = all / 64 * part + (part == 64 ? all % 64 : 0);
            const FlowLayout l = flow_layout(N, w, n, demand, bytes);
            const bool whole = l.rows == n || (l.rows > 0 && l.rows % g.group == 0) || l.rows < g.group;
            check((l.rows == 0 || l.total <= bytes) && l.rows <= n && whole && (long long)l.parts * g.group >= l.rows &&
                  (part < 64 || l.rows == n), "layout", N, n, part);
            // pieces: no more than the largest take, and among as many no fewer rounds of 256 sources
            const auto fits = [&](int k) { return flow_layout_for(N, w, n, demand, std::min(k * g.group, n), k).total <= bytes; };
            const auto rounds = [&](int rows) { return n / rows * ((rows + 255) / 256) + (n % rows + 255) / 256; };
            if (part % 8 == 3 && l.rows >= g.group)
              for (int k = 1; k <= g.groups && fits(k); ++k) {
                const int rows = std::min(k * g.group, n), pieces = (n + rows - 1) / rows, has = (n + l.rows - 1) / l.rows;
                check(has < pieces || (has == pieces && rounds(l.rows) <= rounds(rows)), "pieces", N, n, k);
              }
          }
        }
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
