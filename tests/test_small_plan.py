"""How calls on small topologies are cut into workgroups (csrc/a2a_small_plan.h, plain host arithmetic), checked over the
range of nodes, link table widths, depths and source counts that the kernels take: no device needed."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include <cstdio>
#include "a2a_small_plan.h"
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
