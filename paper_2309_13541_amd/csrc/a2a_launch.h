// Launches of the kernels that are compiled for a width of the link tables.  a2a_words.hip defines them, one translation
// unit per width (A2A_WORDS), compiled side by side: in one unit they took 140 s, more than all else together.
#pragma once

#include <type_traits>

#include "a2a_flow_kernels.h"
#include "a2a_small_kernels.h"
#include "a2a_wide_kernels.h"

namespace a2a_dev {

// How a call is cut up (SmallCut), with the tables.
struct SmallPlan {
  SmallView sv{};
  int T = 0, workgroups = 0, nodes = 0;  // threads, workgroups of the whole call, nodes per thread
  int at_a_time = 0;                     // sources of k_node_loads; 0: another kernel
  size_t lds = 0;
};

template <int KS>
void launch_small_loads(const SmallPlan& p, bool demand, int workgroups, hipStream_t st);
template <int KS>
void launch_node_loads(const SmallPlan& p, bool demand, int workgroups, hipStream_t st);
template <int KS>
void launch_small_outputs(const SmallPlan& p, const SmallOut& out, int workgroups, hipStream_t st);
template <int KS>
void launch_small_levels(const SmallPlan& p, int workgroups, hipStream_t st);
template <int KS>
void launch_small_sssp(const SmallPlan& p, const SmallSssp& ss, hipStream_t st);
template <int KS>
void launch_flow_sssp(const SmallPlan& p, const SmallSssp& ss, int workgroups, hipStream_t st);
template <int KS>
void launch_small_sssp_add(const SmallPlan& p, const SmallSssp& ss, hipStream_t st);
// W sources a word; out: kWideDist (16, 32 or 64; without a matrix its sums alone) or kWideBytes (16 or 64).
template <int KS>
void launch_wide_search(const WideView& wv, int W, int out, int workgroups, hipStream_t st);
// Newly reached of every level; W: 16 or 64.
template <int KS>
void launch_wide_masks(const WideView& wv, int W, int workgroups, hipStream_t st);
template <int KS>
void launch_wide_sigma(const WideSigma& ws, int workgroups, hipStream_t st);
template <int KS>
void launch_flow_sources(const FlowView& fv, bool demand, int workgroups, hipStream_t st);
template <int KS>
void launch_strip_sources(const FlowView& fv, int workgroups, hipStream_t st);
// fv.exact: null after launch_flow_sources.  (With demands only after that.)
template <int KS>
void launch_flow_links(const FlowView& fv, bool demand, hipStream_t st);

// f(KS), a constant, for a table of that many words a node.
template <typename F>
void by_words(int words, F&& f) {
  switch (words) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
  }
}

}  // namespace a2a_dev
