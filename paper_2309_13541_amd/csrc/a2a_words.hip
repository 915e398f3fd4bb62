// The launches of a2a_launch.h for link tables of A2A_WORDS words a node.
#include <hip/hip_runtime.h>

#include "a2a_launch.h"

#ifndef A2A_WORDS
#error "A2A_WORDS: words of the link tables (2, 3, 4, 5 or 8)"
#endif

namespace a2a_dev {

namespace {

template <int KS, bool kDemand>
void small_loads(const SmallPlan& p, int workgroups, hipStream_t st) {
  const auto launch = [&](auto nodes) {
    constexpr int kNodes = decltype(nodes)::value;
    k_small_loads<KS, kNodes, kDemand><<<workgroups, p.T, std::max(p.lds, small_search_bytes(p.sv.N, kNodes)), st>>>(p.sv);
  };
  if (p.nodes <= 1)
    launch(std::integral_constant<int, 1>{});
  else if (p.nodes <= 2)
    launch(std::integral_constant<int, 2>{});
  else if (KS <= 5 && p.nodes <= 4)
    launch(std::integral_constant<int, KS <= 5 ? 4 : 2>{});
  else
    launch(std::integral_constant<int, small_max_nodes(KS)>{});
}

template <int W, int KS, int kOut>
void wide_search(const WideView& wv, int workgroups, hipStream_t st) {
  const size_t lds = wide_words_bytes(wv.slots) + (size_t)wv.list * 2;
  const auto launch = [&](auto kernel) { kernel<<<workgroups, kWideThreads, lds, st>>>(wv); };
  if (kOut != kWideBytes && wv.depth < 8)
    launch(k_wide_dist<W, KS, kOut != kWideBytes ? 3 : 6, kOut>);
  else
    launch(k_wide_dist<W, KS, 6, kOut>);
}

}  // namespace

template <int KS>
void launch_small_loads(const SmallPlan& p, bool demand, int workgroups, hipStream_t st) {
  demand ? small_loads<KS, true>(p, workgroups, st) : small_loads<KS, false>(p, workgroups, st);
}

template <int KS>
void launch_node_loads(const SmallPlan& p, bool demand, int workgroups, hipStream_t st) {
  const auto launch = [&](auto kernel) { kernel<<<workgroups, p.T, p.lds, st>>>(p.sv); };
  constexpr int kTwo = KS <= 5 ? 2 : 1, kTwoPair = KS <= 4 ? 2 : 1, kPair = KS <= 5 ? 2 : 1;  // (node_fits, node_pairs)
  if (p.at_a_time == 2)
    p.nodes == 1 ? launch(k_node_loads<KS, 1, kPair, false>) : launch(k_node_loads<KS, kTwoPair, kPair, false>);
  else if (p.nodes == 1)
    demand ? launch(k_node_loads<KS, 1, 1, true>) : launch(k_node_loads<KS, 1, 1, false>);
  else
    demand ? launch(k_node_loads<KS, kTwo, 1, true>) : launch(k_node_loads<KS, kTwo, 1, false>);
}

template <int KS>
void launch_small_outputs(const SmallPlan& p, const SmallOut& out, int workgroups, hipStream_t st) {
  const auto launch = [&](auto nodes) {
    constexpr int kNodes = decltype(nodes)::value;
    if (out.sigma != nullptr)
      k_small_sigma<KS, kNodes><<<workgroups, p.T, std::max(p.lds, small_search_bytes(p.sv.N, kNodes)), st>>>(p.sv, out);
    else
      k_small_dist<KS, kNodes><<<workgroups, p.T, small_dist_bytes(p.sv.N, kNodes), st>>>(p.sv, out);
  };
  if (p.nodes <= 1)
    launch(std::integral_constant<int, 1>{});
  else if (p.nodes <= 2)
    launch(std::integral_constant<int, 2>{});
  else if (p.nodes <= 4)
    launch(std::integral_constant<int, 4>{});
  else
    launch(std::integral_constant<int, 8>{});
}

template <int KS>
void launch_small_levels(const SmallPlan& p, int workgroups, hipStream_t st) {
  const int nodes = (p.sv.N + kSmallThreads - 1) / kSmallThreads;
  const auto launch = [&](auto kernel, int most) {
    kernel<<<workgroups, kSmallThreads, small_search_bytes(p.sv.N, most), st>>>(p.sv);
  };
  if (p.sv.N > kScaledNodes)
    launch(k_small_levels<KS, 16, 4, true>, 16);
  else if (nodes <= 2)
    launch(k_small_levels<KS, 2, kSmallPlanes, false>, 2);
  else
    launch(k_small_levels<KS, 8, kSmallPlanes, false>, 8);
}

template <int KS>
void launch_small_sssp(const SmallPlan& p, const SmallSssp& ss, hipStream_t st) {
  k_small_sssp<KS><<<p.workgroups, p.T, p.lds, st>>>(p.sv, ss);
}

template <int KS>
void launch_flow_sssp(const SmallPlan& p, const SmallSssp& ss, int workgroups, hipStream_t st) {
  const auto launch = [&](auto kernel) {
    kernel<<<workgroups, kWideThreads, flow_sssp_lds(p.sv.N, p.sv.depth), st>>>(p.sv, ss);
  };
  if (p.sv.N <= kScaledNodes)
    launch(k_flow_sssp<KS, true>);
  else
    launch(k_flow_sssp<KS, false>);
}

template <int KS>
void launch_small_sssp_add(const SmallPlan& p, const SmallSssp& ss, hipStream_t st) {
  k_small_sssp_add<KS><<<(p.sv.N + kWave - 1) / kWave, kSmallThreads, 0, st>>>(ss, p.sv.N, p.sv.src_count);
}

template <int KS>
void launch_wide_search(const WideView& wv, int W, int out, int workgroups, hipStream_t st) {
  if (out == kWideBytes)
    return W == 16 ? wide_search<16, KS, kWideBytes>(wv, workgroups, st) : wide_search<64, KS, kWideBytes>(wv, workgroups, st);
  const auto search = [&](auto w) {
    constexpr int kW = decltype(w)::value;
    wv.dist != nullptr ? wide_search<kW, KS, kWideDist>(wv, workgroups, st) : wide_search<kW, KS, kWideSums>(wv, workgroups, st);
  };
  switch (W) {
    case 16: return search(std::integral_constant<int, 16>{});
    case 32: return search(std::integral_constant<int, 32>{});
    default: return search(std::integral_constant<int, 64>{});
  }
}

template <int KS>
void launch_wide_masks(const WideView& wv, int W, int workgroups, hipStream_t st) {
  const size_t lds = (size_t)wv.slots * kWideThreads * sizeof(uint32_t);
  const auto launch = [&](auto kernel) { kernel<<<workgroups, kWideThreads, lds, st>>>(wv); };
  if (W == 16)
    launch(k_wide_dist<16, KS, 6, kWideMasks>);
  else if (wv.N > kScaledNodes)
    launch(k_wide_dist<64, KS, 6, kWideMasks>);
  else
    launch(k_wide_dist<64, KS, 6, kWideMasks, true>);
}

template <int KS>
void launch_wide_sigma(const WideSigma& ws, int workgroups, hipStream_t st) {
  k_wide_sigma<KS><<<workgroups, kWideThreads, wide_state_bytes(ws.N), st>>>(ws);
}

template <int KS>
void launch_flow_sources(const FlowView& fv, bool demand, int workgroups, hipStream_t st) {
  const size_t lds = flow_source_lds(fv.N, fv.depth, demand);
  const auto launch = [&](auto kernel) { kernel<<<workgroups, kWideThreads, lds, st>>>(fv); };
  static_assert(flow_keep(kScaledNodes, kFlowDeepest, false) == FlowKeep::kRecords);
  if (fv.N <= kScaledNodes) {
    demand ? launch(k_flow_sources<KS, true, true, FlowKeep::kMemory>) : launch(k_flow_sources<KS, true, false, FlowKeep::kRecords>);
    return;
  }
  switch (flow_keep(fv.N, fv.depth, demand)) {
    case FlowKeep::kRecords: return launch(k_flow_sources<KS, false, false, FlowKeep::kRecords>);
    case FlowKeep::kQueue: return launch(k_flow_sources<KS, false, false, FlowKeep::kQueue>);
    case FlowKeep::kMemory:
      demand ? launch(k_flow_sources<KS, false, true, FlowKeep::kMemory>) : launch(k_flow_sources<KS, false, false, FlowKeep::kMemory>);
  }
}

template <int KS>
void launch_strip_sources(const FlowView& fv, int workgroups, hipStream_t st) {
  k_strip_sources<KS><<<workgroups, kWideThreads, kStripState + kStripTail, st>>>(fv);
}

template <int KS>
void launch_flow_links(const FlowView& fv, bool demand, hipStream_t st) {
  const auto launch = [&](auto kernel, int nodes) {  // of a thread
    const int blocks = (fv.N + nodes * kWideThreads - 1) / (nodes * kWideThreads);
    const unsigned workgroups = (unsigned)((fv.groups + 7) / 8 * 8 * blocks);
    kernel<<<workgroups, kWideThreads, fv.exact != nullptr ? strip_link_lds(fv.N) : flow_link_lds(fv.N), st>>>(fv);
  };
  constexpr int kNodes = flow_nodes(KS);
  if (fv.exact != nullptr)
    strip_links_narrow(fv.N, KS, fv.groups) ? launch(k_flow_links<KS, false, false, true, 1>, 2) : launch(k_flow_links<KS, false, false, true>, kNodes);
  else if (fv.N <= kScaledNodes)
    demand ? launch(k_flow_links<KS, true, true>, kNodes) : launch(k_flow_links<KS, true, false>, kNodes);
  else
    demand ? launch(k_flow_links<KS, false, true>, kNodes) : launch(k_flow_links<KS, false, false>, kNodes);
}

template void launch_small_loads<A2A_WORDS>(const SmallPlan&, bool, int, hipStream_t);
template void launch_node_loads<A2A_WORDS>(const SmallPlan&, bool, int, hipStream_t);
template void launch_small_outputs<A2A_WORDS>(const SmallPlan&, const SmallOut&, int, hipStream_t);
template void launch_small_levels<A2A_WORDS>(const SmallPlan&, int, hipStream_t);
template void launch_small_sssp<A2A_WORDS>(const SmallPlan&, const SmallSssp&, hipStream_t);
template void launch_flow_sssp<A2A_WORDS>(const SmallPlan&, const SmallSssp&, int, hipStream_t);
template void launch_small_sssp_add<A2A_WORDS>(const SmallPlan&, const SmallSssp&, hipStream_t);
template void launch_wide_search<A2A_WORDS>(const WideView&, int, int, int, hipStream_t);
template void launch_wide_masks<A2A_WORDS>(const WideView&, int, int, hipStream_t);
template void launch_wide_sigma<A2A_WORDS>(const WideSigma&, int, hipStream_t);
template void launch_flow_sources<A2A_WORDS>(const FlowView&, bool, int, hipStream_t);
template void launch_strip_sources<A2A_WORDS>(const FlowView&, int, hipStream_t);
template void launch_flow_links<A2A_WORDS>(const FlowView&, bool, hipStream_t);

}  // namespace a2a_dev
