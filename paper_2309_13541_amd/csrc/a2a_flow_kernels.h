// Link loads of topologies whose path counts or coefs of one source fit LDS (8 bytes a node: up to 20352 nodes; 16 with demands: 10176)
// but whose link loads do not fit the registers of a workgroup (from 2049 nodes of 16 links, 8192 of 4 links on).
//
// The level kernels gather 64 sources at a time out of rows in memory.  Here a workgroup takes a source from its sorted levels
// to its path counts and coefs with all gathers in LDS (k_flow_sources), and leaves a row of each in memory.  A second kernel
// then goes over the sources with the loads of a block of links in registers and a source's path counts in LDS (k_flow_links),
// and a third adds up its rows.  Whole calls over all sources, level kernels and these: 16384 nodes of a generalized Kautz
// topology of degree 4 3.70 -> 2.23 ms, of a random one 6.51 -> 2.63 ms; random topologies of 20011 nodes of degree 5 (2501 sources)
// 1.46 -> 0.59 ms, 8191 of degree 8 with demands 1.90 -> 1.15 ms, 6000 of degree 8 0.95 -> 0.49 ms, 16384 of degree 16 10.2 -> 4.1 ms.
// Up to 65536 nodes: k_strip_sources.
#pragma once

#include "a2a_wide_kernels.h"

namespace a2a_dev {

struct FlowView {
  const uint32_t *in, *out;    // link tables, as in SmallView
  const unsigned char* level;  // [sources][small_level_bytes(N)]
  void* record;                // [workgroups of k_flow_sources] nodes of a source, level by level, 16 bits each (FlowKeep::kMemory)
  uint32_t* count;             // [sources][stride] FlowWord
  double* coef;                // [sources][stride]; demands before (k_flow_demand)
  double* weighted;            // [sources] demand x distance
  long long* counters;         // [workgroups of k_flow_sources][kSmallCounters]
  double* part;                // [groups][N * 2 KS] link loads, in the places of `in`
  int N, stride, depth;
  int source0, sources;        // node of row 0, rows
  int group, groups;           // rows per group of k_flow_links, groups of this launch
  int resume;                  // the groups' loads so far are in `part`
  // By strips of nodes (k_strip_sources): `count` has 16 bits a node.
  uint32_t* exact;             // [sources][stride] path counts that those do not hold
  int* escaped;                // [sources] whether there are any
};

typedef uint32_t FlowWords __attribute__((ext_vector_type(4)));
typedef double FlowDoubles __attribute__((ext_vector_type(2)));

// A node's word: its path count below its level counted down from 254; 0 if it is not reached (yet).  An in-link of a node of level
// l comes from level l - 1 or later, so the words that count are the largest that can occur: a saturating subtraction of what
// lies above the path count leaves the count of these and 0 of all others.
constexpr int kFlowLevel = 24;
__device__ __forceinline__ uint32_t flow_above(int level) { return (uint32_t)(kSmallUnseen - 1 - level) << kFlowLevel; }
__device__ __forceinline__ uint32_t flow_count(uint32_t word, uint32_t above) { return __builtin_elementwise_sub_sat(word, above); }

// The links of a node as places in an array of 1 << kSize bytes a node: one instruction a link from 8 x id (kScaled), one from ids.
template <int KS, bool kScaled>
struct FlowRow {
  uint32_t w[KS];
  __device__ __forceinline__ void load(const uint32_t* __restrict__ table, uint32_t entry) {  // id or 8 x id
    const uint32_t at = kScaled ? __umul24(entry, KS) >> 1 : __umul24(entry, 4 * KS);
    const uint32_t* const p = reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(table) + at);
#pragma unroll
    for (int k = 0; k < KS; ++k) w[k] = p[k];
  }
  template <int kSize>
  __device__ __forceinline__ uint32_t at(int j) const {
    if constexpr (kScaled) {
      return __builtin_amdgcn_ubfe(w[j >> 1], (j & 1) * 16 + 3 - kSize, 13 + kSize);
    } else {
      uint32_t x;  // a half of the word, shifted: the compiler takes two instructions
      if (j & 1)
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(x) : "v"(kSize), "v"(w[j >> 1]));
      else
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(x) : "v"(kSize), "v"(w[j >> 1]));
      return x;
    }
  }
  // 8 x id of link j + less.
  __device__ __forceinline__ uint32_t strip_at(int j, uint32_t less) const {
    static_assert(!kScaled);
    uint32_t x;
    if (j & 1)
      asm("v_mad_u32_u16 %0, %1, 8, %2 op_sel:[1,0,0,0]" : "=v"(x) : "v"(w[j >> 1]), "s"(less));
    else
      asm("v_mad_u32_u16 %0, %1, 8, %2" : "=v"(x) : "v"(w[j >> 1]), "s"(less));
    return x;
  }
  // Of the node of a table entry.
  template <int kSize>
  static __device__ __forceinline__ uint32_t own(uint32_t entry) {
    return kScaled ? entry >> (3 - kSize) : entry << kSize;
  }
};

// `chunks` times 16 bytes from memory to LDS, a kilobyte a wave and instruction.  They have arrived when vmcnt has come down to the
// requests after them.  (As assembly, because the compiler would wait for all of them before any access to LDS.)
// The compiler puts no wait states inside: a load to LDS needs one after the write of M0, and five after a vector instruction that wrote
// its address registers (a lane read back), whatever stands before this.
__device__ __forceinline__ void flow_to_lds(const void* from, void* to, int chunks, int wave, int lane) {
  const uint32_t place = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)to;
  for (int c = wave * kWave; c < chunks; c += kWideThreads)
    if (c + lane < chunks)
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1"
                   :
                   : "v"(16u * (uint32_t)lane), "s"(static_cast<const char*>(from) + 16 * (size_t)c), "s"(place + 16u * (uint32_t)c)
                   : "memory", "m0");
}

// No memory request is moved from one side of this to the other.
__device__ __forceinline__ void flow_in_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Waits for a node's links.
template <int KS, bool kScaled>
__device__ __forceinline__ void flow_arrived(const FlowRow<KS, kScaled>& row) {
#pragma unroll
  for (int k = 0; k < KS; ++k) asm volatile("" ::"v"(row.w[k]));
}

// Sorts nodes by level, in node order within a level: thread t has the nodes 4 words t, ..., their levels as bytes in lv.
// place(position, node in thread's) is called for every node; those that are not on a level of 1 ... kLevels get positions from
// `spare` on, kFlowSpare at the most.  totals: [kWideThreads / kWave][8] words of LDS; base: room for kLevels + 1
// positions per thread.  Has one barrier inside.  Returns where levels start: lane l has level l (lanes past the last level
// the end).  No atomics: a thread's counts per level are the bytes of 64-bit words, eight levels each, and the sums over threads
// 16-bit fields.  Bound by the vector ALUs (some 20 instructions a node).
constexpr int kFlowSpare = 32;
template <int kLevels, int kMost, typename Place>
__device__ __forceinline__ int flow_sort(uint32_t (&lv)[kMost], int words, uint32_t* totals, unsigned short* base,
                                         int spare, int wave, int lane, Place&& place) {
  constexpr int kHalves = (kLevels + 7) / 8, kFields = 4 * kHalves;
  const auto level = [&](int k, int i) { return min((lv[k] >> (8 * i) & 255u) - 1u, (uint32_t)kLevels); };  // less one
  uint64_t count[kHalves];
  uint32_t rank[kMost];  // of a node among the thread's on its level, a byte each
#pragma unroll
  for (int h = 0; h < kHalves; ++h) count[h] = 0;
  // (steps and not loops: of loops that are unrolled late the compiler keeps the arrays as one tuple of registers, which it moves)
  wide_steps([&](auto word) {
    constexpr int k = decltype(word)::value;
    rank[k] = 0;
    if (k >= words) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t d = level(k, i), shift = d * 8u & 63u;
      const uint64_t one = 1ull << shift;
      rank[k] |= ((uint32_t)((kHalves == 1 || d < 8u ? count[0] : count[kHalves - 1]) >> shift) & 255u) << (8 * i);
#pragma unroll
      for (int h = 0; h < kHalves; ++h) count[h] += d - 8u * h < 8u ? one : 0ull;
    }
  }, std::make_index_sequence<kMost>{});
  // half f of word w of parity p of half h: level 8 h + p + 4 w + 2 f + 1
  uint32_t own[kFields], incl[kFields];
#pragma unroll
  for (int h = 0; h < kHalves; ++h) {
    const uint32_t lo = (uint32_t)count[h], hi = (uint32_t)(count[h] >> 32);
    own[4 * h] = lo & 0x00ff00ffu;
    own[4 * h + 1] = hi & 0x00ff00ffu;
    own[4 * h + 2] = lo >> 8 & 0x00ff00ffu;
    own[4 * h + 3] = hi >> 8 & 0x00ff00ffu;
  }
#pragma unroll
  for (int g = 0; g < kFields; ++g) incl[g] = (uint32_t)wave_scan_incl((int)own[g]);
  if (lane == kWave - 1) {
#pragma unroll
    for (int g = 0; g < kFields; ++g) totals[wave * 8 + g] = incl[g];
  }
  __syncthreads();
  uint32_t all[kFields], pos[kFields];
#pragma unroll
  for (int g = 0; g < kFields; ++g) {
    const uint32_t x = totals[(lane & 15) * 8 + g], upto = (uint32_t)wave_scan_row((int)x);
    all[g] = (uint32_t)__builtin_amdgcn_readlane((int)upto, 15);
    pos[g] = (uint32_t)__builtin_amdgcn_readlane((int)(upto - x), wave) + incl[g] - own[g];
  }
  unsigned short* const mine = base + wave * kWave + lane;
  int at = 0;
  uint32_t sum = 0;
#pragma unroll
  for (int d = 0; d < kLevels; ++d) {
    const int g = (d >> 3) * 4 + (d & 1) * 2 + (d >> 2 & 1), shift = (d >> 1 & 1) * 16;
    mine[d * kWideThreads] = (unsigned short)((pos[g] >> shift) + sum);
    if (lane == d + 1) at = (int)sum;
    sum += all[g] >> shift & 0xffffu;
  }
  if (lane > kLevels) at = (int)sum;
  mine[kLevels * kWideThreads] = (unsigned short)spare;
  wide_steps([&](auto word) {
    constexpr int k = decltype(word)::value;
    if (k >= words) return;
    asm volatile("" : "+v"(lv[k]), "+v"(rank[k]));  // nothing worked out before the barrier is kept
    uint32_t at_level[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) at_level[i] = mine[level(k, i) * kWideThreads];
#pragma unroll
    for (int i = 0; i < 4; ++i) place(at_level[i] + (rank[k] >> (8 * i) & 255u), 4 * k + i);
    __builtin_amdgcn_sched_barrier(0);
  }, std::make_index_sequence<kMost>{});
  return at;
}

// The levels of a source, one after the other (kStep 1: upwards, -1: downwards), in pieces of as many nodes as the workgroup
// has threads; all of it in scalar registers.  Levels past the last and level 0 have no nodes.
template <int kStep>
struct FlowPiece {
  int level, base, end;  // its place in the queue, where the level ends
  __device__ __forceinline__ void enter(int l, int starts) {
    level = l;
    base = __builtin_amdgcn_readlane(starts, l & (kWave - 1));
    end = __builtin_amdgcn_readlane(starts, (l + 1) & (kWave - 1));
  }
  __device__ __forceinline__ void next(int starts) {
    base += kWideThreads;
    if (base >= end) enter(level + kStep, starts);
  }
};

// Path counts and coefs of sources blockIdx.x, + gridDim.x, ...  Per source: sort; sigma = the sum over the in-links from the level
// before, level by level; coef = demand / sigma + the coefs of the successors, deepest level first.  LDS has a word per node in the
// forward sweep, its level above its path count (a whole number below 2^24), so that a gathered word tells whether it counts.  In
// the backward sweep a double per node, 0 until it is written: a node of level l has out-links to levels up to l + 1, of which only
// l + 1 and (some of) l are written, so even levels are kept with a plus sign and odd ones with a minus sign, and a level adds up
// the entries of the other sign only.  Coefs of unequal demands have any sign: even and odd levels have an array each.
// The nodes' order and their path counts go from one sweep to the other in LDS as far as there is room (flow_keep has the rule and its times);
// both are read three pieces ahead, links one piece ahead.  With demands, order and demand / path count go through memory.  Without,
// the forward sweep stores nothing in memory: its pieces waited for what the one before had stored, 6 bytes a node.  Where path counts do not fit in
// the queue's order, a node's stays in the low word of the double that the backward sweep has of it: below 2^-1022, it changes no sum of
// coefs, all of which are above 2^-25; but it is then read in the chain of a backward piece.  All sources, link loads alone in a replayed graph, records
// through memory and now: 9000 nodes of degree 4 893, 867 us, of degree 8 979, 971; 10000 of a generalized Kautz topology of degree 9 1085, 1033; order
// in LDS: 13000 of a generalized Kautz topology of degree 7 1523, 1449, of degree 6 1765, 1702; order in memory: 16384 of a generalized Kautz topology of
// degree 4 2235, 2112; 20000 of degree 4 3893, 3698, of degree 16 6524, 6518.  At the lower end of what has ids and not 8 x id in its tables the old way
// was the faster one by 0.4 % (8300 of degree 8 855, 859).  With 16 links and path counts by node two registers spill.  (Path counts read again by node from the
// output rows: 16384 nodes 1646 us here, then 1791; with demands, quotients stored after the sweep: 8191 of degree 8 774, 801.)  Rows
// of the outputs are written from LDS, in node order.
// Bound by the instructions of a piece and its barriers, which the four waves of a SIMD hide in part: 16384 nodes of degree 4 took 1640 us
// with record stores, forward 490, backward 540, sort 240, rows and zeroes 280; with gathers from the thread's own place in LDS, or
// without any, 1600 and more, without any access to memory 1410.  Two nodes a thread and piece, their gathers at the same time: 2 to 6 % slower.
// Pushing counts to the out-links by LDS additions where that touches fewer nodes took longer (48 for 26 thousand cycles
// forward, 20011 nodes of degree 5), and so did links asked for three pieces ahead (20 for 14 thousand).
// kScaled: the tables have 8 x id.
template <int KS, bool kScaled, bool kDemand, FlowKeep kKeep>
__global__ void __launch_bounds__(kWideThreads) k_flow_sources(FlowView fv) {
  extern __shared__ double s_small[];
  using Row = FlowRow<KS, kScaled>;
  const int t = (int)threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int N = fv.N, S = fv.stride, nl = (int)small_level_bytes(N);
  const int words = (N + 4 * kWideThreads - 1) / (4 * kWideThreads), v0 = 4 * words * t;  // this thread's nodes in the sort
  uint32_t* const x = reinterpret_cast<uint32_t*>(s_small);
  constexpr bool kRecords = kKeep == FlowKeep::kRecords, kStays = kKeep != FlowKeep::kMemory;
  constexpr bool kByNode = !kDemand && !kRecords;  // path counts wait by node
  const uint32_t q_at = (kStays ? 8u : 4u) * (uint32_t)S, paths_at = q_at + 2u * (uint32_t)(S + kFlowSpare);
  unsigned short* const q = reinterpret_cast<unsigned short*>(reinterpret_cast<char*>(s_small) + q_at);
  unsigned short* const base = kStays && flow_gap(N, fv.depth) ? reinterpret_cast<unsigned short*>(x + S) : q + S + kFlowSpare + (kRecords ? 2 * S : 0);
  double* const demand = reinterpret_cast<double*>(reinterpret_cast<char*>(s_small) + flow_demand_at(N, fv.depth));
  // behind all that, so that places in the arrays at the start need no addition
  double* const s_weighted = reinterpret_cast<double*>(reinterpret_cast<char*>(s_small) + flow_tail_at(N, fv.depth, kKeep, kDemand));
  uint32_t* const s_totals = reinterpret_cast<uint32_t*>(s_weighted + kWideThreads / kWave);
  unsigned short* const queue = reinterpret_cast<unsigned short*>(static_cast<char*>(fv.record) + (size_t)blockIdx.x * flow_record_bytes(S, kDemand));
  double* const value = reinterpret_cast<double*>(queue + S);  // demand / path count, with demands
  constexpr int kId = kScaled ? 3 : 0;  // table entries are ids << kId
  constexpr uint32_t kCount = (1u << kFlowLevel) - 1u;
  long long dsum = 0, reached = 0;
  uint32_t lv[kFlowWords];
  const auto levels = [&](int s) {  // of a source
    const unsigned char* const level = fv.level + (size_t)s * (size_t)nl;
#pragma unroll
    for (int k = 0; k < kFlowWords; ++k) {
      lv[k] = ~0u;
      if (k < words && v0 + 4 * k < N) lv[k] = *reinterpret_cast<const uint32_t*>(level + v0 + 4 * k);
    }
  };
  if ((int)blockIdx.x < fv.sources) levels((int)blockIdx.x);
  for (int s = (int)blockIdx.x; s < fv.sources; s += (int)gridDim.x) {
    double* const coef = fv.coef + (size_t)s * (size_t)S;
#pragma unroll
    for (int k = 0; k < kFlowWords; ++k) {  // places past the last node: out of reach
      const int v = v0 + 4 * k;
      if (v < N && v + 4 > N) lv[k] |= ~0u << ((N - v) * 8);
    }
    __syncthreads();
    if (kDemand) flow_to_lds(coef, demand, S / 2, wave, lane);  // arrives while the nodes are sorted
    for (int i = t; i < S / 4; i += kWideThreads) reinterpret_cast<uint4*>(x)[i] = make_uint4(0, 0, 0, 0);
    int v1 = v0;
    asm volatile("" : "+v"(v1));  // not kept from source to source
    const auto place = [&](uint32_t p, int i) { q[p] = (unsigned short)((v1 + i) << kId); };
    const int starts = fv.depth <= 8 ? flow_sort<8>(lv, words, s_totals, base, S, wave, lane, place)
                                     : flow_sort<16>(lv, words, s_totals, base, S, wave, lane, place);
    if (t == 0) x[fv.source0 + s] = flow_above(0) + 1u;
    const int after = __shfl_down(starts, 1, kWave);
    const uint64_t filled = __ballot(lane >= 1 && lane <= fv.depth && after > starts);
    const int deep = filled != 0 ? 63 - __builtin_clzll(filled) : 0;
    const uint32_t last = (uint32_t)max(__builtin_amdgcn_readlane(starts, kWave - 1) - 1, 0);
    if (wave == 0) {
      reached += lane >= 1 && lane <= deep ? after - starts : 0;
      dsum += lane >= 1 && lane <= deep ? (long long)lane * (after - starts) : 0;
    }
    if (kDemand) __builtin_amdgcn_s_waitcnt(0);  // this wave's demands have arrived
    __syncthreads();

    double wd = 0.0;
    if (deep > 0) {  // forward
      FlowPiece<1> a, b, c;
      a.enter(1, starts);
      b = a;
      b.next(starts);
      c = b;
      c.next(starts);
      const uint32_t q0 = q_at + 2u * (uint32_t)t, q1 = q_at + 2u * last;
      const auto node = [&](const FlowPiece<1>& p) {
        return (uint32_t)lds_get<unsigned short>(min(q0 + 2u * (uint32_t)p.base, q1));
      };
      struct Ahead {
        uint32_t node;
        Row row;
      };
      // A piece, after the links of the next one have been asked for; the node after that one takes the piece's place.
      // Registers are not moved from piece to piece: a move would wait for what is on its way.
      const auto step = [&](Ahead& here, Ahead& next) {
        flow_arrived(here.row);
        next.row.load(fv.in, next.node);
        uint32_t then = node(c);
        if (t < a.end - a.base) {
          uint32_t y[2 * KS];
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j) y[j] = lds_get<uint32_t>(here.row.template at<2>(j));
          const double own = kDemand ? lds_at(demand, Row::template own<3>(here.node)) : 1.0;
          __builtin_amdgcn_sched_barrier(0);
          const uint32_t before = flow_above(a.level - 1);
          uint32_t above = flow_above(a.level), sum = 0;
          asm volatile("" : "+s"(above));
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j) sum += flow_count(y[j], before);
          lds_put<uint32_t>(Row::template own<2>(here.node), sum + above);
          if constexpr (kRecords) lds_put<uint32_t>(paths_at + 4u * (uint32_t)(a.base + t), sum);
          if constexpr (kDemand) {
            const uint32_t at = (uint32_t)(a.base + t);
            value[at] = own * recip((double)sum);
            queue[at] = (unsigned short)here.node;
            wd = __builtin_fma((double)a.level, own, wd);
          }
        }
        if (b.level != a.level) lds_barrier();
        asm volatile("" : "+v"(then));  // widened as it is read, not again where it is used
        here.node = then;
        a = b;
        b = c;
        c.next(starts);
      };
      Ahead n0, n1;
      n0.node = node(a);
      n1.node = node(b);
      n0.row.load(fv.in, n0.node);
      for (;;) {
        step(n0, n1);
        if (a.level > deep) break;
        step(n1, n0);
        if (a.level > deep) break;
      }
    }
    if (kDemand) {
      wd = wave_sum_double(wd);
      if (lane == 0) s_weighted[wave] = wd;
    }
    // Path counts leave.  By node, a node's waits for it in the low word of its place in the backward sweep: as a double less than 2^-1022
    // and so nothing beside a coef.
    uint32_t* const count = fv.count + (size_t)s * (size_t)S;
    for (int i = t; i < S / 8 && kByNode && !kStays; i += kWideThreads) reinterpret_cast<FlowWords*>(queue)[i] = reinterpret_cast<const FlowWords*>(q)[i];
    FlowWords words_of[kFlowWords];
#pragma unroll
    for (int k = 0; k < kFlowWords; ++k) {
      const int i = t + k * kWideThreads;
      if (i < S / 4) {
        words_of[k] = reinterpret_cast<const FlowWords*>(x)[i];
        __builtin_nontemporal_store(words_of[k], reinterpret_cast<FlowWords*>(count) + i);
      }
    }
    __syncthreads();
    if (kDemand && t == 0) {
      wd = 0.0;
      for (int k = 0; k < kWideThreads / kWave; ++k) wd += s_weighted[k];
      fv.weighted[s] = wd;
    }
    if (!kByNode) {
      for (int i = t; i < (kDemand ? S : S / 2); i += kWideThreads) reinterpret_cast<double2*>(s_small)[i] = make_double2(0.0, 0.0);
    } else {
#pragma unroll
      for (int k = 0; k < kFlowWords; ++k) {
        const int i = t + k * kWideThreads;
        if (i < S / 4) {
          reinterpret_cast<FlowWords*>(s_small)[2 * i] = FlowWords{words_of[k].x & kCount, 0, words_of[k].y & kCount, 0};
          reinterpret_cast<FlowWords*>(s_small)[2 * i + 1] = FlowWords{words_of[k].z & kCount, 0, words_of[k].w & kCount, 0};
        }
      }
    }
    lds_barrier();
    if (kByNode && t == 0) s_small[fv.source0 + s] = 0.0;

    if (s + (int)gridDim.x < fv.sources) levels(s + (int)gridDim.x);
    if (deep > 0) {  // backward
      FlowPiece<-1> a, b, c, d;
      a.enter(deep, starts);
      b = a;
      b.next(starts);
      c = b;
      c.next(starts);
      d = c;
      d.next(starts);
      struct Entry {
        uint32_t node, paths;
        double value;
      };
      const auto read = [&](const FlowPiece<-1>& p) {
        const uint32_t at = min((uint32_t)t + (uint32_t)p.base, last);
        Entry e;
        e.value = kDemand ? lds_at(value, 8u * at) : 0.0;
        e.paths = kRecords ? lds_get<uint32_t>(paths_at + 4u * at) : 0u;
        e.node = kStays ? lds_get<unsigned short>(q_at + 2u * at) : queue[at];
        return e;
      };
      const auto step = [&](const Entry& here, const Entry& next, Entry& third, Row& row, Row& next_row) {
        flow_arrived(row);
        next_row.load(fv.out, next.node);
        flow_in_order();
        third = read(d);
        flow_in_order();
        if (t < a.end - a.base) {
          const bool odd = (a.level & 1) != 0, inner = a.level < deep;  // the last level has no successors
          const uint32_t from = kDemand && !odd ? 8u * (uint32_t)S : 0u, to = kDemand && odd ? 8u * (uint32_t)S : 0u;
          const uint32_t paths = !kByNode ? here.paths : lds_get<uint32_t>(Row::template own<3>(here.node));
          double y[2 * KS];
          if (inner) {
#pragma unroll
            for (int j = 0; j < 2 * KS; ++j) y[j] = lds_get<double>(row.template at<3>(j) + from);
          }
          __builtin_amdgcn_sched_barrier(0);
          double sum = kDemand ? here.value : recip((double)paths);
          if (kDemand) {
            if (inner) {
              double succ = y[0];
#pragma unroll
              for (int j = 1; j < 2 * KS; ++j) succ += y[j];
              sum += succ;
            }
          } else if (odd) {
            sum = -sum;
            if (inner) {
              double succ = plus_part(y[0]);
#pragma unroll
              for (int j = 1; j < 2 * KS; ++j) succ += plus_part(y[j]);
              sum -= succ;
            }
          } else if (inner) {
            double succ = minus_part(y[0]);
#pragma unroll
            for (int j = 1; j < 2 * KS; ++j) succ += minus_part(y[j]);
            sum -= succ;
          }
          lds_put<double>(Row::template own<3>(here.node) + to, sum);
        }
        if (b.level != a.level) lds_barrier();
        a = b;
        b = c;
        c = d;
        d.next(starts);
      };
      Entry e0 = read(a), e1 = read(b), e2, e3;
      Row w0, w1;
      w0.load(fv.out, e0.node);
      flow_in_order();  // as in the steps: links, then a node
      e2 = read(c);
      flow_in_order();
      for (;;) {
        step(e0, e1, e3, w0, w1);
        if (a.level < 1) break;
        step(e1, e2, e0, w1, w0);
        if (a.level < 1) break;
        step(e2, e3, e1, w0, w1);
        if (a.level < 1) break;
        step(e3, e0, e2, w1, w0);
        if (a.level < 1) break;
      }
    } else {
      lds_barrier();
    }
#pragma unroll
    for (int k = 0; k < kFlowWords; ++k) asm volatile("" : "+v"(lv[k]));  // arrived before anything is stored: a wait for them later on would be one for the stores too
    for (int i = t; i < S / 2; i += kWideThreads) {
      const FlowDoubles y = reinterpret_cast<const FlowDoubles*>(s_small)[i];
      FlowDoubles out;
      if (kDemand) {
        out = y + reinterpret_cast<const FlowDoubles*>(s_small + S)[i];  // one of the two is 0
      } else {
        out.x = __builtin_fabs(y.x);
        out.y = __builtin_fabs(y.y);
      }
      __builtin_nontemporal_store(out, reinterpret_cast<FlowDoubles*>(coef) + i);
    }
  }
  __syncthreads();
  SmallView sv{};
  sv.counters = fv.counters;
  small_totals(sv, s_small, dsum, reached, false, 0.0, false);
}

// What k_flow_sources does, for topologies whose coefs of one source do not fit LDS (up to 65536 nodes).  16-bit words of all nodes do:
// the levels that occur counted down, above the path count.  A count that does not fit leaves all ones there, and itself
// in memory (fv.exact), where the few that meet it read it.  So the forward sweep is that of k_flow_sources, with the queue in memory.
// Backward, a level's coefs come into LDS a strip of nodes at a time, and the nodes of the level before go over their
// links once per strip: a link that leads elsewhere reads the 0 behind the strip (all lanes the same word, which costs little).
// Their sums stay in registers in between, kPieces nodes a thread.  A level of few nodes needs no strips: a bit per node says
// which are on it, and the coefs are a list.  The last level, and a level before one of few nodes, is worked out strip by strip
// as it goes into LDS; others come from memory, where they wait in the row of the output.
// A source of 65536 nodes of degree 8 takes 540 thousand cycles: sort 53, forward 102, levels of few nodes 25, level 6 into LDS 62, levels 5
// and 4 into LDS 30, the sums over strips 109, waiting for each other and for records around a strip 76, what a level is by itself 58.
// Vector ALUs are busy 42, LDS 38 % of the time, and 1.6 MB are read and as much is written a source (3.9 TB/s): bound by chains within
// a piece (links, gathers, sum) and by what a strip begins and ends with.  Memory requests come back in order, so queue
// entries, which miss L2, are asked for many at a time (a call 80, now 77 ms), and the first strip's coefs do not go through
// memory (77, now 75).  Link tables that have a node's links by strips took less LDS time, but 4 MB more in L2: 97 ms, 80 without.
template <int KS>
__global__ void __launch_bounds__(kWideThreads) k_strip_sources(FlowView fv) {
  extern __shared__ double s_small[];
  using Row = FlowRow<KS, false>;
  constexpr int T = kWideThreads, kPieces = KS <= 4 ? 24 : KS == 5 ? 16 : 8;
  const int t = (int)threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int N = fv.N, S = fv.stride, nl = (int)small_level_bytes(N);
  const int words = (N + 4 * T - 1) / (4 * T);
  const int count_bits = strip_count_bits(fv.depth);
  const uint32_t count_most = (1u << count_bits) - 1u;
  const StripCut strips = strip_cut(N);
  unsigned short* const x = reinterpret_cast<unsigned short*>(s_small);  // the queue, then the nodes' words
  unsigned short* const base = x + S;
  uint32_t* const s_totals = reinterpret_cast<uint32_t*>(s_small + kStripState / 8);
  int* const s_strip = reinterpret_cast<int*>(s_totals + T / kWave * 8);  // [strip][level less one]: place in the queue
  int* const s_escaped = s_strip + kStripMost * 16;
  unsigned short* const queue = reinterpret_cast<unsigned short*>(static_cast<char*>(fv.record) + (size_t)blockIdx.x * strip_record_bytes(S));
  uint32_t* const record = reinterpret_cast<uint32_t*>(queue + S);  // node, path count above it (all ones: in fv.exact)
  const auto above = [&](int level) { return (uint32_t)(fv.depth - level) << count_bits; };
  const auto clear = [&](uint32_t bytes) {
    for (uint32_t i = (uint32_t)t; i < bytes / 16; i += T) reinterpret_cast<uint4*>(s_small)[i] = make_uint4(0, 0, 0, 0);
  };
  uint32_t reached = 0;  // by lane l of the first wave on level l (at most 256 sources)
  for (int s = (int)blockIdx.x; s < fv.sources; s += (int)gridDim.x) {
    double* const coef = fv.coef + (size_t)s * (size_t)S;
    uint32_t* const exact = fv.exact + (size_t)s * (size_t)S;
    const int source = fv.source0 + s;
    int tt = t;
    asm volatile("" : "+v"(tt));  // addresses are not kept from source to source
    const int v0 = 4 * words * tt;  // this thread's nodes in the sort
    uint32_t lv[kStripWords];
    const unsigned char* const level = fv.level + (size_t)s * (size_t)nl;
#pragma unroll
    for (int k = 0; k < kStripWords; k += 4) {
      const int v = v0 + 4 * k;
      Int4 four = {-1, -1, -1, -1};
      if (k < words && v + 16 <= nl) {
        four = *reinterpret_cast<const Int4*>(level + v);
      } else if (k < words) {
        if (v < nl) four.x = *reinterpret_cast<const int*>(level + v);
        if (v + 4 < nl) four.y = *reinterpret_cast<const int*>(level + v + 4);
        if (v + 8 < nl) four.z = *reinterpret_cast<const int*>(level + v + 8);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        lv[k + i] = (uint32_t)four[i];
        const int u = v + 4 * i;
        if (u < N && u + 4 > N) lv[k + i] |= ~0u << ((N - u) * 8);  // places past the last node: out of reach
      }
    }
    __syncthreads();
    int v1 = v0;
    asm volatile("" : "+v"(v1));
    // (those on no level have the last place: there is the source too, so that no other node has it)
    const auto place = [&](uint32_t p, int i) { x[min(p, (uint32_t)N - 1u)] = (unsigned short)(v1 + i); };
    const int levels = strip_levels(fv.depth);
    const int starts = levels == 8    ? flow_sort<8>(lv, words, s_totals, base, N - 1, wave, lane, place)
                       : levels == 12 ? flow_sort<12>(lv, words, s_totals, base, N - 1, wave, lane, place)
                                      : flow_sort<16>(lv, words, s_totals, base, N - 1, wave, lane, place);
    if (t % strips.threads == 0 && t / strips.threads < strips.count)
      for (int l = 0; l < levels; ++l) s_strip[t / strips.threads * 16 + l] = base[l * T + t];
    if (t == 0) *s_escaped = 0;
    const auto start = [&](int l) { return __builtin_amdgcn_readlane(starts, l & (kWave - 1)); };  // of a level
    const int after = __shfl_down(starts, 1, kWave);
    const uint64_t filled = __ballot(lane >= 1 && lane <= fv.depth && after > starts);
    const int deep = filled != 0 ? 63 - __builtin_clzll(filled) : 0;
    const int total = __builtin_amdgcn_readlane(starts, kWave - 1);
    const uint32_t last = (uint32_t)max(total - 1, 0);
    if (wave == 0) reached += lane >= 1 && lane <= deep ? (uint32_t)(after - starts) : 0u;
    lds_barrier();
    for (int i = t; i < S / 8; i += T) reinterpret_cast<uint4*>(queue)[i] = reinterpret_cast<const uint4*>(x)[i];
    lds_barrier();
    clear(2u * (uint32_t)S);
    lds_barrier();
    if (t == 0) {
      x[source] = (unsigned short)(above(0) + 1u);
      coef[source] = 0.0;
    }
    __syncthreads();

    bool escaped = false;
    if (deep > 0) {  // forward: nodes are asked for a dozen pieces at a time, links two pieces ahead
      constexpr int kDozen = 12;
      FlowPiece<1> a, b, e;
      a.enter(1, starts);
      b = a;
      b.next(starts);
      e = a;
      uint32_t node[kDozen], then[kDozen];
      const auto ask = [&](uint32_t (&to)[kDozen]) {
        wide_steps([&](auto number) {
          to[decltype(number)::value] = lds_at(queue, 2u * min((uint32_t)(e.base + tt), last));
          e.next(starts);
        }, std::make_index_sequence<kDozen>{});
        flow_in_order();
      };
      Row row[3];
      const auto step = [&](auto step_number) {
        constexpr int i = decltype(step_number)::value;
        const Row& here = row[i % 3];
        const uint32_t own = node[i];
        flow_arrived(here);
        row[(i + 2) % 3].load(fv.in, i + 2 < kDozen ? node[i + 2 < kDozen ? i + 2 : 0] : then[i + 2 < kDozen ? 0 : i + 2 - kDozen]);
        flow_in_order();
        if (tt < a.end - a.base) {
          uint32_t y[2 * KS];
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j) y[j] = lds_get<unsigned short>(here.template at<1>(j));
          __builtin_amdgcn_sched_barrier(0);
          const uint32_t before = above(a.level - 1);
          uint32_t sum = 0;
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j) sum += y[j] = flow_count(y[j], before);
          if (__builtin_expect(sum >= count_most, 0)) {
            sum = 0;
#pragma unroll
            for (int j = 0; j < 2 * KS; ++j) sum += y[j] == count_most ? exact[here.template at<0>(j)] : y[j];
            if (__builtin_expect(sum >= count_most, 0)) {
              exact[own] = sum;
              escaped = true;
            }
            __builtin_amdgcn_s_waitcnt(0);  // there before the barrier
          }
          lds_put<unsigned short>(2 * own, (unsigned short)(min(sum, count_most) + above(a.level)));
          lds_at(record, 4u * (uint32_t)(a.base + tt)) = own | min(sum, 0xffffu) << 16;
        }
        if (b.level != a.level) lds_barrier();
        a = b;
        b.next(starts);
        return a.level <= deep;
      };
      ask(node);
      row[0].load(fv.in, node[0]);
      row[1].load(fv.in, node[1]);
      flow_in_order();
      for (;;) {
        ask(then);
        if (!wide_steps_while(step, std::make_index_sequence<kDozen>{})) break;
        wide_steps([&](auto number) { node[decltype(number)::value] = then[decltype(number)::value]; }, std::make_index_sequence<kDozen>{});
      }
    }
    if (escaped) *s_escaped = 1;
    // Other threads read the records and path counts in memory from here on, for which lds_barrier() does not wait.  (65536 nodes of
    // degree 8, without this and the bound on the rows that records name, and with both: 75.8, 76.4 ms.)
    __syncthreads();
    unsigned short* const count = reinterpret_cast<unsigned short*>(fv.count) + (size_t)s * (size_t)S;
    for (int i = t; i < S / 8; i += T)
      __builtin_nontemporal_store(reinterpret_cast<const FlowWords*>(x)[i], reinterpret_cast<FlowWords*>(count) + i);
    if (total < N - 1)  // nodes out of reach have no coef
      for (int v = t; v < N; v += T)
        if (x[v] == 0) coef[v] = 0.0;

    // What a node of a level is to its predecessors, without its successors.
    const auto alone = [&](uint32_t r) {
      uint32_t n = r >> 16;
      if (n == 0xffffu) n = exact[r & 0xffffu];
      return recip((double)n);
    };
    const uint32_t bits_at = (uint32_t)strips.bits, before_at = (uint32_t)strips.before;
    // The coefs of a node's successors on a level of few nodes: which links lead there (bits), then their sum.
    uint32_t few_at = 0;
    const auto few_bits = [&](const Row& row, uint32_t (&bits)[2 * KS]) {
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) bits[j] = lds_get<uint32_t>(__builtin_amdgcn_ubfe(row.w[j >> 1] & 0xffe0ffe0u, (j & 1) * 16 + 3, 13) + bits_at);
      __builtin_amdgcn_sched_barrier(0);
    };
    const auto few_sum = [&](const Row& row, const uint32_t (&bits)[2 * KS]) {
      uint32_t links = 0;
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) links |= __builtin_amdgcn_ubfe(bits[j], row.w[j >> 1] >> (j & 1) * 16, 1) << j;
      double sum = 0.0;
      while (links != 0) {
        const uint32_t j = (uint32_t)__builtin_ctz(links);
        links &= links - 1u;
        uint32_t w = row.w[0];
#pragma unroll
        for (int k = 1; k < KS; ++k) w = j >> 1 == (uint32_t)k ? row.w[k] : w;
        const uint32_t v = w >> (j & 1u) * 16u & 0xffffu;
        const uint32_t word = lds_get<uint32_t>((v >> 3 & 0x1ffcu) + bits_at), first = lds_get<unsigned short>((v >> 4 & 0xffeu) + before_at);
        sum += lds_get<double>(8u * (first + (uint32_t)__popc(word & ((1u << (v & 31u)) - 1u))) + few_at);
      }
      return sum;
    };
    // Pieces of the places first ... end of the queue: f(place, record, successors' coefs from the list).  Records are asked for a
    // dozen pieces at a time, links two pieces ahead, and the first of them before start().  Places past the end too, with the
    // record of the last.
    const auto pieces = [&](int first, int end, auto&& start, auto&& f) {
      constexpr int kDozen = 12;
      uint32_t r[kDozen];
      Row row[3];
      int t1 = tt;
      asm volatile("" : "+v"(t1));
      const auto ask = [&](int at) {
#pragma unroll
        for (int k = 0; k < kDozen; ++k) r[k] = lds_at(record, 4u * (uint32_t)max(min(at + k * T + t1, end - 1), 0));
        flow_in_order();
#pragma unroll
        for (int k = 0; k < 2; ++k) row[k].load(fv.out, min(r[k] & 0xffffu, (uint32_t)N - 1u));
        flow_in_order();
      };
      ask(first);
      start();
      for (int at = first; at < end;) {
        const bool more = wide_steps_while([&](auto number) {
          constexpr int i = decltype(number)::value;
          if constexpr (i + 2 < kDozen) row[(i + 2) % 3].load(fv.out, min(r[i + 2] & 0xffffu, (uint32_t)N - 1u));
          flow_in_order();
          uint32_t bits[2 * KS];
          few_bits(row[i % 3], bits);
          f(at + i * T + t1, r[i], few_sum(row[i % 3], bits));
          flow_in_order();
          return at + (i + 1) * T < end;
        }, std::make_index_sequence<kDozen>{});
        if (!more) break;
        at += kDozen * T;
        ask(at);
      }
    };
    // A level is one of few nodes if there is room for its list behind a strip; if the level before it is one as well, there
    // is no strip then, and the list may lie in its place.
    // Makes a level of few nodes what few_sum reads; node and coef of place start(l) + tt + k T in v[k], c[k].
    constexpr int kFewPieces = kStripFew / T;
    const auto size = [&](int l) { return start(l + 1) - start(l); };
    const auto few_on = [&](int l) { return size(l) <= (size(l - 1) <= strips.most ? kStripFew : strips.most); };
    const auto list = [&](int l, const uint32_t (&v)[kFewPieces], const double (&c)[kFewPieces]) {
      const int first = start(l), end = start(l + 1);
      few_at = size(l) <= strips.most ? (uint32_t)strips.few : 0u;
      uint32_t previous[kFewPieces];
#pragma unroll
      for (int k = 0; k < kFewPieces; ++k) previous[k] = lds_at(queue, 2u * (uint32_t)min(max(first + k * T + tt - 1, first), end - 1));
      lds_barrier();
      for (uint32_t i = (uint32_t)tt; i < (before_at - bits_at) / 16; i += T) lds_put<FlowWords>(16u * i + bits_at, FlowWords{0, 0, 0, 0});
      lds_barrier();
#pragma unroll
      for (int k = 0; k < kFewPieces; ++k) {
        const int i = first + k * T + tt;
        if (i < end) {
          lds_put<double>(8u * (uint32_t)(i - first) + few_at, c[k]);
          __hip_atomic_fetch_or(&lds_at(reinterpret_cast<uint32_t*>(s_small), (v[k] >> 3 & 0x1ffcu) + bits_at), 1u << (v[k] & 31u), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_WORKGROUP);
          if (i == first || previous[k] >> 5 != v[k] >> 5) lds_put<unsigned short>((v[k] >> 4 & 0xffeu) + before_at, (unsigned short)(i - first));
        }
      }
      lds_barrier();
    };
    // Where the coefs of the level behind the present one are: in the list (or there is no such level); still to be worked out, from
    // the list or without successors; in memory.
    enum { kListed, kOpen, kStored };
    int behind = kListed;
    bool ready = false;  // the first strip of the level behind is in LDS
    for (int l = deep; l >= 1; --l) {
      const int from = start(l), to = start(l + 1), next = start(l + 2);
      const bool few = few_on(l);
      if (behind == kListed) {
        if (!few) {
          behind = kOpen;
          continue;
        }
        uint32_t v[kFewPieces];
        double c[kFewPieces];
#pragma unroll
        for (int k = 0; k < kFewPieces; ++k) {
          v[k] = 0;
          c[k] = 0.0;
          const int i = from + k * T + tt;
          if (i < to) {
            const uint32_t r = lds_at(record, 4u * (uint32_t)i);
            v[k] = r & 0xffffu;
            Row row;
            if (l < deep) row.load(fv.out, v[k]);
            c[k] = alone(r);
            if (l < deep) {
              uint32_t bits[2 * KS];
              few_bits(row, bits);
              c[k] += few_sum(row, bits);
            }
            lds_at(coef, 8u * v[k]) = c[k];
          }
        }
        if (l > 1) list(l, v, c);
        continue;
      }
      for (int b = from; b < to; b += kPieces * T) {
        const int here = to - b;
        uint32_t node_first[4];  // the same for every strip
        Row row_first[2];
#pragma unroll
        for (int k = 0; k < 4; ++k) node_first[k] = lds_at(queue, 2u * (uint32_t)min(b + k * T + tt, to - 1));
        flow_in_order();
        row_first[0].load(fv.out, node_first[0]);
        row_first[1].load(fv.out, node_first[1]);
        flow_in_order();
        double sum[kPieces];
        wide_steps([&](auto number) { sum[decltype(number)::value] = 0.0; }, std::make_index_sequence<kPieces>{});
        for (int h = 0; h < strips.count; ++h) {
          const uint32_t v_first = (uint32_t)(h * strips.nodes);
          const int first = h == 0 ? to : __builtin_amdgcn_readfirstlane(s_strip[h * 16 + l]);
          const int end = h + 1 == strips.count ? next : __builtin_amdgcn_readfirstlane(s_strip[(h + 1) * 16 + l]);
          const auto put = [&](uint32_t v, double c) { lds_put<double>(8u * (v - v_first), c); };
          const auto room = [&] {
            lds_barrier();
            clear(8u * (uint32_t)strips.nodes + 16u);
            lds_barrier();
          };
          if (behind == kOpen && b == from) {
            if (l + 1 == deep) {
              constexpr int kAtOnce = 8;
              uint32_t r[kAtOnce];
              const auto records = [&](int i) {
#pragma unroll
                for (int k = 0; k < kAtOnce; ++k) r[k] = lds_at(record, 4u * (uint32_t)max(min(i + k * T, end - 1), 0));
                flow_in_order();
              };
              records(first + tt);
              room();
              for (int i = first + tt; i < end;) {
#pragma unroll
                for (int k = 0; k < kAtOnce; ++k)
                  if (i + k * T < end) {
                    const uint32_t v = r[k] & 0xffffu;
                    const double c = alone(r[k]);
                    lds_at(coef, 8u * v) = c;
                    put(v, c);
                  }
                i += kAtOnce * T;
                if (i < end) records(i);
              }
            } else {
              pieces(first, end, room, [&](int i, uint32_t r, double succ) {
                if (i < end) {
                  const uint32_t v = r & 0xffffu;
                  const double c = alone(r) + succ;
                  lds_at(coef, 8u * v) = c;
                  put(v, c);
                }
              });
            }
          } else if (!ready || h > 0 || b > from) {
            constexpr int kAtOnce = 12;
            uint32_t v[kAtOnce];
            const auto nodes = [&](int i) {
#pragma unroll
              for (int k = 0; k < kAtOnce; ++k) v[k] = lds_at(queue, 2u * (uint32_t)max(min(i + k * T, end - 1), 0));
            };
            nodes(first + tt);
            if (h == (ready && b == from ? 1 : 0)) __syncthreads();  // coefs are in memory
            room();
            for (int i = first + tt; i < end;) {
              double c[kAtOnce];
#pragma unroll
              for (int k = 0; k < kAtOnce; ++k) c[k] = lds_at(coef, 8u * v[k]);
#pragma unroll
              for (int k = 0; k < kAtOnce; ++k)
                if (i + k * T < end) put(v[k], c[k]);
              i += kAtOnce * T;
              if (i < end) nodes(i);
            }
          }
          // the block's nodes, asked for four pieces ahead, their links two
          uint32_t node[6];
          Row row[3];
#pragma unroll
          for (int k = 0; k < 4; ++k) node[k] = node_first[k];
          row[0] = row_first[0];
          row[1] = row_first[1];
          int t1 = tt;
          asm volatile("" : "+v"(t1));  // addresses are not kept from strip to strip
          lds_barrier();
          const uint32_t zero = 8u * (uint32_t)strips.nodes, less = 0u - 8u * v_first;
          wide_steps_while([&](auto number) {
            constexpr int k = decltype(number)::value;
            if constexpr (k + 2 < kPieces) row[(k + 2) % 3].load(fv.out, node[(k + 2) % 6]);
            flow_in_order();
            if constexpr (k + 4 < kPieces) node[(k + 4) % 6] = lds_at(queue, 2u * (uint32_t)min(b + (k + 4) * T + t1, to - 1));
            flow_in_order();
            double y[2 * KS];
#pragma unroll
            for (int j = 0; j < 2 * KS; ++j) y[j] = lds_get<double>(min(row[k % 3].strip_at(j, less), zero));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 2 * KS; ++j) sum[k] += y[j];
            asm volatile("" : "+v"(sum[k]));
            flow_in_order();
            return (k + 1) * T < here;
          }, std::make_index_sequence<kPieces>{});
        }
        uint32_t few_v[kFewPieces];
        double few_c[kFewPieces];
        ready = !few && l > 1 && to - from <= kPieces * T;
        if (ready) {
          lds_barrier();
          clear(8u * (uint32_t)strips.nodes + 16u);
          lds_barrier();
        }
        constexpr int kAtOnce = kPieces % 12 == 0 ? 12 : 8;
        static_assert(kPieces % kAtOnce == 0 && kFewPieces <= kPieces);
        wide_steps_while([&](auto number) {
          constexpr int k0 = decltype(number)::value * kAtOnce;
          uint32_t r[kAtOnce];
          wide_steps([&](auto n) { constexpr int k = decltype(n)::value; r[k] = lds_at(record, 4u * (uint32_t)min(b + (k0 + k) * T + tt, to - 1)); },
                     std::make_index_sequence<kAtOnce>{});
          flow_in_order();
          wide_steps([&](auto n) {
            constexpr int k = decltype(n)::value;
            double c = sum[k0 + k];
            if (b + (k0 + k) * T + tt < to) {
              const uint32_t v = r[k] & 0xffffu;
              c += alone(r[k]);
              lds_at(coef, 8u * v) = c;
              if (ready && v < (uint32_t)strips.nodes) lds_put<double>(8u * v, c);
            }
            if constexpr (k0 + k < kFewPieces) {
              few_v[k0 + k] = r[k] & 0xffffu;
              few_c[k0 + k] = c;
            }
          }, std::make_index_sequence<kAtOnce>{});
          flow_in_order();
          return (k0 + kAtOnce) * T < here;
        }, std::make_index_sequence<kPieces / kAtOnce>{});
        if (few && l > 1) list(l, few_v, few_c);
      }
      behind = few ? kListed : kStored;
    }
    __syncthreads();
    if (t == 0) fv.escaped[s] = *s_escaped;
  }
  __syncthreads();
  SmallView sv{};
  sv.counters = fv.counters;
  small_totals(sv, s_small, (long long)lane * reached, reached, false, 0.0, false);
}

// coef[s][v] = demand of node v from source s: tiles of 64 x 64.
static __global__ void __launch_bounds__(kBlock)
k_flow_demand(FlowView fv, const double* __restrict__ dem, long long ld) {
  __shared__ double s_tile[kWave][kWave + 1];
  const int t = (int)threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  const int tiles = (fv.N + kWave - 1) / kWave;
  const int v0 = (int)(blockIdx.x % (unsigned)tiles) * kWave, s0 = (int)(blockIdx.x / (unsigned)tiles) * kWave;
  constexpr int kRows = kWave / (kBlock / kWave);  // of a wave
  double x[kRows];
#pragma unroll
  for (int k = 0; k < kRows; ++k) {
    const int v = v0 + wave + k * (kBlock / kWave);
    x[k] = v < fv.N && s0 + lane < fv.sources ? __builtin_nontemporal_load(&dem[(size_t)v * (size_t)ld + (size_t)(s0 + lane)]) : 0.0;
  }
#pragma unroll
  for (int k = 0; k < kRows; ++k) s_tile[wave + k * (kBlock / kWave)][lane] = x[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRows; ++k) {
    const int s = s0 + wave + k * (kBlock / kWave);
    if (s < fv.sources && v0 + lane < fv.N)
      __builtin_nontemporal_store(s_tile[lane][s - s0], &fv.coef[(size_t)s * (size_t)fv.stride + (size_t)(v0 + lane)]);
  }
}

// Loads of the links into a block of nodes, of a group of sources: load of in-link j of node v += sigma(u) coef(v) of each
// source, in source order, in registers.  A thread has kPairs pairs of adjacent nodes.  A source's path counts are brought into
// LDS while the last one's are worked on.  The blocks of a group read the same path counts: they go to the same XCD, one after
// the other.  Bound by memory where nodes have few links (16384 nodes of degree 4: 3.3 GB in 0.59 ms), else by LDS and the vector ALUs.
template <int KS, bool kScaled, bool kDemand, bool kHalves = false, int kPairs = flow_nodes(KS) / 2>
__global__ void __launch_bounds__(kWideThreads) k_flow_links(FlowView fv) {
  constexpr int kXcds = 8;
  extern __shared__ double s_small[];
  const int t = (int)threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t / kWave), N = fv.N;
  const int blocks = (N + 2 * kPairs * kWideThreads - 1) / (2 * kPairs * kWideThreads);
  const int place = (int)blockIdx.x / kXcds;
  const int group = place / blocks * kXcds + (int)blockIdx.x % kXcds, v0 = place % blocks * (2 * kPairs * kWideThreads) + 2 * t;
  if (group >= fv.groups) return;
  const int s_first = group * fv.group, s_last = min(fv.sources, s_first + fv.group);
  using Word = std::conditional_t<kHalves, unsigned short, uint32_t>;
  constexpr int kSize = kHalves ? 1 : 2;
  const int count_bits = kHalves ? strip_count_bits(fv.depth) : kFlowLevel;
  const bool single = kHalves && strip_links_single(N);
  const uint32_t row_bytes = (uint32_t)fv.stride << kSize, buffer = single ? 0u : row_bytes;  // of a source; to the other one's
  const int lane = lane_id();
  const auto stage = [&](int s, uint32_t at) {
    flow_to_lds(reinterpret_cast<const char*>(fv.count) + (size_t)s * row_bytes, &lds_at(s_small, at), (int)row_bytes / 16, wave, lane);
  };
  FlowRow<KS, kScaled> link[kPairs][2];
  double acc[kPairs][2][2 * KS];
  double* const part = fv.part + (size_t)group * (size_t)N * (2 * KS);
  const auto last = [&](int k, int i) { return min(v0 + 2 * kWideThreads * k + i, N - 1); };  // past the last node: nothing comes of it
#pragma unroll
  for (int k = 0; k < kPairs; ++k)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int j = 0; j < KS; ++j) link[k][i].w[j] = fv.in[(size_t)last(k, i) * KS + j];
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) acc[k][i][j] = 0.0;
    }
  if (fv.resume) {
#pragma unroll
    for (int k = 0; k < kPairs; ++k)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) acc[k][i][j] = part[(size_t)last(k, i) * (2 * KS) + j];
  }
  // Even, and rows are a multiple of 64 nodes, so the second of the pair is there; pairs past the last node work on node 0.
  const auto pair = [&](int k) { return v0 + 2 * kWideThreads * k < N ? v0 + 2 * kWideThreads * k : 0; };
  struct Coefs {
    double2 pair[kPairs];
  };
  const auto request = [&](int s, uint32_t at, Coefs& c) {
    if (!single) stage(s, at);
#pragma unroll
    for (int k = 0; k < kPairs; ++k)
      c.pair[k] = *reinterpret_cast<const double2*>(fv.coef + (size_t)s * (size_t)fv.stride + (size_t)pair(k));
    flow_in_order();
  };
  // Where LDS has no room for two sources' words, the next one's are asked for into L2 meanwhile, a word of each line, the lines shared
  // out among the group's blocks.  Staged from memory itself they kept a workgroup waiting for half of its time (8192 sources of 65536
  // nodes of degree 8 2350 us here, now 1740; without staging 1330, without gathers still 2310; whole calls over 4096 sources 5.05, now 4.74 ms,
  // 50000 nodes of a generalized Kautz topology of degree 5 2.66, 2.51; two sources ahead the same).  Where two sources fit, the next one's are
  // staged a step ahead, and this gains nothing (16384 nodes of degree 4 617, 645 us).
  constexpr uint32_t kLine = 128;
  const uint32_t lines = row_bytes / kLine, share = (lines + (uint32_t)blocks - 1) / (uint32_t)blocks;
  const uint32_t line = (uint32_t)(place % blocks) * share + (uint32_t)t;
  uint32_t touched = 0;
  const auto touch = [&](int s) {
    if ((uint32_t)t < share && line < lines)
      touched = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(fv.count) + (size_t)s * row_bytes + kLine * line);
  };
  // A node's words are asked for before the last one's are worked on, where there are registers for both.
  constexpr int kAhead = KS == 4 || KS == 8 ? 0 : 1;
  struct Got {
    uint32_t own, y[2 * KS];
  };
  const auto step = [&](int s, uint32_t here, const Coefs& c, Coefs& next) {
    __builtin_amdgcn_s_waitcnt(0);  // what was asked for a step ago has arrived
    __syncthreads();
    const int escaped = kHalves ? fv.escaped[s] : 0;
    const uint32_t* const exact = fv.exact + (kHalves ? (size_t)s * (size_t)fv.stride : 0);
    if (single) asm volatile("" ::"v"(touched));
    if (s + 1 < s_last) request(s + 1, buffer - here, next);
    if (single && s + 1 < s_last) {
      touch(s + 1);
      flow_in_order();
    }
    const auto gather = [&](int u, Got& g) {
      const int k = u / 2, i = u % 2;
#pragma unroll
      for (int j = 0; j < KS; ++j) asm volatile("" : "+v"(link[k][i].w[j]));  // no addresses kept from source to source
      g.own = lds_get<Word>(here + ((uint32_t)(pair(k) + i) << kSize));
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) g.y[j] = lds_get<Word>(link[k][i].template at<kSize>(j) + here);
    };
    const auto add = [&](int u, const Got& g) {
      const int k = u / 2, i = u % 2;
      const uint32_t before = (g.own & ~((1u << count_bits) - 1u)) + (1u << count_bits);
      const double f = i == 0 ? c.pair[k].x : c.pair[k].y;
      uint32_t n[2 * KS];
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) n[j] = flow_count(g.y[j], before);
      if (kHalves && escaped != 0) {
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j)
          if (n[j] == (1u << count_bits) - 1u) n[j] = exact[link[k][i].template at<0>(j)];
      }
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) acc[k][i][j] = __builtin_fma(kDemand && n[j] == 0 ? 0.0 : f, (double)n[j], acc[k][i][j]);
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) asm volatile("" : "+v"(acc[k][i][j]));  // here and now: put off, the sums would hold on to what was gathered
    };
    Got g[2];
    if (kAhead) gather(0, g[0]);
#pragma unroll
    for (int u = 0; u < 2 * kPairs; ++u) {
      if (u + kAhead < 2 * kPairs) gather(u + kAhead, g[(u + kAhead) % 2]);
      __builtin_amdgcn_sched_barrier(0);
      add(u, g[u % 2]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (single) {
      __syncthreads();
      if (s + 1 < s_last) stage(s + 1, 0);
    }
  };
  if (s_first < s_last) {
    Coefs c0, c1;
    if (single) stage(s_first, 0);
    request(s_first, 0, c0);
    for (int s = s_first;;) {
      step(s, 0, c0, c1);
      if (++s == s_last) break;
      step(s, buffer, c1, c0);
      if (++s == s_last) break;
    }
  }
#pragma unroll
  for (int k = 0; k < kPairs; ++k)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int v = v0 + 2 * kWideThreads * k + i;
      if (v < N) {
        double2* const out = reinterpret_cast<double2*>(part + (size_t)v * (2 * KS));
#pragma unroll
        for (int j = 0; j < KS; ++j) out[j] = make_double2(acc[k][i][2 * j], acc[k][i][2 * j + 1]);
      }
    }
}

// load of every link = (first ? 0 : load) + the groups' rows, in order.
static __global__ void __launch_bounds__(kBlock)
k_flow_reduce(const double* __restrict__ part, int groups, int places, int N, int first, const int32_t* __restrict__ in_ptr,
              const int32_t* __restrict__ in_link, double* __restrict__ load) {
  const int p = (int)(blockIdx.x * kBlock + threadIdx.x), v = p / places, a = v < N ? in_ptr[v] + p % places : 0;
  if (v >= N || a >= in_ptr[v + 1]) return;
  const int link = in_link[a];
  const size_t row = (size_t)N * (size_t)places;
  double sum = first ? 0.0 : load[link];
  int g = 0;
  for (; g + 16 <= groups; g += 16) {  // sixteen requests in flight
    double x[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = part[(size_t)(g + k) * row + p];
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += x[k];
  }
  for (; g < groups; ++g) sum += part[(size_t)g * row + p];
  load[link] = sum;
}

// Sum over all sources of demand x distance: a thread's share in source order, then a tree.
static __global__ void __launch_bounds__(kWideThreads)
k_flow_weighted(const double* __restrict__ weighted, int sources, double* __restrict__ out) {
  __shared__ double s_sum[kWideThreads / kWave];
  const int t = (int)threadIdx.x;
  double sum = 0.0;
  for (int s = t; s < sources; s += kWideThreads) sum += weighted[s];
  sum = wave_sum_double(sum);
  if (lane_id() == 0) s_sum[t / kWave] = sum;
  __syncthreads();
  if (t != 0) return;
  for (int k = 1; k < kWideThreads / kWave; ++k) sum += s_sum[k];
  *out = sum;
}

// The single-path baseline of k_small_sssp with the sort and the cursors of k_flow_sources: sources blockIdx.x, + gridDim.x, ... of
// an iteration.  LDS has a word per node and a word per queue entry.  Forward: a node's cost, with the parity of its
// level as its highest bit (all ones before it has one), so that a gathered word tells whether it counts.  Costs are below 2^31 - 1
// (the host checks).  On odd levels, as unsigned numbers, the costs of the level before are smaller than all else, and on even
// ones, as signed numbers, too; both also after an addition that saturates.
// The node's entry in the queue takes the chosen link's place and neighbour beside the node.  Backward: the paths that end in
// or pass through a node, below the chosen link's place, which leave as whole rows.
// Per source of 16384 nodes of degree 4, thousands of cycles: sort 16, forward 17.5, backward and rows 14; in k_small_sssp sort 21,
// forward 22.5, backward 25.  Iteration by 512 sources 71 us, now 49.  Bound by the vector ALUs and LDS in turns.
constexpr int kFlowSsspNode = 14;  // bits of a node
static_assert(kBothTables <= 1 << kFlowSsspNode && kHandedShift == 2 * kFlowSsspNode, "a queue entry: node, neighbour, place");
template <int KS, bool kScaled>
__global__ void __launch_bounds__(kWideThreads) k_flow_sssp(SmallView sv, SmallSssp ss) {
  extern __shared__ double s_small[];
  using Row = FlowRow<KS, kScaled>;
  constexpr int kId = kScaled ? 3 : 0;  // table entries are ids << kId
  constexpr uint32_t kNode = (1u << kFlowSsspNode) - 1, kPaths = (1u << kHandedShift) - 1;
  const int t = (int)threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int N = sv.N, S = flow_stride(N), nl = (int)small_level_bytes(N);
  const int words = (N + 4 * kWideThreads - 1) / (4 * kWideThreads), v0 = 4 * words * t;  // this thread's nodes in the sort
  uint32_t* const x = reinterpret_cast<uint32_t*>(s_small);
  const uint32_t q_at = (uint32_t)flow_sssp_queue(N, sv.depth);
  uint32_t* const q = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(s_small) + q_at);
  uint32_t* const s_totals = q + S + kFlowSpare;
  const bool apart = flow_sssp_apart(N, sv.depth);
  unsigned short* const base = apart ? reinterpret_cast<unsigned short*>(s_totals + 128) : reinterpret_cast<unsigned short*>(s_small);
  long long dsum = 0, reached = 0;
  uint32_t lv[kFlowWords];
  const auto levels = [&](int s) {  // of a source
    const unsigned char* const level = sv.level + (size_t)s * (size_t)nl;
#pragma unroll
    for (int k = 0; k < kFlowWords; ++k) {
      lv[k] = ~0u;
      if (k < words && v0 + 4 * k < N) lv[k] = *reinterpret_cast<const uint32_t*>(level + v0 + 4 * k);
    }
  };
  levels((int)blockIdx.x);
  for (int s = (int)blockIdx.x; s < sv.src_count; s += (int)gridDim.x) {
#pragma unroll
    for (int k = 0; k < kFlowWords; ++k) {  // places past the last node: out of reach
      const int v = v0 + 4 * k;
      if (v < N && v + 4 > N) lv[k] |= ~0u << ((N - v) * 8);
    }
    int v1 = v0;
    asm volatile("" : "+v"(v1));  // not kept from source to source
    __syncthreads();
    const auto clear = [&] {
      const int source = sv.src_begin + s;
      for (int i = t; i < S / 4; i += kWideThreads) {
        const auto none_yet = [&](int k) { return 4 * i + k == source ? 0u : ~0u; };
        reinterpret_cast<uint4*>(x)[i] = make_uint4(none_yet(0), none_yet(1), none_yet(2), none_yet(3));
      }
    };
    if (apart) clear();
    const auto place = [&](uint32_t p, int i) { q[p] = (uint32_t)(v1 + i); };
    const int starts = sv.depth <= 8 ? flow_sort<8>(lv, words, s_totals, base, S, wave, lane, place)
                                     : flow_sort<16>(lv, words, s_totals, base, S, wave, lane, place);
    const int after = __shfl_down(starts, 1, kWave);
    const uint64_t filled = __ballot(lane >= 1 && lane <= sv.depth && after > starts);
    const int deep = filled != 0 ? 63 - __builtin_clzll(filled) : 0;
    const int total = __builtin_amdgcn_readlane(starts, kWave - 1);
    if (wave == 0) {
      reached += lane >= 1 && lane <= deep ? after - starts : 0;
      dsum += lane >= 1 && lane <= deep ? (long long)lane * (after - starts) : 0;
    }
    if (!apart) {
      __syncthreads();  // the positions of the sort have been read
      clear();
    }
    if (s + (int)gridDim.x < sv.src_count) levels(s + (int)gridDim.x);  // of the next source, in time for its sort
    __syncthreads();
    const uint32_t q0 = q_at + 4u * (uint32_t)t, q1 = q_at + 4u * (uint32_t)max(total - 1, 0);
    if (deep > 0) {
      FlowPiece<1> a, b, c;
      a.enter(1, starts);
      b = a;
      b.next(starts);
      c = b;
      c.next(starts);
      // An entry that has been worked on has its node too.
      const auto node = [&](const FlowPiece<1>& p) { return (lds_get<uint32_t>(min(q0 + 4u * (uint32_t)p.base, q1)) & kNode) << kId; };
      struct Ahead {
        uint32_t node, weight[2 * KS];
        Row row;
        __device__ __forceinline__ void request(const SmallView& sv, const SmallSssp& ss) {
          row.load(sv.in, node);
          const uint32_t* const w = ss.weight + (size_t)((node >> kId) * (uint32_t)(2 * KS));
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j) weight[j] = w[j];
        }
      };
      // A piece, after the links of the next one have been asked for; the node after that one takes the piece's place.
      const auto step = [&](Ahead& here, Ahead& next) {
        flow_arrived(here.row);
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) asm volatile("" ::"v"(here.weight[j]));
        next.request(sv, ss);
        const uint32_t then = node(c);
        if (t < a.end - a.base) {
          uint32_t from[2 * KS], y[2 * KS];
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j) {
            from[j] = here.row.template at<2>(j);
            y[j] = lds_get<uint32_t>(from[j]);
          }
          __builtin_amdgcn_sched_barrier(0);
          // The chosen link, place and neighbour, as in a queue entry.
          uint32_t cost, link = 0;
          const auto choose = [&](auto zero) {
            using Cost = decltype(zero);
            uint32_t sum[2 * KS];
#pragma unroll
            for (int j = 0; j < 2 * KS; ++j) sum[j] = (uint32_t)__builtin_elementwise_add_sat((Cost)y[j], (Cost)here.weight[j]);
            Cost best = (Cost)sum[0];
#pragma unroll
            for (int j = 1; j < 2 * KS; ++j) best = min(best, (Cost)sum[j]);
            cost = (uint32_t)best;
#pragma unroll
            for (int j = 2 * KS - 1; j >= 0; --j) {  // the lowest link of equals stays
              const uint32_t one = from[j] << (kFlowSsspNode - 2) | (uint32_t)j << kHandedShift;
              link = sum[j] == cost ? one : link;
            }
          };
          if (a.level & 1)
            choose(0u);
          else
            choose(0);
          lds_put<uint32_t>(Row::template own<2>(here.node), cost ^ 0x80000000u);
          lds_put<uint32_t>(q0 + 4u * (uint32_t)a.base, here.node >> kId | link);
        }
        if (b.level != a.level) __syncthreads();
        here.node = then;
        a = b;
        b = c;
        c.next(starts);
      };
      Ahead n0, n1;
      n0.node = node(a);
      n1.node = node(b);
      n0.request(sv, ss);
      for (;;) {
        step(n0, n1);
        if (a.level > deep) break;
        step(n1, n0);
        if (a.level > deep) break;
      }
    }
    for (int i = t; i < S / 4; i += kWideThreads) reinterpret_cast<uint4*>(x)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    for (int p = t; p < total; p += kWideThreads) {
      const uint32_t r = q[p];
      x[r & kNode] = 1u | (r >> kHandedShift) << kHandedShift;
    }
    __syncthreads();
    if (deep > 1) {
      FlowPiece<-1> a, b;
      a.enter(deep, starts);
      b = a;
      b.next(starts);
      const auto entry = [&](const FlowPiece<-1>& p) { return lds_get<uint32_t>(min(q0 + 4u * (uint32_t)max(p.base, 0), q1)); };
      uint32_t r = entry(a);
      for (;;) {
        const uint32_t next = entry(b);
        if (t < a.end - a.base) {
          const uint32_t paths = x[r & kNode] & kPaths;
          __hip_atomic_fetch_add(&x[r >> kFlowSsspNode & kNode], paths, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (b.level != a.level) __syncthreads();
        r = next;
        a = b;
        b.next(starts);
        if (a.level < 2) break;
      }
    }
    uint32_t* const handed = ss.handed + (size_t)s * (size_t)N;
    for (int v = t; v < N; v += kWideThreads) handed[v] = x[v];
  }
  __syncthreads();
  small_totals(sv, s_small, dsum, reached, false, 0.0, false);
}

}  // namespace a2a_dev
