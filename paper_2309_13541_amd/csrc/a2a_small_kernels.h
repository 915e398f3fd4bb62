// Device code for topologies whose whole per-source state fits the LDS of a compute unit.
//
// The level kernels of a2a_kernels.h need three dependent launches per BFS level; a topology of a few
// thousand nodes is bound by that chain (about 5 us per launch), not by bytes or arithmetic.  Here one
// workgroup takes its sources from the breadth-first search to the link loads: path counts and coefs live
// in LDS (19 bytes per node and source), levels are separated by workgroup barriers, and the global traffic
// is the link table (a few tens of KB, L2-resident), a level byte per node and source, and one row of
// link loads per workgroup.  Whole calls with the level kernels and with this one: 8x8 torus 138 and 12 us, hypercube
// of 1024 nodes 262 and 42 us, 16x16x16 torus 1025 and 246 us.  Bound in the first two by the chain of LDS accesses and barriers
// from level to level, in the third by the number of LDS instructions: the vector ALUs are 1, 22 and 43 % busy, and LDS takes an
// instruction every 17 and 10 cycles in the last two, where it gives a wave random words in 7.3 and 8-byte ones in 9.9.  Every sum is
// taken in a fixed order, so the results are the same bits from run to run and for every workspace size.
#pragma once

#include <type_traits>

#include "a2a_kernels.h"
#include "a2a_plan.h"

namespace a2a_dev {

struct SmallView {
  // [N][KS] out- and in-neighbours, two per word, in link order, as 8 x id (an LDS offset that costs one addition);
  // places past a node's last link hold the node itself, which is never one level from itself.  (More than
  // 8191 nodes, single-path baseline only: the ids as they are.)
  const uint32_t* out;
  const uint32_t* in;
  double* part;             // [workgroups of the launch][KS * 2][N] link loads: of link j of node v in row j
  long long* counters;      // [workgroups of the launch][kSmallCounters]
  unsigned char* level;     // [workgroups of the launch][per_wg][small_level_bytes(N)]
  int N;
  int per;                  // sources a workgroup works on at a time, tg threads each
  int tg, ts;               // multiples of 64: ts of them at the least work on the levels
  int depth;                // deepest level of the topology
  int qshift;               // a queue entry is node id << qshift: 3, or 0 with more than 8191 nodes
  int per_wg;               // sources per workgroup: a multiple of per, at most kSmallBatch
  int wg0;                  // first workgroup of the launch among those of the call
  int src_begin, src_count;
  const double* dem;        // as in GroupView (nullptr: every pair has demand 1)
  long long dem_ld;
};

template <typename T>
__device__ __forceinline__ T& lds_at(T* base, uint32_t bytes) {
  return *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + bytes);
}
template <typename T>
__device__ __forceinline__ const T& lds_at(const T* base, uint32_t bytes) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + bytes);
}

// LDS by its byte address, for kernels that have no other than their dynamic array, which starts at 0: the compiler adds the
// array's address to every place, which is an instruction also where it is 0.  A __shared__ array in such a kernel, or in a function
// that it calls, would move the dynamic one and these would miss it (tests/test_machine_code.py looks for that in what was built).
template <typename T>
__device__ __forceinline__ T lds_get(uint32_t at) {
  return *(const __attribute__((address_space(3))) T*)at;
}
template <typename T>
__device__ __forceinline__ void lds_put(uint32_t at, T x) {
  *(__attribute__((address_space(3))) T*)at = x;
}

// Threads of a workgroup wait for each other and for what they have asked of LDS, not for memory.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The links of a node.  at<kShift>(j): 8 x id of link j shifted right, i.e. its place in an array of doubles (0), words
// (1) or bytes (3); the two halves of a word are shifted together.
template <int KS>
struct SmallRow {
  uint32_t w[KS];
  template <int kShift = 0>
  __device__ __forceinline__ uint32_t at(int j) const {
    const uint32_t x = w[j >> 1] >> kShift;
    return j & 1 ? x >> 16 : x & 0xffffu;
  }
  __device__ __forceinline__ void load(const uint32_t* __restrict__ table, uint32_t v8) {  // v8: 8 x id
    const uint32_t* const p = reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(table) + (v8 * KS >> 1));
#pragma unroll
    for (int k = 0; k < KS; ++k) w[k] = p[k];
  }
};

// Bit-parallel search from the `count` (at most kSmallBatch) consecutive sources s0, ...: bit j = source j.
// A thread owns nodes t, t + T, ...; a level ORs the words of their in-neighbours, which lie in LDS (two arrays in turn,
// so that one barrier per level is enough), and nodes that all sources have reached look no more.  (Levels that ORed
// their nodes' words into those of the out-neighbours were bound by the atomics, 18 cycles per wave and link where a
// gather takes 7.)  Bound by the instructions: so the arrays lie a constant apart, which takes no additions, and a level
// touches only those planes whose bit is set in it.  On return bit j of `seen` says whether source j reaches the node,
// bit j of plane p is bit p of the distance.  In the first small_search_bytes(N, kNodes) of the LDS.
constexpr int kSmallPlanes = 8, kSmallFewPlanes = 5;  // the few where they do
template <int kNodes, int kPlanes>
struct SmallPlanes {
  uint32_t seen[kNodes], plane[kNodes][kPlanes];
  __device__ __forceinline__ unsigned distance(int k, int j) const {  // from source j
    unsigned d = 0;
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) d |= ((plane[k][p] >> j) & 1u) << p;
    return d;
  }
  // From sources j to j + 3 (j: a multiple of 4), a byte each, kSmallUnseen where there is no path.  A multiplication takes the four
  // bits of a plane to where their bytes begin: four instructions per plane for four sources.  (Bit by bit the bytes of 32
  // sources and 16384 nodes were 65 of a search's 228 thousand cycles: 95 us, now 66.)
  __device__ __forceinline__ uint32_t distances(int k, int j) const {
    const auto spread = [&](uint32_t bits) {
      uint32_t x = __umul24(bits >> j & 15u, 0x204081u) & 0x01010101u;
      asm("" : "+v"(x));  // a factor with a shift in it would be too large for this kind of multiplication
      return x;
    };
    const uint32_t none = spread(~seen[k]);
    uint32_t d = none << 8;
    asm("" : "+v"(d));
    d -= none;
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) d |= spread(plane[k][p]) << p;
    return d;
  }
};
template <int KS, int kNodes, int kPlanes, bool kWide = false>
__device__ __forceinline__ void small_search(const SmallView& sv, int s0, int count, SmallPlanes<kNodes, kPlanes>& out) {
  const int T = (int)blockDim.x, t = (int)threadIdx.x, N = sv.N;
  const uint32_t all = ~0u >> (kSmallBatch - count);
  // links in registers, or fetched again for every level
  constexpr bool kHold = kNodes * (KS + kPlanes) <= (kPlanes > kSmallFewPlanes ? 88 : 72);
  constexpr bool kPlaces = kNodes * KS <= 12;  // held as places in LDS, a register each
  constexpr int kApart = small_search_apart(kNodes);
  SmallRow<KS> row[kHold ? kNodes : 1];
  uint32_t place[kPlaces ? kNodes : 1][2 * KS];
#pragma unroll
  for (int k = 0; k < kNodes; ++k) {
    const int v = t + T * k;
    if (kHold && v < N) {
      row[kHold ? k : 0].load(sv.in, 8 * v);
#pragma unroll
      for (int j = 0; kPlaces && j < 2 * KS; ++j) place[kPlaces ? k : 0][j] = row[kHold ? k : 0].template at<1>(j);
    }
    out.seen[k] = v >= s0 && v < s0 + count ? 1u << (v - s0) : 0u;
    if (v < N) lds_put(4 * v, out.seen[k]);
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) out.plane[k][p] = 0;
  }
  constexpr bool kLater = kNodes <= 4;  // the planes after all nodes: registers for what is new in each
  const auto level = [&](auto odd, int l) {
    constexpr int kBefore = decltype(odd)::value ? 0 : kApart, kNow = kApart - kBefore;
    uint32_t fresh[kLater ? kNodes : 1];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kNodes; ++k) {
      const int v = t + T * k;
      uint32_t& x = fresh[kLater ? k : 0];
      x = 0;
      if (v < N) {
        if (out.seen[k] != all) {
          SmallRow<KS>& r = row[kHold ? k : 0];
          if (!kHold) {
            int u = v;
            asm volatile("" : "+v"(u));  // not kept from level to level
            r.load(sv.in, 8 * u);
          }
          uint32_t m[2 * KS];
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j)
            m[j] = lds_get<uint32_t>((kPlaces ? place[kPlaces ? k : 0][j] : kWide ? 4 * r.at(j) : r.template at<1>(j)) + kBefore);
#pragma unroll
          for (int j = 1; j < 2 * KS; ++j) m[0] |= m[j];
          x = m[0] & ~out.seen[k];
        }
        lds_put(4 * v + kNow, x);
        if (!kLater) {
          out.seen[k] |= x;
#pragma unroll
          for (int p = 0; p < kPlanes; ++p) out.plane[k][p] |= (l >> p) & 1 ? x : 0u;
        }
      }
    }
    if (!kLater) return;
#pragma unroll
    for (int k = 0; k < kNodes; ++k) out.seen[k] |= fresh[kLater ? k : 0];
#pragma unroll
    for (int p = 0; p < kPlanes; ++p)
      if ((l >> p) & 1) {
#pragma unroll
        for (int k = 0; k < kNodes; ++k) out.plane[k][p] |= fresh[kLater ? k : 0];
      }
  };
  for (int l = 1; l <= sv.depth; l += 2) {
    level(std::true_type{}, l);
    if (l == sv.depth) break;
    level(std::false_type{}, l + 1);
  }
}

// The same, the levels written as a byte per source and node; to `lds`, not to `level`, where the workgroup's sources
// all have room there (loads of an 8x8 torus from 8 sources: 11.7 -> 10.8 us, with the sums by lanes).
template <int KS, int kNodes, int kPlanes = kSmallPlanes, bool kWide = false>
__device__ __forceinline__ void small_levels(const SmallView& sv, int s0, int count, unsigned char* __restrict__ level,
                                             unsigned char* lds = nullptr) {
  const auto levels = [&](auto used) {
    SmallPlanes<kNodes, decltype(used)::value> planes;
    small_search<KS, kNodes, decltype(used)::value, kWide>(sv, s0, count, planes);
    if (lds != nullptr) __syncthreads();  // the search's words may lie there
    const int T = (int)blockDim.x, t = (int)threadIdx.x, nl = (int)small_level_bytes(sv.N);
    const int rows = __builtin_amdgcn_readfirstlane(count);
#pragma unroll 1
    for (int j = 0; j < rows; j += 4) {
#pragma unroll
      for (int k = 0; k < kNodes; ++k) {
        uint32_t v = (uint32_t)(t + T * k);
        asm volatile("" : "+v"(v));  // no addresses kept from row to row
        if (v >= (uint32_t)sv.N) continue;
        const uint32_t d = planes.distances(k, j);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (j + i >= rows) break;
          if (lds != nullptr)
            lds[(uint32_t)((j + i) * nl) + v] = (unsigned char)(d >> 8 * i);
          else
            (level + (size_t)(j + i) * (size_t)nl)[v] = (unsigned char)(d >> 8 * i);
        }
      }
    }
  };
  if (kPlanes <= kSmallFewPlanes || sv.depth < 1 << kSmallFewPlanes)
    levels(std::integral_constant<int, kPlanes <= kSmallFewPlanes ? kPlanes : kSmallFewPlanes>{});
  else
    levels(std::integral_constant<int, kPlanes>{});
}

// Deepest level of any source, for a2a_topo_create: a workgroup searches from kSmallBatch sources as above, with its
// masks in LDS (three words per node), until a level finds nothing new.  deepest: host memory, a word per workgroup,
// negative before (the host waits for the last of them to change).
static __global__ void __launch_bounds__(kSmallThreads)
k_small_probe(const uint32_t* __restrict__ table, int words, int N, int* __restrict__ deepest) {
  extern __shared__ uint32_t s_masks[];
  __shared__ int s_new[2];
  uint32_t *const cur = s_masks, *const nxt = cur + N, *const seen = nxt + N;
  const int T = (int)blockDim.x, t = (int)threadIdx.x, s0 = (int)blockIdx.x * kSmallBatch;
  for (int v = t; v < N; v += T) {
    cur[v] = seen[v] = v >= s0 && v < s0 + kSmallBatch ? 1u << (v - s0) : 0u;
    nxt[v] = 0;
  }
  if (t < 2) s_new[t] = 0;
  __syncthreads();
  int l = 1;
  for (;; ++l) {  // ends: a shortest path has less than N links
    for (int v = t; v < N; v += T) {
      const uint32_t c = cur[v];
      if (c == 0) continue;
      for (int k = 0; k < words; ++k) {
        const uint32_t w = table[v * words + k];
        __hip_atomic_fetch_or(&nxt[(w & 0xffffu) >> 3], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_or(&nxt[w >> 19], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    __syncthreads();
    bool any = false;
    for (int v = t; v < N; v += T) {
      const uint32_t c = nxt[v] & ~seen[v];
      nxt[v] = 0;
      cur[v] = c;
      seen[v] |= c;
      any |= c != 0;
    }
    if (__ballot(any) != 0 && lane_id() == 0) s_new[l & 1] = l;
    __syncthreads();
    if (s_new[l & 1] != l) break;
  }
  if (t == 0) __hip_atomic_store(&deepest[blockIdx.x], l - 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// max(x, 0) and min(x, 0): one instruction each (the compiler's own adds one that quiets signalling NaNs).
__device__ __forceinline__ double plus_part(double x) {
  double r;
  asm("v_max_f64 %0, %1, 0" : "=v"(r) : "v"(x));
  return r;
}
__device__ __forceinline__ double minus_part(double x) {
  double r;
  asm("v_min_f64 %0, %1, 0" : "=v"(r) : "v"(x));
  return r;
}

// A node that a lane works on: its place in an array of doubles (8 x id) and links.  kWide: the table has the ids
// themselves (above 8191 nodes).
template <int KS, bool kWide = false>
struct SmallNode {
  uint32_t v8;
  SmallRow<KS> row;
  __device__ __forceinline__ void request(const uint32_t* __restrict__ table, uint32_t node8) {
    v8 = node8;
    row.load(table, v8);
  }
  __device__ __forceinline__ void gather(const double* x, double (&y)[2 * KS]) const {
#pragma unroll
    for (int j = 0; j < 2 * KS; ++j) y[j] = lds_at(x, kWide ? row.at(j) << 3 : row.at(j));
  }
  __device__ __forceinline__ void levels(const unsigned char* lvl, int (&m)[2 * KS]) const {
#pragma unroll
    for (int j = 0; j < 2 * KS; ++j) m[j] = lds_at(lvl, row.template at<3>(j));
  }
  // Sum of what was gathered, of the entries that are positive (negative: of the negative ones, made positive), in pairs
  // (three additions one after the other for eight links, not seven) or in link order.
  template <bool kNegative, bool kPairs>
  static __device__ __forceinline__ double sum(double (&y)[2 * KS]) {
#pragma unroll
    for (int j = 0; j < 2 * KS; ++j) y[j] = kNegative ? minus_part(y[j]) : plus_part(y[j]);
    if (kPairs) return kNegative ? -sum_pairs(y) : sum_pairs(y);
    double a = y[0];
#pragma unroll
    for (int j = 1; j < 2 * KS; ++j) a += y[j];
    return kNegative ? -a : a;
  }
  // The same in pairs over the links that lead to the given level.
  static __device__ __forceinline__ double sum_level(double (&y)[2 * KS], const int (&m)[2 * KS], int level) {
#pragma unroll
    for (int j = 0; j < 2 * KS; ++j) y[j] = m[j] == level ? y[j] : 0.0;
    return sum_pairs(y);
  }
  static __device__ __forceinline__ double sum_pairs(double (&y)[2 * KS]) {
#pragma unroll
    for (int o = 1; o < 2 * KS; o *= 2)
#pragma unroll
      for (int j = 0; j + o < 2 * KS; j += 2 * o) y[j] += y[j + o];
    return y[0];
  }
};

// Goes over the levels first, first + step, ... last (step 1 or -1), a node per lane, a barrier after every level:
// x of a node becomes f(node, look(node), sum of x over its links of `table` to the level gone over before).  For that the
// levels need not be looked up.  An in-link of a node on level l comes from level l - 1 or later and an out-link leads
// to level l + 1 or before, so at the other ends there are only: nodes of the level before; nodes of the same
// level, written or not; and nodes not written yet, whose x is 0.  Even levels are kept with a plus sign and odd ones
// with a minus sign, and a level adds up the entries of the other sign only (kSigns; x must not be negative).
// Without kSigns the levels are looked up, and x may hold anything at first.  kPairs: the links of a node are added up in
// pairs; path counts that are a result themselves keep the order of the links, which shows above 2^53.
// What a level costs is its chain of LDS accesses (64 cycles each) and branches, so there is one branch that is
// taken for two levels, and once a level's gathers are on their way, so are the next one's links, the nodes of the one after
// that and the places of the third.  (Loads of a 16x16x16 torus, 282 us, took 296 with one trip to the queue more in
// the chain and the links added up one after the other.  Scalar cursors over pieces of levels, with no loop in a
// level, took 318: their code is in the chain too.)
// tl: this thread's place among those of the source, of which the first tg take part; wide: levels may have more nodes
// than that; start[l]: where level l starts
// in the queue, for all levels up to three past the deepest gone over; the queue has one valid entry at least.
template <int KS, bool kSigns, bool kPairs, bool kWide, typename Start, typename Look, typename F>
__device__ __forceinline__ void small_sweep(const uint32_t* __restrict__ table, const unsigned short* q, const Start& start,
                                            const unsigned char* lvl, double* x, int tl, int tg, bool wide, int first, int last,
                                            int step, Look&& look, F&& f) {
  int l = first, left = (last - first) * step;  // levels after this one
  if (tl - lane_id() >= tg) {  // waves that would rarely find a node
    do {
      __syncthreads();
    } while (--left >= 0);
    return;
  }
  using Node = SmallNode<KS, kWide>;
  const int most = max(first, last) + 2;
  struct Places {
    int p, end;
  };
  const auto places = [&](int level) {
    const int k = min(max(level, 0), most);
    return Places{start[k] + tl, start[k + 1]};
  };
  const auto node = [&](const Places& a) { return (uint32_t)q[min(a.p, max(a.end - 1, 0))] << (kWide ? 3 : 0); };
  Places a = places(l), b = places(l + step), c = places(l + 2 * step);
  Node n0, n1;
  n0.request(table, node(a));
  uint32_t v = node(b);
  asm volatile("" : "+v"(v), "+v"(c.p), "+v"(c.end));  // arrived: not waited for in the first level, and so in all of them
  const auto level = [&](auto odd, const Node& cur, Node& next) {
    constexpr bool kOdd = decltype(odd)::value;
    struct Ends {
      double own, y[2 * KS];
      int m[2 * KS];
    };
    const auto gather = [&](const Node& n, Ends& e) {
      e.own = look(n.v8);
      n.gather(x, e.y);
      if (!kSigns) n.levels(lvl, e.m);
    };
    const auto finish = [&](const Node& n, Ends& e) {
      double r;
      if constexpr (kSigns) {
        r = f(n.v8, e.own, Node::template sum<!kOdd, kPairs>(e.y));
        if (kOdd) r = -r;
      } else {
        r = f(n.v8, e.own, Node::sum_level(e.y, e.m, l - step));
      }
      lds_at(x, n.v8) = r;
    };
    const bool in = a.p < a.end;
    Ends e;
    if (in) gather(cur, e);
    __builtin_amdgcn_sched_barrier(0);  // all requests first: the scheduler would rather save registers
    next.request(table, v);
    v = node(c);
    const Places d = places(l + 3 * step);
    __builtin_amdgcn_sched_barrier(0);
    if (in) finish(cur, e);
    if (wide) {
#pragma unroll 1
      for (int p = a.p + tg; p < a.end; p += tg) {
        Node n;
        Ends other;
        n.request(table, (uint32_t)q[p] << (kWide ? 3 : 0));
        gather(n, other);
        __builtin_amdgcn_sched_barrier(0);
        finish(n, other);
      }
    }
    __syncthreads();
    l += step;
    a = b;
    b = c;
    c = d;
  };
  using Odd = std::true_type;
  using Even = std::false_type;
  if (!(l & 1)) {
    level(Even{}, n0, n1);
    n0 = n1;
    if (--left < 0) return;
  }
  for (;;) {
    level(Odd{}, n0, n1);
    if (--left < 0) return;
    level(Even{}, n1, n0);
    if (--left < 0) return;
  }
}

// Where things lie in a workgroup's LDS (small_lds_bytes), and this thread's part in it.
struct SmallLds {
  unsigned short* q_all;
  int *start_all, *at_all;
  unsigned char* lvl_all;
  int slots, nq, nl;  // level slots (two of them empty for certain), queue entries, level bytes of a source
  int sg, tl;         // which of the sources this thread's wave is on, its place among the threads of that source
  __device__ __forceinline__ SmallLds(const SmallView& sv, double* lds, int state) {
    slots = sv.depth + 4;
    nq = (sv.N + 1) & ~1;
    nl = (int)small_level_bytes(sv.N);
    q_all = reinterpret_cast<unsigned short*>(lds + small_state_bytes(sv.N, sv.per, state) / 8);
    start_all = reinterpret_cast<int*>(q_all + sv.per * nq);
    at_all = start_all + sv.per * slots;
    lvl_all = reinterpret_cast<unsigned char*>(at_all + sv.per * slots * small_spread(sv.depth));
    sg = __builtin_amdgcn_readfirstlane((int)threadIdx.x / sv.tg);
    tl = (int)threadIdx.x - sg * sv.tg;
  }
  __device__ __forceinline__ unsigned short* q() const { return q_all + sg * nq; }
  __device__ __forceinline__ int* start() const { return start_all + sg * slots; }
  __device__ __forceinline__ unsigned char* lvl() const { return lvl_all + sg * nl; }
  // Most nodes of a level of the source.
  __device__ __forceinline__ int widest() const {
    int most = 0;
    for (int l = lane_id(); l < slots - 1; l += kWave) most = max(most, start()[l + 1] - start()[l]);
    return wave_max_int(most, 0);
  }
  // Threads of the source that work on the levels: enough for the widest one at a time, if the source has them.
  __device__ __forceinline__ int busy(const SmallView& sv, int widest) const {
    return min(sv.tg, max(sv.ts, (widest + kWave - 1) / kWave * kWave));
  }
};

// Takes the levels of the next `left` sources (up to sv.per of them) from `level` (null: they are in LDS) and sorts
// their nodes by level into the queues; init(v, level) is called once per node.  Adds up distances and reached nodes.  Returns the deepest
// level of these sources, the same in all threads.  kRanks: the counting pass keeps what its atomics return, so that
// the placing pass needs none (single-path baseline of 16384 nodes 2.71 -> 2.60 ms); for kernels with registers to spare
// and at most kSmallStripes nodes a thread.
template <bool kRanks, typename Init>
__device__ __forceinline__ int small_sort(const SmallView& sv, const SmallLds& lds, const unsigned char* __restrict__ level,
                                          int left, Init&& init, long long& dsum, long long& reached) {
  const int T = (int)blockDim.x, t = (int)threadIdx.x, lane = lane_id();
  const int N = sv.N, per = sv.per, slots = lds.slots, spread = small_spread(sv.depth);
  int* const start = lds.start();
  int* const at = lds.at_all + lds.sg * slots * spread;
  const unsigned char* const lvl = lds.lvl();
  unsigned short* const q = lds.q();
  for (int i = t; i < per * slots * spread; i += T) lds.at_all[i] = 0;
  const int here = min(per, left) * (lds.nl / 4);
  for (int i = t + (level != nullptr ? 0 : here); i < per * (lds.nl / 4); i += T)
    reinterpret_cast<uint32_t*>(lds.lvl_all)[i] = i < here ? reinterpret_cast<const uint32_t*>(level)[i] : 0xffffffffu;
  __syncthreads();
  int* const mine = at + (spread > 1 ? lane >> 3 : 0);
  const auto count = [&](int l) {
    return __hip_atomic_fetch_add(&mine[l * spread], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  int rank[kSmallStripes];  // of this thread's nodes among those with the same counter
  if (kRanks) {
#pragma unroll
    for (int k = 0; k < kSmallStripes; ++k) {
      if (k * sv.tg >= N) break;  // the same in all threads
      const int v = lds.tl + k * sv.tg;
      const int l = v < N ? lvl[v] : kSmallUnseen;
      if (l != kSmallUnseen) rank[k] = count(l);
      if (v < N) init(v, l);
    }
  } else {
    for (int v = lds.tl; v < N; v += sv.tg) {
      const int l = lvl[v];
      if (l != kSmallUnseen) count(l);
      init(v, l);
    }
  }
  __syncthreads();
  if (lds.tl < kWave) {
    int carry = 0;
    for (int i0 = 0; i0 < slots * spread; i0 += kWave) {
      const int i = i0 + lane, c = i < slots * spread ? at[i] : 0, l = spread > 1 ? i >> 3 : i;
      const int incl = wave_scan_incl(c);
      if (i < slots * spread) {
        at[i] = carry + incl - c;
        if (spread == 1 || (i & 7) == 0) start[l] = carry + incl - c;
      }
      carry += __builtin_amdgcn_readlane(incl, kWave - 1);
      dsum += (long long)c * l;
      reached += l > 0 ? c : 0;
    }
    if (carry == 0 && lane == 0) q[0] = 0;  // no source: the sweeps look at an entry all the same
  }
  __syncthreads();
  if (kRanks) {
#pragma unroll
    for (int k = 0; k < kSmallStripes; ++k) {
      if (k * sv.tg >= N) break;
      const int v = lds.tl + k * sv.tg;
      const int l = v < N ? lvl[v] : kSmallUnseen;
      if (l != kSmallUnseen) q[mine[l * spread] + rank[k]] = (unsigned short)(v << sv.qshift);
    }
  } else {
    for (int v = lds.tl; v < N; v += sv.tg) {
      const int l = lvl[v];
      if (l != kSmallUnseen) q[count(l)] = (unsigned short)(v << sv.qshift);
    }
  }
  __syncthreads();
  int depth = 0;
  for (int l0 = 1; l0 < slots - 1; l0 += kWave) {
    const int l = l0 + lane;
    bool any = false;
    if (l < slots - 1)
      for (int k = 0; k < per; ++k) any |= lds.start_all[k * slots + l + 1] > lds.start_all[k * slots + l];
    const uint64_t m = __ballot(any);
    if (m != 0) depth = l0 + 63 - __builtin_clzll(m);
  }
  return depth;
}

// A workgroup's totals into its counters (all threads call it).  lds: kSmallTotals words of 8 bytes, the caller's.
constexpr int kSmallTotals = kSmallThreads / kWave * 4;
__device__ __forceinline__ void small_totals(const SmallView& sv, double* lds, long long dsum, long long reached, bool inexact,
                                             double wd, bool weighted) {
  double* const s_wd = lds;
  long long(*const s_tot)[3] = reinterpret_cast<long long(*)[3]>(lds + kSmallThreads / kWave);
  const int t = (int)threadIdx.x;
  long long bad = __ballot(inexact) != 0 ? 1 : 0;
  dsum = wave_sum_long(dsum);
  reached = wave_sum_long(reached);
  if (weighted) wd = wave_sum_double(wd);
  if (lane_id() == 0) {
    s_tot[t / kWave][0] = dsum;
    s_tot[t / kWave][1] = reached;
    s_tot[t / kWave][2] = bad;
    s_wd[t / kWave] = wd;
  }
  __syncthreads();
  if (t != 0) return;
  for (int k = 1; k < (int)blockDim.x / kWave; ++k) {
    dsum += s_tot[k][0];
    reached += s_tot[k][1];
    bad |= s_tot[k][2];
    wd += s_wd[k];
  }
  long long* const c = sv.counters + (size_t)blockIdx.x * kSmallCounters;
  c[0] = dsum;
  c[1] = reached;
  c[2] = bad;
  c[3] = __double_as_longlong(wd);
}

// Link loads of sources [per_wg * workgroup, + per_wg) of the call, as one row of `part`.  The search takes up to
// kSmallBatch sources together; then, up to `per` sources at a time: the nodes are sorted by level; sigma = the
// sum over the in-links from the level before, level by level; coef = demand / sigma + the coefs of the successors,
// deepest level first; then every thread goes over the out-links of its own nodes (t, t + T, ...) and adds
// sigma(u) * coef(w) of each source, in source order, to the loads it keeps in registers for as long as the
// workgroup lives.  KS: words per node of the link tables; kNodes: nodes per thread.
template <int KS, int kNodes, bool kDemand>
__global__ void __launch_bounds__(kSmallThreads) k_small_loads(SmallView sv) {
  extern __shared__ double s_small[];
  const int T = (int)blockDim.x, t = (int)threadIdx.x;
  const int N = sv.N, per = sv.per;
  const SmallLds lds(sv, s_small, kStateLoads);
  const int sg = lds.sg, tl = lds.tl, nl = lds.nl;
  double* const coef_all = s_small;
  double* const sig_all = s_small + per * N;
  const unsigned char* const lvl_all = lds.lvl_all;
  double* const coef = coef_all + sg * N;
  double* const sig = sig_all + sg * N;
  const unsigned short* const q = lds.q();
  const int* const start = lds.start();
  const unsigned char* const lvl = lds.lvl();
  unsigned char* const level = sv.level + (size_t)blockIdx.x * (size_t)sv.per_wg * (size_t)nl;

  long long dsum = 0, reached = 0;
  double largest = 0.0, wd = 0.0;

  const int s_first = (sv.wg0 + (int)blockIdx.x) * sv.per_wg;
  const int s_last = min(sv.src_count, s_first + sv.per_wg);
  const bool at_once = sv.per_wg <= per;
  small_levels<KS, kNodes>(sv, sv.src_begin + s_first, s_last - s_first, level,
                           at_once ? lds.lvl_all : nullptr);
  __syncthreads();
  double acc[kNodes][2 * KS];
#pragma unroll
  for (int k = 0; k < kNodes; ++k)
#pragma unroll
    for (int j = 0; j < 2 * KS; ++j) acc[k][j] = 0.0;
  for (int s0 = s_first; s0 < s_last; s0 += per) {
    const bool valid = s0 + sg < s_last;
    const auto init = [&](int v, int l) {
      sig[v] = l == 0 ? 1.0 : 0.0;
      if (kDemand) {
        const double d = valid ? sv.dem[(size_t)v * (size_t)sv.dem_ld + (size_t)(s0 + sg)] : 0.0;
        coef[v] = d;  // becomes coef in the backward sweep
        if (l != kSmallUnseen && l != 0) wd = __builtin_fma((double)l, d, wd);
      } else {
        coef[v] = 0.0;
      }
    };
    const int depth = small_sort<false>(sv, lds, at_once ? nullptr : level + (size_t)(s0 - s_first) * nl, s_last - s0,
                                        init, dsum, reached);
    const int widest = lds.widest(), busy = lds.busy(sv, widest);
    const bool wide = widest > busy;
    const auto nothing = [](uint32_t) { return 0.0; };
    const auto own_sigma_at = [&](uint32_t v8) { return lds_at(sig, v8); };
    if (depth > 0) {
      small_sweep<KS, true, true, false>(sv.in, q, start, lvl, sig, tl, busy, wide, 1, depth, 1, nothing, [&](uint32_t, double, double a) {
        largest = larger(largest, a);
        return a;
      });
      small_sweep<KS, !kDemand, true, false>(sv.out, q, start, lvl, coef, tl, busy, wide, depth, 1, -1, own_sigma_at,
                                [&](uint32_t v8, double s, double a) {
        const double r = recip(__builtin_fabs(s));
        return (kDemand ? lds_at(coef, v8) * r : r) + a;
      });
    }
    // The links of this thread's nodes.  They are the same in every round: the empty asm keeps the compiler
    // from holding on to them (it would spill registers for that).
    int u = t;
#pragma unroll
    for (int k = 0; k < kNodes; ++k, u += T) {
      asm volatile("" : "+v"(u));
      if (u < N) {
        SmallNode<KS> n;
        n.row.load(sv.out, 8 * u);
#pragma unroll 1
        for (int s = 0; s < per; ++s) {
          const double* const c_s = coef_all + s * N;
          const unsigned char* const l_s = lvl_all + s * nl;
          const double g = __builtin_fabs(sig_all[s * N + u]);
          int m[2 * KS];
          n.levels(l_s, m);
          double y[2 * KS];
          n.gather(c_s, y);
          const int next = (int)l_s[u] + 1;
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j) {
            const double c = m[j] == next ? y[j] : 0.0;
            acc[k][j] = __builtin_fma(g, kDemand ? c : __builtin_fabs(c), acc[k][j]);
          }
        }
      }
    }
    __syncthreads();
  }

  // A row of nodes per link number: a wave stores 512 bytes in one piece.  (With a node's links side by side a store touched 64
  // pieces of 16 bytes: 1024 nodes of degree 10 12.5 of the kernel's 72 thousand cycles, whole call 55.4 us, now 51.5; 16x16x16
  // torus 270, now 263.)
#pragma unroll
  for (int k = 0; k < kNodes; ++k) {
    const int u = t + T * k;
    if (u < N) {
      double* const out = sv.part + (size_t)blockIdx.x * (size_t)(2 * KS) * (size_t)N + (size_t)u;
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) out[(size_t)j * (size_t)N] = acc[k][j];
    }
  }
  small_totals(sv, s_small, dsum, reached, largest >= kTwo53, wd, kDemand);
}

// Link loads of topologies that give a thread a node or two, a source at a time, as rows like those of k_small_loads.  A thread keeps
// its nodes' links, levels, path counts and link loads in registers.  Forward, a level has the nodes without a level
// add up their in-neighbours' path counts: a sum that is not zero is the node's own and puts it on this level, so the
// search and the path counts are one sweep, and nothing is sorted.  Backward, the nodes of a level add up the coefs of their
// out-neighbours, and what each link brought, times the path count, is its load.  Values of even and of odd levels lie in two arrays, 0
// where there is none: a node without a level at level l has in-links from level l - 1 or later, and the later ones are not in
// the array of the level before; out-links of level l lead to levels up to l + 1, and those below l are not yet written.
// Bound by the chain of a level: gathers, sum, store, barrier (hypercube of 1024 nodes: waves wait half of the time, vector ALUs are busy
// 27, LDS 32 % of it).  Whole calls, k_small_loads and this, in a replayed graph: 8x8 torus 10.3, 6.2 us, 256 nodes of degree 8 12.7, 9.5,
// 512 of degree 4 16.2, 13.0, 1000 of degree 8 34.7, 31.2; one by one the smallest take as long as the host takes to launch them (8x8 torus
// 11.5 us for both).  Where k_small_loads is the faster one: node_fits.  kSources of them at a time, side by side in LDS (unit demands;
// where that is faster: node_pairs); a link's loads from two sources are then added up level by level, the deepest first, and not source
// by source.  One at a time has no loop over sources in its backward sweep, not even one of a single pass: with it 10 links of two nodes a
// thread spilled 12 bytes, with demands 52 where they spill 32, and demands were asked for before the first stores to LDS (1300 nodes of degree 10
// 30.4, 30.8 us, with demands 31.5, 32.9, of 768 sources 54.2, 57.9; now 30.4, 31.7, 54.3).
template <int KS, int kNodes, int kSources, bool kDemand>
__global__ void __launch_bounds__(kSmallThreads) k_node_loads(SmallView sv) {
  static_assert(kSources == 1 || !kDemand);
  extern __shared__ double s_small[];
  typedef double Several __attribute__((ext_vector_type(kSources)));
  using Values = std::conditional_t<kSources == 1, double, Several>;  // of a node, a source each
  // sigma of even and odd levels, coefs of even and odd levels
  constexpr uint32_t kApart = node_apart(kNodes, kSources, KS), kBytes = 8 * kSources;
  constexpr int kNever = -2, kNone = -1;
  // A node's place in an array of pairs.  Links of a generalized Kautz topology of degree 8 lead from consecutive nodes to every eighth one: 16
  // bytes each, those lie in two sixteenths of the banks.  So with 7 and 8 links the nodes of each block of 16 are permuted, another way from
  // block to block; with fewer that costs other families more than it gives this one.  (us, the faster of k_small_loads and one at a time, pairs with
  // nodes in order, permuted.  Generalized Kautz of degree 8, 1024 nodes 24.3, 26.5, 21.1, 1368 37.4, 41.3, 33.4, 1800 74.8, 57.8, 44.9, of degree 7, 900 nodes
  // 20.2, 19.6, 20.3; random, 1000 of degree 8 31.4, 30.3, 30.6; 5x5x6x6 torus, 512 sources, 23.6, 22.8, 23.5.  With up to 6 links, so left in order, 1024
  // sources of 1800 of a generalized Kautz topology of degree 5 28.2, 27.5, 30.3, 512 of a 38x40 torus 48.1, 39.9, 42.4.)
  constexpr bool kPermuted = node_permuted(KS, kSources);
  const auto place = [](uint32_t v) { return kPermuted ? v ^ (v >> 4 & 15u) : v; };
  const int T = (int)blockDim.x, t = (int)threadIdx.x, N = sv.N;
  const int s_first = (sv.wg0 + (int)blockIdx.x) * sv.per_wg;
  const int s_last = min(sv.src_count, s_first + sv.per_wg);
  SmallRow<KS> in[kNodes], out[kNodes];
  double acc[kNodes][2 * KS];
#pragma unroll
  for (int k = 0; k < kNodes; ++k) {
    const int v = min(t + T * k, N - 1);
    in[k].load(sv.in, 8 * v);
    out[k].load(sv.out, 8 * v);
#pragma unroll
    for (int j = 0; j < KS; ++j) {  // places of 16 bits: ids are below 2048
      const auto places = [&](uint32_t w) {
        return kPermuted ? place(w >> 3 & 0x1fffu) * kBytes | place(w >> 19) * kBytes << 16 : w * kSources;
      };
      in[k].w[j] = places(in[k].w[j]);
      out[k].w[j] = places(out[k].w[j]);
    }
#pragma unroll
    for (int j = 0; j < 2 * KS; ++j) acc[k][j] = 0.0;
  }
  long long dsum = 0, reached = 0;
  double largest = 0.0, wd = 0.0;
  for (int s = s_first; s < s_last; s += kSources) {
    int lvl[kNodes][kSources];
    double own[kNodes][kSources], demand[kNodes];
    if (s != s_first) __syncthreads();
    int n = N;
    if (kSources > 1) asm volatile("" : "+s"(n));  // what it is compared with is not kept from source to source
#pragma unroll
    for (int k = 0; k < kNodes; ++k) {
      const int v = t + T * k;
      Values first = 0.0;
#pragma unroll
      for (int i = 0; i < kSources; ++i) {
        const bool there = v < n && (kSources == 1 || s + i < s_last), source = (kSources == 1 || there) && v == sv.src_begin + s + i;
        lvl[k][i] = !there ? kNever : source ? 0 : kNone;
        own[k][i] = source ? 1.0 : 0.0;
        if constexpr (kSources == 1)
          first = own[k][i];
        else
          first[i] = own[k][i];
      }
      demand[k] = 0.0;
      if (v < n) {
        lds_put(kBytes * place(v), first);
#pragma unroll
        for (int a = 1; a < 4; ++a) lds_put(kBytes * place(v) + a * kApart, (Values)0.0);
        if (kDemand) demand[k] = sv.dem[(size_t)v * (size_t)sv.dem_ld + (size_t)s];
      }
    }
    // of source i, from what was gathered of a node's links
    const auto of = [&](const Values (&y)[2 * KS], int i, double (&x)[2 * KS]) {
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j)
        if constexpr (kSources == 1)
          x[j] = y[j];
        else
          x[j] = y[j][i];
    };
    const auto gather = [&](const SmallRow<KS>& row, uint32_t from, Values (&y)[2 * KS]) {
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) y[j] = lds_get<Values>(row.at(j) + from);
    };
    const auto any = [&](const int (&l)[kSources], int is) {
      bool x = false;
#pragma unroll
      for (int i = 0; i < kSources; ++i) x |= l[i] == is;
      return x;
    };
    const auto forward = [&](auto odd, int l) {
      constexpr uint32_t kNow = decltype(odd)::value ? kApart : 0, kBefore = kApart - kNow;
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kNodes; ++k) {
        if (!any(lvl[k], kNone)) continue;
        Values y[2 * KS];
        gather(in[k], kBefore, y);
#pragma unroll
        for (int i = 0; i < kSources; ++i) {
          double x[2 * KS];
          of(y, i, x);
          const double a = SmallNode<KS>::sum_pairs(x);
          if ((kSources == 1 || lvl[k][i] == kNone) && a > 0.0) {
            lvl[k][i] = l;
            own[k][i] = a;
            lds_put(kBytes * place(t + T * k) + 8 * i + kNow, a);
          }
        }
      }
    };
    for (int l = 1; l <= sv.depth; l += 2) {
      forward(std::true_type{}, l);
      if (l == sv.depth) break;
      forward(std::false_type{}, l + 1);
    }
    const auto backward = [&](auto odd, int l) {
      constexpr uint32_t kNow = 2 * kApart + (decltype(odd)::value ? kApart : 0), kAfter = 5 * kApart - kNow;
#pragma unroll
      for (int k = 0; k < kNodes; ++k) {
        if (!any(lvl[k], l)) continue;
        Values y[2 * KS];
        gather(out[k], kAfter, y);
        const auto add = [&](int i) {
          double x[2 * KS];
          of(y, i, x);
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j) acc[k][j] = __builtin_fma(own[k][i], x[j], acc[k][j]);
          const double r = recip(own[k][i]);
          lds_put(kBytes * place(t + T * k) + 8 * i + kNow, (kDemand ? demand[k] * r : r) + SmallNode<KS>::sum_pairs(x));
        };
        if constexpr (kSources == 1) {
          add(0);
        } else {  // (not a loop of one pass: see above)
#pragma unroll
          for (int i = 0; i < kSources; ++i)
            if (lvl[k][i] == l) add(i);
        }
      }
      __syncthreads();
    };
    int l = sv.depth;
    if (!(l & 1)) backward(std::false_type{}, l--);
    for (; l > 0; l -= 2) {
      backward(std::true_type{}, l);
      backward(std::false_type{}, l - 1);
    }
#pragma unroll
    for (int k = 0; k < kNodes; ++k)
#pragma unroll
      for (int i = 0; i < kSources; ++i) {
        dsum += max(lvl[k][i], 0);
        reached += lvl[k][i] > 0 ? 1 : 0;
        largest = larger(largest, own[k][i]);
        if (kDemand && lvl[k][i] > 0) wd = __builtin_fma((double)lvl[k][i], demand[k], wd);
      }
  }
#pragma unroll
  for (int k = 0; k < kNodes; ++k) {
    const int v = t + T * k;
    if (v < N) {
      double* const to = sv.part + (size_t)blockIdx.x * (size_t)(2 * KS) * (size_t)N + (size_t)v;
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j) to[(size_t)j * (size_t)N] = acc[k][j];
    }
  }
  small_totals(sv, &lds_at(s_small, 3 * kApart + kBytes * (uint32_t)node_places(N)), dsum, reached, largest >= kTwo53, wd, kDemand);
}

// Distances and path counts of the sources of a workgroup: rows of the outputs (any of them may be null), search and
// forward sweep as above.
struct SmallOut {
  int32_t* dist;    // [src_count][N]
  double* sigma;    // [src_count][N]
  long long* sums;  // [src_count]
};
template <int KS, int kNodes>
__global__ void __launch_bounds__(kSmallThreads) k_small_sigma(SmallView sv, SmallOut out) {
  extern __shared__ double s_small[];
  const int N = sv.N;
  const SmallLds lds(sv, s_small, kStateSigma);
  const int nl = lds.nl, tl = lds.tl;
  double* const sig = s_small + lds.sg * N;
  const unsigned char* const lvl = lds.lvl();
  unsigned char* const level = sv.level + (size_t)blockIdx.x * (size_t)sv.per_wg * (size_t)nl;
  long long dsum = 0, reached = 0;
  double largest = 0.0;
  const int s_first = (sv.wg0 + (int)blockIdx.x) * sv.per_wg;
  const int s_last = min(sv.src_count, s_first + sv.per_wg);
  const bool at_once = sv.per_wg <= sv.per;
  small_levels<KS, kNodes>(sv, sv.src_begin + s_first, s_last - s_first, level,
                           at_once ? lds.lvl_all : nullptr);
  __syncthreads();
  for (int s0 = s_first; s0 < s_last; s0 += sv.per) {
    long long own = 0;
    const int depth = small_sort<false>(sv, lds, at_once ? nullptr : level + (size_t)(s0 - s_first) * nl, s_last - s0,
                                        [&](int v, int l) { sig[v] = l == 0 ? 1.0 : 0.0; }, own, reached);
    const int widest = lds.widest(), busy = lds.busy(sv, widest);
    const bool wide = widest > busy;
    const auto nothing = [](uint32_t) { return 0.0; };
    if (depth > 0)
      small_sweep<KS, true, false, false>(sv.in, lds.q(), lds.start(), lvl, sig, tl, busy, wide, 1, depth, 1, nothing, [&](uint32_t, double, double a) {
        largest = larger(largest, a);
        return a;
      });
    const int s = s0 + lds.sg;
    if (s < s_last) {
      const size_t row = (size_t)s * (size_t)N;
      for (int v = tl; v < N; v += sv.tg) {
        const int l = lvl[v];
        __builtin_nontemporal_store(__builtin_fabs(sig[v]), &out.sigma[row + v]);
        if (out.dist != nullptr) __builtin_nontemporal_store(l == kSmallUnseen ? -1 : l, &out.dist[row + v]);
      }
      if (out.sums != nullptr && tl < kWave) {
        long long d = own;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o, kWave);
        if (tl == 0) out.sums[s] = d;
      }
    }
    dsum += own;
    __syncthreads();
  }
  small_totals(sv, s_small, dsum, reached, largest >= kTwo53, 0.0, false);
}

// Distances alone come straight from the planes of the search.
template <int KS, int kNodes>
__global__ void __launch_bounds__(kSmallThreads) k_small_dist(SmallView sv, SmallOut out) {
  extern __shared__ double s_small[];
  const int T = (int)blockDim.x, t = (int)threadIdx.x, N = sv.N, lane = lane_id();
  double* const s_totals = s_small + (small_search_bytes(N, kNodes) + 7) / 8;
  int* const s_sum = reinterpret_cast<int*>(s_totals + kSmallTotals);
  if (t < kSmallBatch) s_sum[t] = 0;
  const int s_first = (sv.wg0 + (int)blockIdx.x) * sv.per_wg;
  const int count = min(sv.src_count - s_first, sv.per_wg);
  long long reached = 0;
  const auto rows = [&](auto used) {
    SmallPlanes<kNodes, decltype(used)::value> planes;
    small_search<KS, kNodes, decltype(used)::value>(sv, sv.src_begin + s_first, count, planes);
#pragma unroll
    for (int k = 0; k < kNodes; ++k)
      if (t + T * k < N) reached += __popc(planes.seen[k]);
    if (t == 0) reached -= count;  // the sources themselves
#pragma unroll 1
    for (int j = 0; j < count; ++j) {
      int sum = 0;
#pragma unroll
      for (int k = 0; k < kNodes; ++k) {
        const int v = t + T * k;
        const int d = (int)planes.distance(k, j);
        if (v < N) {
          sum += d;
          if (out.dist != nullptr)
            __builtin_nontemporal_store(((planes.seen[k] >> j) & 1u) != 0 ? d : -1, &out.dist[(size_t)(s_first + j) * (size_t)N + v]);
        }
      }
      if (out.sums != nullptr) {
        sum = wave_sum_int(sum);
        if (lane == 0) __hip_atomic_fetch_add(&s_sum[j], sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  };
  if (sv.depth < 8)
    rows(std::integral_constant<int, 3>{});
  else if (sv.depth < 1 << kSmallFewPlanes)
    rows(std::integral_constant<int, kSmallFewPlanes>{});
  else
    rows(std::integral_constant<int, kSmallPlanes>{});
  if (out.sums != nullptr) {
    __syncthreads();
    if (t < count) out.sums[s_first + t] = s_sum[t];
  }
  small_totals(sv, s_totals, 0, reached, false, 0.0, false);
}

// load[a] = (first ? 0 : load[a]) + chunk sums of the launch's partial rows, kSmallChunk rows to a chunk, in
// row order throughout (a launch but the last has whole chunks, so the bits do not depend on how the
// call's workgroups are cut into launches).  A workgroup takes 32 places of the link table; thread
// (place, c) adds up chunks c, c + 8, ...  The last workgroup adds up the counters instead: running
// totals in misc[0..3] (inexact, sum of distances, reached pairs, demand x distance), and with `last` the
// call's outputs.
struct SmallTotals {
  long long pairs;  // source_count * (N - 1)
  long long* dist_sum_total;
  long long* unreachable;
  long long* flags;
  double* weighted;
};
static __global__ void __launch_bounds__(kBlock)
k_small_reduce(SmallView sv, int KS, int rows, int first, int last, const int32_t* __restrict__ out_ptr,
               double* __restrict__ load, long long* __restrict__ misc, SmallTotals tot) {
  const int t = (int)threadIdx.x;
  const int places = sv.N * KS * 2;
  if (blockIdx.x == gridDim.x - 1) {
    if (t >= kWave) return;
    long long bad = 0, dsum = 0, reached = 0;
    double wd = first ? 0.0 : __longlong_as_double(misc[3]);
    if (tot.weighted == nullptr) {  // sums of integers, and their largest: in any order
#pragma unroll 8
      for (int r = t; r < rows; r += kWave) {
        const longlong2* const c = reinterpret_cast<const longlong2*>(sv.counters + (size_t)r * kSmallCounters);
        const longlong2 sums = c[0];
        dsum += sums.x;
        reached += sums.y;
        bad |= c[1].x;
      }
    }
    for (int r0 = 0; tot.weighted != nullptr && r0 < rows; r0 += kWave) {
      const int r = r0 + t;
      double x = 0.0;
      if (r < rows) {
        const long long* const c = sv.counters + (size_t)r * kSmallCounters;
        dsum += c[0];
        reached += c[1];
        bad |= c[2];
        x = __longlong_as_double(c[3]);
      }
      for (int k = 0; k < min(kWave, rows - r0); ++k)  // one after the other, in row order
        wd += __longlong_as_double((long long)readlane64((uint64_t)__double_as_longlong(x), k));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      dsum += __shfl_xor(dsum, o, kWave);
      reached += __shfl_xor(reached, o, kWave);
      bad |= __shfl_xor(bad, o, kWave);
    }
    if (t == 0) {
      if (!first) {
        bad |= misc[0];
        dsum += misc[1];
        reached += misc[2];
      }
      misc[0] = bad;
      misc[1] = dsum;
      misc[2] = reached;
      misc[3] = __double_as_longlong(wd);
      if (last) {
        if (tot.dist_sum_total) *tot.dist_sum_total = dsum;
        if (tot.unreachable) *tot.unreachable = tot.pairs - reached;
        if (tot.flags) *tot.flags = (bad ? 1 : 0) | (tot.pairs != reached ? 2 : 0);
        if (tot.weighted) *tot.weighted = wd;
      }
    }
    return;
  }
  constexpr int kPlaces = 32, kAhead = kBlock / kPlaces;
  __shared__ double s_sum[kAhead][kPlaces];
  const int p = (int)blockIdx.x * kPlaces + (t & (kPlaces - 1)), c = t / kPlaces;
  const int j = min(p, places - 1) / sv.N, u = min(p, places - 1) - j * sv.N;
  const int a = out_ptr[u] + j;
  const bool link = p < places && a < out_ptr[u + 1];
  double run = 0.0;
  if (link && c == 0 && !first) run = load[a];
  const int chunks = (rows + kSmallChunk - 1) / kSmallChunk;
  for (int c0 = 0; c0 < chunks; c0 += kAhead) {
    double sum = 0.0;
    if (link && c0 + c < chunks) {
      const int r0 = (c0 + c) * kSmallChunk;
      const double* const x = sv.part + (size_t)r0 * (size_t)places + p;
      if (r0 + kSmallChunk <= rows) {
        double y[kSmallChunk];
#pragma unroll
        for (int k = 0; k < kSmallChunk; ++k) y[k] = x[(size_t)k * (size_t)places];
#pragma unroll
        for (int k = 0; k < kSmallChunk; ++k) sum += y[k];
      } else {
        for (int k = 0; k < rows - r0; ++k) sum += x[(size_t)k * (size_t)places];
      }
    }
    s_sum[c][t & (kPlaces - 1)] = sum;
    __syncthreads();
    if (c == 0)
      for (int k = 0; k < min(kAhead, chunks - c0); ++k) run += s_sum[k][t];
    __syncthreads();
  }
  if (link && c == 0) load[a] = run;
}

// ---------------------------------------------------------------------------------------
// single-path baseline (the reading is described in a2a_sssp_kernels.h)
// ---------------------------------------------------------------------------------------
//
// The levels do not depend on the weights: they are found for as many iterations at once as the workspace holds.
// An iteration then is two launches: its workgroups take a source at a time from the levels to what every
// node hands to the link it picked, all in LDS (8 bytes per node), and a second kernel adds that up.  Weights and
// what is handed on are kept in the places of the in-link table (node, place of the link in its in-list): a
// node's weights are one piece of memory, in ascending link id, and every node adds to one place of its own,
// so nothing is added atomically.

template <int KS, int kNodes, int kPlanes, bool kWide>
__global__ void __launch_bounds__(kSmallThreads) k_small_levels(SmallView sv) {
  extern __shared__ double s_small[];
  const int s_first = (sv.wg0 + (int)blockIdx.x) * sv.per_wg;
  small_levels<KS, kNodes, kPlanes, kWide>(sv, sv.src_begin + s_first,
                                           min(sv.src_count - s_first, sv.per_wg),
                                           sv.level + (size_t)blockIdx.x * (size_t)sv.per_wg * small_level_bytes(sv.N));
}

struct SmallSssp {
  uint32_t* weight;       // [N][2 KS] commodities routed so far over the in-links
  uint32_t* handed;       // [sources of the iteration][N]: paths that end in or pass through the node, + place << 28
};
constexpr int kHandedShift = 28;
static_assert(kBothTables < 1 << kHandedShift, "paths from one source, and the place among 16 links above them");

// Sources [per_wg * workgroup, + per_wg) of an iteration; sv.level: the levels of its first source.  Costs are
// below 2^32 - 1 (the host checks).
template <int KS>
__global__ void __launch_bounds__(kSmallThreads) k_small_sssp(SmallView sv, SmallSssp ss) {
  extern __shared__ double s_small[];
  __shared__ double s_totals[kSmallTotals];
  constexpr uint32_t kNone = 0xffffffffu;
  const int N = sv.N;
  const SmallLds lds(sv, s_small, kStateSssp);
  const int tl = lds.tl, nl = lds.nl;
  uint32_t* const cost = reinterpret_cast<uint32_t*>(s_small) + lds.sg * N;
  unsigned char* const pick = reinterpret_cast<unsigned char*>(reinterpret_cast<uint32_t*>(s_small) + sv.per * N) + lds.sg * N;
  const unsigned short* const q = lds.q();
  const int* const start = lds.start();
  const unsigned char* const lvl = lds.lvl();
  long long dsum = 0, reached = 0;
  const int s_first = (int)blockIdx.x * sv.per_wg;
  const int s_last = min(sv.src_count, s_first + sv.per_wg);
  for (int s0 = s_first; s0 < s_last; s0 += sv.per) {
    const int s = s0 + lds.sg;
    const int depth = small_sort<true>(sv, lds, sv.level + (size_t)s0 * nl, s_last - s0, [&](int v, int l) {
      if (l == 0) cost[v] = 0;
    }, dsum, reached);
    for (int l = 1; l <= depth; ++l) {
      const int end = start[l + 1];
      for (int p = start[l] + tl; p < end; p += sv.tg) {
        const int v = q[p] >> sv.qshift;
        SmallRow<KS> row;
        row.load(sv.in, 8 * v);
        uint32_t w[2 * KS];
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) w[j] = ss.weight[(size_t)v * (2 * KS) + j];
        uint32_t c[2 * KS];
        int m[2 * KS];
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) {
          const int u = (int)(row.at(j) >> sv.qshift);
          m[j] = lvl[u];
          c[j] = cost[u];
        }
        __builtin_amdgcn_sched_barrier(0);
        uint32_t best = kNone;
        int at = 0;
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) {  // ascending link id: the lowest of equals stays
          const uint32_t x = m[j] == l - 1 ? c[j] + w[j] : kNone;
          if (x < best) {
            best = x;
            at = j;
          }
        }
        cost[v] = best;
        pick[v] = (unsigned char)at;
      }
      __syncthreads();
    }
    // from here on the cost array holds the paths that end in or pass through a node
    uint32_t* const paths = cost;
    uint32_t* const handed = ss.handed + (size_t)s * (size_t)N;
    for (int v = tl; v < N; v += sv.tg) {
      paths[v] = 1;
      if (s < s_last && (lvl[v] == 0 || lvl[v] == kSmallUnseen)) handed[v] = 0;
    }
    __syncthreads();
    for (int l = depth; l >= 1; --l) {
      const int end = start[l + 1];
      for (int p = start[l] + tl; p < end; p += sv.tg) {
        const int v = q[p] >> sv.qshift;
        const uint32_t x = paths[v];
        const int j = pick[v];
        handed[v] = x | (uint32_t)j << kHandedShift;
        if (l > 1) {
          const uint32_t w = sv.in[v * KS + (j >> 1)];
          const int u = (int)((j & 1 ? w >> 16 : w & 0xffffu) >> sv.qshift);
          __hip_atomic_fetch_add(&paths[u], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
      __syncthreads();
    }
  }
  small_totals(sv, s_totals, dsum, reached, false, 0.0, false);
}

// weight[v][j] += what the sources of the iteration handed from node v to its in-link j.  A workgroup takes 64
// nodes, a lane each; its waves take every 16th source, and their sums meet in LDS.
template <int KS>
__global__ void __launch_bounds__(kSmallThreads) k_small_sssp_add(SmallSssp ss, int N, int sources) {
  __shared__ uint32_t s_sum[kSmallThreads / kWave][kWave];
  const int lane = lane_id(), wave = (int)threadIdx.x / kWave, v = (int)blockIdx.x * kWave + lane;
  constexpr int kWaves = kSmallThreads / kWave, kAhead = 8;
  uint32_t acc[2 * KS];
#pragma unroll
  for (int j = 0; j < 2 * KS; ++j) acc[j] = 0;
  if (v < N) {
    for (int s = wave; s < sources; s += kWaves * kAhead) {
      uint32_t x[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) x[k] = s + kWaves * k < sources ? ss.handed[(size_t)(s + kWaves * k) * (size_t)N + v] : 0u;
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        const uint32_t n = x[k] & ((1u << kHandedShift) - 1), at = x[k] >> kHandedShift;
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) acc[j] += at == (uint32_t)j ? n : 0u;
      }
    }
  }
  for (int j = 0; j < 2 * KS; ++j) {
    uint32_t mine = acc[0];
#pragma unroll
    for (int k = 1; k < 2 * KS; ++k) mine = j == k ? acc[k] : mine;
    s_sum[wave][lane] = mine;
    __syncthreads();
    if (wave == 0 && v < N) {
      uint32_t sum = 0;
      for (int k = 0; k < kWaves; ++k) sum += s_sum[k][lane];
      if (sum != 0) ss.weight[(size_t)v * (2 * KS) + j] += sum;
    }
    __syncthreads();
  }
}

// load of every link from its place in the in-link table.
static __global__ void __launch_bounds__(kBlock)
k_small_sssp_output(const uint32_t* __restrict__ weight, int places, const int32_t* __restrict__ in_ptr,
                    const int32_t* __restrict__ in_link, int N, double* __restrict__ load) {
  const int v = (int)(blockIdx.x * kBlock + threadIdx.x) / places, j = (int)(blockIdx.x * kBlock + threadIdx.x) % places;
  if (v >= N) return;
  const int a = in_ptr[v] + j;
  if (a < in_ptr[v + 1]) load[in_link[a]] = (double)weight[(size_t)v * places + j];
}

}  // namespace a2a_dev
