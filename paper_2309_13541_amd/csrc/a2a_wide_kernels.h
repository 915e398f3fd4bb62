// Distances of topologies with 8192 to 65536 nodes, and path counts of 8192 to 16384 (a2a_distances).
//
// The level kernels search from 512 sources at a time with the masks in memory: every level of every source reads a
// mask per link through the L2, whatever its frontier holds, and the rate of that is the copy rate (6.5 of 12.4 ms
// for 65536 nodes of degree 8).  Here a workgroup searches from 16, 32 or 64 sources with the frontier of a whole
// topology in LDS (a bit per node and source, 128 KB at the most): the reads per link stay in the compute unit.
// Bound by those reads (7.7 cycles for a wave's 64 in the search for link loads, where LDS gives random words in 7.3) and
// by the stores of the matrix.  Whole matrix with its sums, before and after, into the same buffers from call to call: 65536
// nodes of degree 8 12.4 -> 3.98 ms (4.3 TB/s of stores; 4.1 ms where the 17 GB are others on every call), 20011 of
// degree 5 1.31 -> 0.54 ms, 16384 of degree 4 0.79 -> 0.28 ms, torus 25x25x26 2.09 -> 0.65 ms; sums alone of 65536 nodes
// 8.45 -> 2.31 ms.
#pragma once

#include <utility>

#include "a2a_small_kernels.h"

namespace a2a_dev {

constexpr int kWideThreads = 1024;
constexpr int kWideSlots = 32;      // words of masks per thread
constexpr int kWideMost = 65536;    // nodes, with 16 sources a word
constexpr int kWideDepth = 64;      // levels are below this
constexpr int kWideEntries = kWideList / kWideThreads;  // of a sparse level's list, per thread

struct WideView {
  const uint32_t* in;   // [rows][KS] in-links, two 16-bit ids a word; rows: N rounded up to whole slots
  const uint32_t* out;  // [N][KS] out-links (not for kWideMasks)
  uint32_t* masks;      // [workgroups][depth / 2 + 1][slots][kWideThreads]; kWideMasks: see there
  long long* counters;  // [workgroups][kSmallCounters]
  int32_t* dist;        // [src_count][N], may be null
  unsigned char* level; // [src_count][small_level_bytes(N)]: the same as bytes (instead of dist)
  long long* sums;      // [src_count], may be null
  int together;         // whether the waves of a workgroup store the same row of dist at a time (wide_together)
  int N, depth, src_begin, src_count;
  int slots;            // words of masks per thread that hold nodes, at most kWideSlots
  int list;             // most entries of a sparse level's list
  long long* ltot;      // [batches of 64][Lcap]: newly reached pairs per level are added (kWideMasks)
  int Lcap;
};

// Masks of W sources: which part of a thread's slots a node has.  A slot is a 32-bit word: two nodes (W = 16),
// one (32) or half of one (64).
typedef int Int4 __attribute__((ext_vector_type(4), aligned(4)));
template <int W>
struct WideWord;
template <>
struct WideWord<16> {
  using type = uint16_t;
};
template <>
struct WideWord<32> {
  using type = uint32_t;
};
template <>
struct WideWord<64> {
  using type = uint64_t;
};

__device__ __forceinline__ uint4 wide_or(const uint4& a, const uint4& b) {
  return make_uint4(a.x | b.x, a.y | b.y, a.z | b.z, a.w | b.w);
}

__device__ __forceinline__ uint4 wide_xnor(const uint4& a, const uint4& b) {
  return make_uint4(~(a.x ^ b.x), ~(a.y ^ b.y), ~(a.z ^ b.z), ~(a.w ^ b.w));
}

// Bit planes to packed numbers: before, bit b of plane[p] is bit p of number b; after, number b is the kBits bits at
// b / kBits * kBits of plane[b % kBits].  log2(kBits) exchanges of half the bits between pairs of planes: half an
// instruction per number and stage.
template <int kBits>
__device__ __forceinline__ void wide_unpack(uint4 (&plane)[kBits]) {
#pragma unroll
  for (int s = 1; s < kBits; s *= 2) {
    const uint32_t low = s == 1 ? 0x55555555u : s == 2 ? 0x33333333u : 0x0f0f0f0fu;  // bits that stay in the lower plane
#pragma unroll
    for (int p = 0; p < kBits; ++p) {
      if (p & s) continue;
      const uint4 a = plane[p], b = plane[p + s];
      const auto lower = [&](uint32_t x, uint32_t y) { return (x & low) | ((y << s) & ~low); };
      const auto upper = [&](uint32_t x, uint32_t y) { return ((x >> s) & low) | (y & ~low); };
      plane[p] = make_uint4(lower(a.x, b.x), lower(a.y, b.y), lower(a.z, b.z), lower(a.w, b.w));
      plane[p + s] = make_uint4(upper(a.x, b.x), upper(a.y, b.y), upper(a.z, b.z), upper(a.w, b.w));
    }
  }
}

// f(0), f(1), ... in straight code.
template <typename F, size_t... I>
__device__ __forceinline__ void wide_steps(F&& f, std::index_sequence<I...>) {
  (f(std::integral_constant<int, (int)I>{}), ...);
}

// The same until one of them is false.
template <typename F, size_t... I>
__device__ __forceinline__ bool wide_steps_while(F&& f, std::index_sequence<I...>) {
  return (f(std::integral_constant<int, (int)I>{}) && ...);
}

// A workgroup takes groups of W sources, blockIdx.x, + gridDim.x, ...  Search: R_l = what a source reaches within l
// links; LDS holds R_{l-1} of all nodes, a thread R of its own (every 1024th node) and in a level ORs in the words of
// the in-neighbours.  Bit k of a distance d counts the l < d with l + 1 divisible by 2^k, so that bit plane k is the
// parity of the complements of those R_l: plane 0 is kept in registers, the others come from the R_l of the odd levels,
// which go to memory.  Then a lane takes the words of four adjacent nodes, unpacks them into distances and writes a row
// per source.  kPlanes: bits of a level.
// The first levels have few new nodes.  While those of the level before fit a list (wide_list), they are what is gone over: their
// R_{l-1} is ORed into the words of their out-neighbours, those that gain by it are the next list (a node once for every
// link that brought something), and a thread finds R_l of its own there.  65536 nodes of degree 8: four of seven levels, some 20
// thousand cycles each where the others take 66; sums alone, then in the same kernel, 3.57, 2.31 ms (with distances, then with rows a wave at a time, 4.09, 3.98).
// kOut: what is wanted.  kWideSums: no distances, a kernel of its own (18000 nodes of degree 5 207.8, 204.0 us, 65536 of degree 8 2318, 2266).  kWideMasks: the newly reached of every level 1..depth, [groups][depth][slots][kWideThreads].
// kScaled: the table has 8 x id (up to 8191 nodes; 64 sources a word only).
enum { kWideDist, kWideBytes, kWideMasks, kWideSums };
template <int W, int KS, int kPlanes, int kOut = kWideDist, bool kScaled = false>
__global__ void __launch_bounds__(kWideThreads) k_wide_dist(WideView wv) {
  using Word = typename WideWord<W>::type;
  static_assert(!kScaled || W == 64, "8 x id is the place of a 64-bit word");
  constexpr bool kBytes = kOut == kWideBytes, kMasks = kOut == kWideMasks, kSparse = !kMasks && wide_sparse(W);
  constexpr int kPerStep = W == 16 ? 2 : 1;                    // nodes a thread takes at a time
  constexpr int kWords = W == 64 ? 2 : 1;                      // slots they have
  constexpr int kSteps = kWideSlots / kWords;
  constexpr int kStride = kPerStep * kWideThreads;             // nodes per step of the workgroup
  constexpr int kLanes = W == 16 ? 16 : 32;                    // sources of a slot
  constexpr int kBits = kPlanes == 3 ? 4 : 8;                  // of a distance as it is unpacked: all set stands for -1
  constexpr auto kEach = std::make_index_sequence<kSteps>{};
  extern __shared__ double s_small[];
  Word* const front = reinterpret_cast<Word*>(s_small);
  __shared__ int s_more;
  __shared__ int s_list[2];  // entries of the list: of the odd and of the even levels
  __shared__ int s_sum[W];
  __shared__ double s_totals[kSmallTotals];
  const int t = (int)threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave), N = wv.N;
  const int last = (N - 1) / kStride;  // step
  const size_t level_words = (size_t)wv.slots * kWideThreads;
  // R_1, R_3, ..., then R of the deepest level; plane 0 takes the place of the frontier
  uint32_t* const kept = wv.masks + (size_t)blockIdx.x * (wv.depth / 2 + 1) * level_words;
  uint32_t* const kept_last = kept + (size_t)(wv.depth / 2) * level_words;
  uint32_t* const plane0 = reinterpret_cast<uint32_t*>(s_small);
  const auto source_bits = [](int v, int s0) -> Word {
    return (unsigned)(v - s0) < W ? (Word)((Word)1 << (v - s0)) : (Word)0;
  };
  long long reached = 0;
  const int groups = (wv.src_count + W - 1) / W;
  // All workgroups start together and their phases are equally long: all would search at a time and then all write at a
  // time.  The first start is spread over about the length of a search.  Without, with half, with one and a half times the spread, and as
  // it is: 65536 nodes of degree 8 3.96, 3.89, 3.92, 3.77 ms; 40001 of degree 5 1.71, 1.63, 1.52, 1.49; 20011 of degree 5 518, 473, 442, 427 us; a
  // 40x40x40 torus (60 levels) 15.6, 15.1, 16.0, 15.7 ms; rows not stored together, without, with half, as it is: 65536 of degree 3 (13 levels) 5.24, 4.57, 4.06.
  if (kOut == kWideDist && groups > 2 * (int)gridDim.x)
    for (int k = ((int)blockIdx.x >> 3) * wv.depth * wv.slots * KS / 64; k > 0; --k) __builtin_amdgcn_s_sleep(16);
  for (int g = (int)blockIdx.x; g < groups; g += (int)gridDim.x) {
    const int s_first = g * W, count = min(W, wv.src_count - s_first), s0 = wv.src_begin + s_first;
    const Word none = count == W ? (Word)0 : (Word)(~(Word)0 << count);  // bits without a source: taken for reached
    uint32_t* const group_masks = wv.masks + (size_t)g * wv.depth * level_words;
    uint32_t r[kWideSlots], even[kWideSlots];
    // conditions and addresses of the steps are worked out where they are used, not kept in registers
    int end = last, own = t;
    asm volatile("" : "+s"(end), "+v"(own));
    wide_steps([&](auto step) {
      constexpr int i = decltype(step)::value;
      const int v = i * kStride + own;
      const auto init = [&](int u) -> Word { return u < N ? (Word)(none | source_bits(u, s0)) : (Word)~(Word)0; };
      const Word x = init(v);
      if constexpr (W == 16) {
        const Word y = init(v + kWideThreads);
        r[i] = (uint32_t)x | (uint32_t)y << 16;
        if (i <= end) front[v + kWideThreads] = y;
      } else if constexpr (W == 32) {
        r[i] = x;
      } else {
        r[2 * i] = (uint32_t)x;
        r[2 * i + 1] = (uint32_t)((uint64_t)x >> 32);
      }
      if (i <= end) front[v] = x;
#pragma unroll
      for (int w = 0; w < kWords; ++w) even[i * kWords + w] = 0;
    }, kEach);
    if (t == 0) s_more = 0;
    if (t < W) s_sum[t] = 0;
    unsigned short* const list = reinterpret_cast<unsigned short*>(reinterpret_cast<uint32_t*>(s_small) + level_words);
    bool sparse = kSparse && count <= wv.list;
    if (kSparse) {
      if (t < count && sparse) list[t] = (unsigned short)(s0 + t);
      if (t == 0) {
        s_list[0] = count;
        s_list[1] = 0;
      }
    }
    __syncthreads();

    int deep = wv.depth, l = 1;
    // Of a step: which of its nodes (kPerStep) are new, and with what.
    const auto update = [&](auto step, const uint32_t (&found)[2]) {
      constexpr int i = decltype(step)::value;
#pragma unroll
      for (int w = 0; w < kWords; ++w) {
        const int slot = i * kWords + w;
        if (kMasks)
          even[slot] = found[w] & ~r[slot];  // new on this level
        else
          even[slot] ^= ~r[slot];
        r[slot] |= found[w];
      }
    };
    // Ends a level: false if it was the last.
    const auto finish = [&] {
      asm volatile("" : "+s"(end), "+v"(own));
      uint32_t* const keep = (kMasks ? group_masks + (size_t)(l - 1) * level_words : kept + (size_t)(l / 2) * level_words) + (uint32_t)own;
      uint32_t all = ~0u;
      int fresh = 0;
      wide_steps([&](auto step) {
        constexpr int i = decltype(step)::value;
        if (i > end) return;
        const int v = i * kStride + own;
        if constexpr (W == 16) {
          front[v] = (uint16_t)r[i];
          front[v + kWideThreads] = (uint16_t)(r[i] >> 16);
        } else if constexpr (W == 32) {
          front[v] = r[i];
        } else {
          front[v] = (uint64_t)r[2 * i] | (uint64_t)r[2 * i + 1] << 32;
        }
#pragma unroll
        for (int w = 0; w < kWords; ++w) {
          all &= r[i * kWords + w];
          if (kMasks) {
            keep[(i * kWords + w) * kWideThreads] = even[i * kWords + w];
            fresh += __popc(even[i * kWords + w]);
          }
        }
      }, kEach);
      if (kMasks) {
        fresh = wave_sum_int(fresh);
        if (lane == 0 && fresh != 0)
          atomicAdd((unsigned long long*)&wv.ltot[(size_t)(s_first / 64) * wv.Lcap + l], (unsigned long long)fresh);
      }
      if (__ballot(all != ~0u) != 0 && lane == 0) s_more = l;
      if (!kMasks && (l & 1) != 0 && l < wv.depth)
        wide_steps([&](auto step) {
          constexpr int i = decltype(step)::value;
          if (i > end) return;
#pragma unroll
          for (int w = 0; w < kWords; ++w) keep[(i * kWords + w) * kWideThreads] = r[i * kWords + w];
        }, kEach);
      lds_barrier();
      return s_more == l;
    };
    if constexpr (kSparse) {
      while (sparse && l <= wv.depth) {
        asm volatile("" : "+s"(end), "+v"(own));
        const int entries = s_list[(l - 1) & 1];
        uint32_t node[kWideEntries / 2];  // two a word
        Word mask[kWideEntries];
        wide_steps([&](auto k2) {
          constexpr int k = 2 * decltype(k2)::value;
          const int e = own + k * kWideThreads;
          uint32_t n0 = 0, n1 = 0;
          if (e < entries) n0 = list[e];
          if (e + kWideThreads < entries) n1 = list[e + kWideThreads];
          node[k / 2] = n0 | n1 << 16;
          mask[k] = front[n0];
          mask[k + 1] = front[n1];
        }, std::make_index_sequence<kWideEntries / 2>{});
        lds_barrier();
        if (t == 0) s_list[(l - 1) & 1] = 0;
        wide_steps_while([&](auto number) {
          constexpr int k = decltype(number)::value;
          const bool there = own + k * kWideThreads < entries;
          uint32_t gains = 0;  // a bit per link
          uint32_t link[KS];
          if (there) {
            const uint32_t* const p = wv.out + (k & 1 ? node[k / 2] >> 16 : node[k / 2] & 0xffffu) * KS;
#pragma unroll
            for (int i = 0; i < KS; ++i) link[i] = p[i];
            Word old[2 * KS];
#pragma unroll
            for (int j = 0; j < 2 * KS; ++j) {
              const uint32_t u = j & 1 ? link[j >> 1] >> 16 : link[j >> 1] & 0xffffu;
              if constexpr (W == 16)
                old[j] = (Word)(__hip_atomic_fetch_or(reinterpret_cast<uint32_t*>(front) + (u >> 1), (uint32_t)mask[k] << (u & 1) * 16,
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >> (u & 1) * 16);
              else
                old[j] = __hip_atomic_fetch_or(&front[u], mask[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 2 * KS; ++j) gains |= (mask[k] & (Word)~old[j]) != 0 ? 1u << j : 0u;
          }
          const int mine = __popc(gains), upto = wave_scan_incl(mine);
          int place = 0;
          if (lane == kWave - 1 && upto != 0) place = __hip_atomic_fetch_add(&s_list[l & 1], upto, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          place = __builtin_amdgcn_readlane(place, kWave - 1) + upto - mine;
          if (place + mine <= wv.list) {
#pragma unroll
            for (int j = 0; j < 2 * KS; ++j)
              if (gains >> j & 1) list[place++] = (unsigned short)(j & 1 ? link[j >> 1] >> 16 : link[j >> 1]);
          }
          return (k + 1) * kWideThreads < entries;
        }, std::make_index_sequence<kWideEntries>{});
        lds_barrier();
        sparse = s_list[l & 1] <= wv.list;
        uint32_t* const keep = kept + (size_t)(l / 2) * level_words + (uint32_t)own;
        const bool odd = (l & 1) != 0 && l < wv.depth;
        uint32_t all = ~0u;
        constexpr int kAtOnce = 4;  // steps
        wide_steps([&](auto four) {
          constexpr int i0 = decltype(four)::value * kAtOnce;
          if (i0 > end) return;
          uint32_t found[kAtOnce][2];
          static_assert(kWords == 1);
          wide_steps([&](auto number) {
            constexpr int k = decltype(number)::value;
            const int v = min(i0 + k, end) * kStride + own;
            found[k][0] = (uint32_t)front[v];
            if constexpr (W == 16) found[k][0] |= (uint32_t)front[v + kWideThreads] << 16;
          }, std::make_index_sequence<kAtOnce>{});
          __builtin_amdgcn_sched_barrier(0);
          wide_steps([&](auto number) {
            constexpr int k = decltype(number)::value, i = i0 + k;
            if (i > end) return;
            update(std::integral_constant<int, i>{}, found[k]);
            all &= r[i];
            if (odd) keep[i * kWideThreads] = r[i];
          }, std::make_index_sequence<kAtOnce>{});
          __builtin_amdgcn_sched_barrier(0);
        }, std::make_index_sequence<kSteps / kAtOnce>{});
        if (__ballot(all != ~0u) != 0 && lane == 0) s_more = l;
        lds_barrier();
        if (s_more != l) {
          deep = l;
          l = wv.depth;
        }
        ++l;
      }
    }
    for (; l <= wv.depth; ++l) {
      asm volatile("" : "+s"(end), "+v"(own));
      uint32_t row[2][kPerStep][KS];
      const auto fetch = [&](uint32_t (&x)[kPerStep][KS], int i) {
#pragma unroll
        for (int n = 0; n < kPerStep; ++n) {
          const uint32_t* const p = wv.in + (i * kStride + n * kWideThreads) * KS + (uint32_t)own * KS;
#pragma unroll
          for (int k = 0; k < KS; ++k) x[n][k] = p[k];
        }
      };
      fetch(row[0], 0);
      wide_steps([&](auto step) {
        constexpr int i = decltype(step)::value;
        if (i > end) return;  // the same in all threads
        fetch(row[(i + 1) & 1], min(i + 1, end));
        const uint32_t(&link)[kPerStep][KS] = row[i & 1];
        Word x[kPerStep][2 * KS];
#pragma unroll
        for (int n = 0; n < kPerStep; ++n)
#pragma unroll
          for (int j = 0; j < 2 * KS; ++j) {
            const uint32_t u = j & 1 ? link[n][j >> 1] >> 16 : link[n][j >> 1] & 0xffffu;
            x[n][j] = kScaled ? lds_at(front, u) : front[u];
          }
        __builtin_amdgcn_sched_barrier(0);
        Word acc[kPerStep];
#pragma unroll
        for (int n = 0; n < kPerStep; ++n) {
          acc[n] = x[n][0];
#pragma unroll
          for (int j = 1; j < 2 * KS; ++j) acc[n] |= x[n][j];
        }
        uint32_t found[2];
        if constexpr (W == 16) {
          found[0] = (uint32_t)acc[0] | (uint32_t)acc[kPerStep - 1] << 16;
        } else if constexpr (W == 32) {
          found[0] = acc[0];
        } else {
          found[0] = (uint32_t)acc[0];
          found[1] = (uint32_t)((uint64_t)acc[0] >> 32);
        }
        update(step, found);
      }, kEach);
      lds_barrier();
      if (!finish()) {
        deep = l;
        break;
      }
    }
    if constexpr (kMasks) {
      for (int l = deep + 1; l <= wv.depth; ++l)
        for (int i = 0; i < wv.slots; ++i) group_masks[((size_t)(l - 1) * wv.slots + i) * kWideThreads + t] = 0;
      __syncthreads();
      continue;
    }
    const bool missing = s_more == deep;  // pairs out of reach
    int bits = 0;
    asm volatile("" : "+s"(end), "+v"(own));
    wide_steps([&](auto step) {
      constexpr int i = decltype(step)::value;
      if (i > end) return;
#pragma unroll
      for (int w = 0; w < kWords; ++w) {
        const int slot = i * kWords + w;
        plane0[slot * kWideThreads + own] = even[slot];
        if (missing) kept_last[slot * kWideThreads + own] = r[slot];
        bits += __popc(~r[slot]);
      }
    }, kEach);
    reached -= bits;
    if (t == 0) reached += (long long)count * (N - 1);
    __syncthreads();

    // Distances: four waves take a slot of all the threads.  With 64 sources a wave keeps to one half of them.
    const int first = W == 64 ? (wave >> 2 & 1) * 32 : 0;  // source of bit 0
    int sum[kLanes];
#pragma unroll
    for (int j = 0; j < kLanes; ++j) sum[j] = 0;
    constexpr int kGroups = kWideThreads / (4 * kWave);
    for (int slot0 = 0; slot0 < wv.slots; slot0 += kGroups) {
      const bool there = slot0 + (wave >> 2) < wv.slots;
      // Waves without a slot stay for the barriers of the rows only (664 sources of 8300 nodes of degree 3, with barriers and without 55.5, 48.7 us).
      if (!there && (kOut != kWideDist || !wv.together)) break;
      const int slot = min(slot0 + (wave >> 2), wv.slots - 1);
      const uint32_t at = (uint32_t)slot * kWideThreads + 4 * (t & 255);
      const auto words = [&](const uint32_t* p) { return *reinterpret_cast<const uint4*>(p + at); };
      uint4 plane[kBits];
      plane[0] = words(plane0);
#pragma unroll
      for (int p = 1; p < kBits; ++p) plane[p] = make_uint4(0, 0, 0, 0);
      for (int l0 = 0; l0 < deep; l0 += 8) {
        uint4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // levels l0 + 2u + 1
          x[u] = make_uint4(~0u, ~0u, ~0u, ~0u);
          if (l0 + 2 * u + 1 < deep) x[u] = words(kept + (size_t)(l0 / 2 + u) * level_words);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int p = 1; p < kPlanes; ++p)
            if (p == 1 || (p == 2 && u % 2 == 1) || (p > 2 && u == 3 && (l0 + 8) % (1 << p) == 0)) plane[p] = wide_xnor(plane[p], x[u]);
      }
      if (missing) {
        uint4 x = words(kept_last);
        x = make_uint4(~x.x, ~x.y, ~x.z, ~x.w);
#pragma unroll
        for (int p = 0; p < kBits; ++p) plane[p] = wide_or(plane[p], x);
        if (!kBytes && wv.sums != nullptr && there)  // these are about to be counted as -1
#pragma unroll
          for (int b = 0; b < 32; ++b) sum[b % kLanes] += (x.x >> b & 1) + (x.y >> b & 1) + (x.z >> b & 1) + (x.w >> b & 1);
      }
      wide_unpack<kBits>(plane);
      const auto number = [&](int b) {  // of bit b of the words
        const uint4 x = plane[b % kBits];
        const int up = 32 - kBits - b / kBits * kBits;
        Int4 d;
        d.x = (int)(x.x << up) >> (32 - kBits);
        d.y = (int)(x.y << up) >> (32 - kBits);
        d.z = (int)(x.z << up) >> (32 - kBits);
        d.w = (int)(x.w << up) >> (32 - kBits);
        return d;
      };
      if (!kBytes && wv.sums != nullptr && there) {
#pragma unroll
        for (int b = 0; b < 32; ++b) {
          const Int4 d = number(b);
          sum[b % kLanes] += d.x + d.y + d.z + d.w;
        }
      }
      if (kOut == kWideSums) continue;
      const int v = slot / kWords * kStride + 4 * (t & 255);  // first of the lane's nodes
      int32_t* out = wv.dist + (size_t)(s_first + first) * (size_t)N;
      const auto rows = [&](auto part, auto together) {
        // Stores alone, without a search: 4.6 TB/s, 5.7 with the barrier (65536 nodes).  (The rows of two slots at a time: 65536 of degree 8 3731, 3772 us,
        // of degree 3 3921, 3789, 40001 of degree 5 1511, 1493, 20011 432, 427, a 40x40x40 torus 15.4, 15.7 ms.)
#pragma unroll
        for (int j = 0; j < kLanes; ++j) {
          if constexpr (decltype(together)::value) {
            if (j >= count) break;  // the same in all threads
            asm volatile("s_barrier" ::: "memory");
            if (first + j >= count) continue;
          } else {
            if (first + j >= count) break;
          }
#pragma unroll
          for (int n = 0; n < kPerStep; ++n) {
            const Int4 d = number(n * 16 + j);
            const uint32_t u = (uint32_t)(v + n * kWideThreads);
            if constexpr (!decltype(part)::value) {
              __builtin_nontemporal_store(d, reinterpret_cast<Int4*>(out + u));
            } else if (there && (int)u + 3 < N) {
              __builtin_nontemporal_store(d, reinterpret_cast<Int4*>(out + u));
            } else if (there) {
              if ((int)u < N) out[u] = d.x;
              if ((int)u + 1 < N) out[u + 1] = d.y;
              if ((int)u + 2 < N) out[u + 2] = d.z;
            }
          }
          out += N;
        }
      };
      if constexpr (kBytes) {
        const size_t nl = small_level_bytes(N);
        unsigned char* row = wv.level + (size_t)(s_first + first) * nl;
#pragma unroll
        for (int j = 0; j < kLanes; ++j) {
#pragma unroll
          for (int n = 0; n < kPerStep; ++n) {
            const Int4 d = number(n * 16 + j);
            const uint32_t u = (uint32_t)(v + n * kWideThreads);
            if (there && first + j < count && u < (uint32_t)N)
              *reinterpret_cast<uint32_t*>(row + u) =
                  (uint32_t)(d.x & 255) | (uint32_t)(d.y & 255) << 8 | (uint32_t)(d.z & 255) << 16 | (uint32_t)d.w << 24;
          }
          row += nl;
        }
      } else if (wv.together) {
        (slot0 + kGroups) / kWords * kStride <= N ? rows(std::false_type{}, std::true_type{}) : rows(std::true_type{}, std::true_type{});
      } else {
        (slot / kWords + 1) * kStride <= N ? rows(std::false_type{}, std::false_type{}) : rows(std::true_type{}, std::false_type{});
      }
    }
    if (!kBytes && wv.sums != nullptr) {
#pragma unroll
      for (int j = 0; j < kLanes; ++j) {
        const int x = wave_sum_int(sum[j]);
        if (lane == 0) __hip_atomic_fetch_add(&s_sum[first + j], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      __syncthreads();
      if (t < count) wv.sums[s_first + t] = s_sum[t];
    }
    __syncthreads();
  }
  if (kMasks) return;
  SmallView sv{};
  sv.counters = wv.counters;
  small_totals(sv, s_totals, 0, reached, false, 0.0, false);
}

// Index entries of the level kernels from the masks of the search: a workgroup takes a level of a batch of 64 sources
// (64 / W groups of the search), blockIdx.x = level * G + batch.  Rows follow each other in node order, levels follow
// each other.  Level 0 is the sources; a level past gv.ltot's last is empty.  Bound by the 16 bytes per node and level
// that it writes, a kilobyte per wave and store: 12.4 GB in 2.47 ms for 65536 nodes of degree 8, the rate of a copy.
template <int W>
__global__ void __launch_bounds__(kWideThreads) k_wide_index(WideView wv, GroupView gv) {
  static_assert(W == 16 || W == 64, "");
  constexpr int kGroups = 64 / W;
  __shared__ int s_wave[2][4][kWideThreads / kWave];
  const int t = (int)threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int level = (int)blockIdx.x / gv.G, g = (int)blockIdx.x % gv.G;
  const int s0 = wv.src_begin + g * 64, count = min(64, wv.src_count - g * 64);
  long long* const lt = gv.ltot + (size_t)g * gv.Lcap;
  NodeIdx* const out = gv.idxb + ((size_t)g * gv.Lcap + level) * gv.Npad;
  const int groups = (wv.src_count + W - 1) / W;
  const size_t level_words = (size_t)wv.slots * kWideThreads;
  const bool empty = level > wv.depth || (level > 0 && lt[level] == 0);
  if (empty && level > 1 && lt[level - 1] == 0) return;  // past the batch's first empty level: nothing looks at it
  // 64 levels at a time (one after the other, loads of a ring of 8000 nodes, 4000 levels, took 372 ms instead of 233, and
  // 286 with the level search).  What is read here stays below a quarter of what is written.
  uint32_t off = 0;
  for (int l = lane; l < level; l += kWave) off += l == 0 ? (uint32_t)count : (uint32_t)lt[l];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) off += (uint32_t)__shfl_xor((int)off, o, kWave);
  if (level == 0) {
    if (t < count) gv.datf[(size_t)g * gv.Npad * 128 + t] = 1.0f;
    if (t == 0) lt[0] = count;
    for (int l = t; l < gv.Lcap; l += kWideThreads) gv.dag[(size_t)g * gv.Lcap + l] = 0;
  }
  for (int b0 = 0; b0 * kWideThreads < gv.Npad; b0 += 4) {  // four blocks of a thousand nodes
    uint64_t m[4] = {0, 0, 0, 0};
    if (level == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const unsigned j = (unsigned)((b0 + k) * kWideThreads + t - s0);
        m[k] = j < (unsigned)count ? 1ull << j : 0ull;
      }
    } else if (!empty) {
      const auto word = [&](int group, int slot) -> uint64_t {
        return slot < wv.slots ? wv.masks[((size_t)group * wv.depth + (level - 1)) * level_words + (size_t)slot * kWideThreads + t] : 0u;
      };
      if constexpr (W == 64) {
#pragma unroll
        for (int k = 0; k < 4; ++k) m[k] = word(g, 2 * (b0 + k)) | word(g, 2 * (b0 + k) + 1) << 32;
      } else {
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
          if (g * kGroups + i >= groups) continue;
#pragma unroll
          for (int k = 0; k < 4; k += 2) {
            const uint64_t x = word(g * kGroups + i, (b0 + k) / 2);
            m[k] |= (x & 0xffffu) << (i * W);
            m[k + 1] |= (x >> 16) << (i * W);
          }
        }
      }
    }
    int c[4], incl[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = __popcll(m[k]);
#pragma unroll
    for (int k = 0; k < 4; k += 2) {  // at most 64 x 64 in a wave
      const int two = wave_scan_incl(c[k] | c[k + 1] << 16);
      incl[k] = two & 0xffff;
      incl[k + 1] = two >> 16;
    }
    if (lane == kWave - 1) {
#pragma unroll
      for (int k = 0; k < 4; ++k) s_wave[b0 / 4 & 1][k][wave] = incl[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      // lane w (of each 16) has wave w's sum
      const int x = s_wave[b0 / 4 & 1][k][lane & 15];
      int upto = x;
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        const int y = __shfl_up(upto, o, 16);
        if ((lane & 15) >= o) upto += y;
      }
      const int before = __builtin_amdgcn_readlane(upto - x, wave), all = __builtin_amdgcn_readlane(upto, 15);
      const int v = (b0 + k) * kWideThreads + t;
      if (v < gv.Npad)
        *reinterpret_cast<ulonglong2*>(&out[v]) = make_ulonglong2(m[k], (unsigned long long)(off + (uint32_t)(before + incl[k] - c[k])));
      off += (uint32_t)all;
    }
  }
}

// ---------------------------------------------------------------------------------------
// path counts of 8192 to 16384 nodes
// ---------------------------------------------------------------------------------------
//
// As in the small kernels a source's path counts stay in LDS, 8 bytes per node, with the queue of its nodes behind
// them: 10 bytes per node, all of the 160 KB for 16384 nodes.  So the levels come from a search of its own (bytes in
// memory), the counters of the sort lie where the path counts will be, and where a level starts in the queue is kept
// in a register, a level per lane.  (The level kernels wrote an index entry per node, level and batch, and gathered the
// counts out of their compact rows one memory latency at a time.)  Bound by the sort, the sweep and the stores: 27, 21
// and 11 thousand cycles per source of 16384 nodes of degree 5.  All sources, before and after: torus 25x25x26 27.5 -> 2.5
// ms, 16384 nodes of degree 5 11.1 -> 1.75 ms, 9000 nodes of degree 8 3.20 -> 0.63 ms.

constexpr int kWideStateNodes = 16384, kWideStateDepth = 60;
__host__ __device__ inline size_t wide_state_bytes(int N) { return (size_t)N * 8 + ((size_t)N * 2 + 7) / 8 * 8; }

struct WideStarts {
  int at;  // lane l: where level l starts
  __device__ __forceinline__ int operator[](int l) const { return __builtin_amdgcn_readlane(at, l); }
};

// Sorts the nodes of a source by level into q; `level`: its level bytes.  lds: room for the counters, free again on
// return (after a barrier).  own: sum of the distances, in wave 0 (a share per lane); reached: pairs, likewise.
__device__ __forceinline__ WideStarts wide_sort(int N, int spread, const uint32_t (&lv)[4], unsigned short* q, int* lds,
                                                long long& own, long long& reached) {
  const int t = (int)threadIdx.x, lane = lane_id();
  constexpr int kSlots = kWave;
  int *const start = lds, *const at = lds + kSlots;
  for (int i = t; i < kSlots * spread; i += kWideThreads) at[i] = 0;
  __syncthreads();
  int* const mine = at + (spread > 1 ? lane >> 3 : 0);
  uint32_t rank[8];  // of this thread's nodes among those with the same counter, two a word
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int l = (int)(lv[i / 4] >> (i % 4 * 8) & 255u);
    uint32_t r = 0;
    if (l != kSmallUnseen)
      r = (uint32_t)__hip_atomic_fetch_add(&mine[l * spread], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    rank[i / 2] = i % 2 == 0 ? r : rank[i / 2] | r << 16;
  }
  __syncthreads();
  if (t < kWave) {
    int carry = 0;
    for (int i0 = 0; i0 < kSlots * spread; i0 += kWave) {
      const int i = i0 + lane, c = at[i], l = spread > 1 ? i >> 3 : i;
      const int incl = wave_scan_incl(c);
      at[i] = carry + incl - c;
      if (spread == 1 || (i & 7) == 0) start[l] = carry + incl - c;
      carry += __builtin_amdgcn_readlane(incl, kWave - 1);
      own += (long long)c * l;
      reached += l > 0 ? c : 0;
    }
    if (carry == 0 && lane == 0) q[0] = 0;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int l = (int)(lv[i / 4] >> (i % 4 * 8) & 255u), v = 4 * (t + i / 4 * kWideThreads) + i % 4;
    if (l != kSmallUnseen) q[mine[l * spread] + (int)(rank[i / 2] >> (i % 2 * 16) & 0xffffu)] = (unsigned short)v;
  }
  WideStarts s;
  s.at = start[lane];
  __syncthreads();
  return s;
}

struct WideSigma {
  const uint32_t* in;          // [N][KS] in-links
  const unsigned char* level;  // [src_count][small_level_bytes(N)]
  long long* counters;         // [workgroups][kSmallCounters]
  int N, depth, src_count;
  SmallOut out;
};

typedef double Double2 __attribute__((ext_vector_type(2), aligned(8)));
typedef int Int2 __attribute__((ext_vector_type(2), aligned(4)));

template <int KS>
__global__ void __launch_bounds__(kWideThreads) k_wide_sigma(WideSigma ws) {
  extern __shared__ double s_small[];
  const int t = (int)threadIdx.x, lane = lane_id(), N = ws.N, nl = (int)small_level_bytes(N);
  double* const x = s_small;
  unsigned short* const q = reinterpret_cast<unsigned short*>(s_small + N);
  long long reached = 0;
  double largest = 0.0;
  for (int s = (int)blockIdx.x; s < ws.src_count; s += (int)gridDim.x) {
    const unsigned char* const level = ws.level + (size_t)s * (size_t)nl;
    uint32_t lv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = 4 * (t + k * kWideThreads);
      lv[k] = ~0u;
      if (v < N) lv[k] = *reinterpret_cast<const uint32_t*>(level + v);
      if (v + 4 > N && v < N) lv[k] |= ~0u << ((N - v) * 8);
    }
    long long own = 0;
    const WideStarts start = wide_sort(N, small_spread(ws.depth), lv, q, reinterpret_cast<int*>(x), own, reached);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int v = 4 * (t + i / 4 * kWideThreads) + i % 4;
      if (v < N) x[v] = (lv[i / 4] >> (i % 4 * 8) & 255u) == 0 ? 1.0 : 0.0;
    }
    __syncthreads();
    const int after = __shfl_down(start.at, 1, kWave);
    const uint64_t filled = __ballot(lane >= 1 && lane < kWave - 1 && after > start.at);
    const int widest = wave_max_int(lane < kWave - 1 ? after - start.at : 0, 0);
    const int busy = min(kWideThreads, (widest + kWave - 1) / kWave * kWave);
    if (filled != 0)
      small_sweep<KS, true, false, true>(ws.in, q, start, nullptr, x, t, busy, widest > busy, 1,
                                  63 - __builtin_clzll(filled), 1, [](uint32_t) { return 0.0; }, [&](uint32_t, double, double a) {
        largest = larger(largest, a);
        return a;
      });
    const size_t row = (size_t)s * (size_t)N;
    for (int v = 2 * t; v < N; v += 2 * kWideThreads) {
      const unsigned two = *reinterpret_cast<const unsigned short*>(level + v);
      const int l0 = (int)(two & 255u), l1 = (int)(two >> 8);
      if (v + 1 < N) {
        Double2 y;
        y.x = __builtin_fabs(x[v]);
        y.y = __builtin_fabs(x[v + 1]);
        __builtin_nontemporal_store(y, reinterpret_cast<Double2*>(&ws.out.sigma[row + v]));
        Int2 d;
        d.x = l0 == kSmallUnseen ? -1 : l0;
        d.y = l1 == kSmallUnseen ? -1 : l1;
        if (ws.out.dist != nullptr) __builtin_nontemporal_store(d, reinterpret_cast<Int2*>(&ws.out.dist[row + v]));
      } else {
        ws.out.sigma[row + v] = __builtin_fabs(x[v]);
        if (ws.out.dist != nullptr) ws.out.dist[row + v] = l0 == kSmallUnseen ? -1 : l0;
      }
    }
    if (ws.out.sums != nullptr && t < kWave) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) own += __shfl_xor(own, o, kWave);
      if (t == 0) ws.out.sums[s] = own;
    }
    __syncthreads();
  }
  SmallView sv{};
  sv.counters = ws.counters;
  small_totals(sv, s_small, 0, reached, largest >= kTwo53, 0.0, false);
}

}  // namespace a2a_dev
