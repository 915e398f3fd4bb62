// How calls are cut into workgroups: plain host arithmetic, no HIP, so that it can be checked over its whole range
// without a device.  Included by a2a_small_kernels.h (the layout functions are constexpr: device code calls them too).
#pragma once

#include <algorithm>
#include <cstddef>

namespace a2a_dev {

// ---------------------------------------------------------------------------------------
// a handle's memory
// ---------------------------------------------------------------------------------------

// Blocks of this size at the most are kept for later handles; uploads of this size at the most go through pinned memory.
constexpr size_t kPooledBytes = 2u << 20, kStagedBytes = 4u << 20;

// A handle has one block on the device and one of pinned host memory.  What is uploaded, in this order, then scratch of the
// bound functions on the device; on the host their read-back slots and the results of the depth probe, behind the
// place where the upload is put together.  That copy stays for as long as the handle, so a larger upload goes from the
// caller's and the builder's arrays, piece by piece.  Handles made one after the other, through pinned memory and from
// the arrays: 16384 nodes of degree 8 (2.2 MB) 1.41 and 1.51 ms, 65536 of degree 8 (7.9 MB) 15.9 and 16.0 ms (the first
// of a process 19.7 and 16.7); with the table of out-links, which all topologies have by now, 8.9 MB and 16.1 ms.
enum HandlePart { kOutPtr, kOutCol, kInPtr, kInCol, kInLink, kEllOut, kEllIn, kArrived, kHandleParts };
struct HandleBlocks {
  size_t at[kHandleParts] = {}, bytes[kHandleParts] = {};
  size_t upload = 0;  // all of them, with the gaps
  bool staged = false;
  size_t scratch = 0, device = 0;
  size_t slots = 0, probe = 0, host = 0;
};
inline HandleBlocks handle_blocks(long long N, long long E, size_t ell_out, size_t ell_in, size_t arrived, size_t scratch,
                                  size_t slots, size_t probe) {
  HandleBlocks b;
  size_t off = 0;
  const auto part = [&off](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) / 256 * 256;
    return at;
  };
  const size_t ptr = ((size_t)N + 1) * 4, col = (size_t)std::max(E, 1ll) * 4;
  const size_t bytes[kHandleParts] = {ptr, col, ptr, col, col, ell_out, ell_in, arrived};
  for (int i = 0; i < kHandleParts; ++i) {
    b.bytes[i] = bytes[i];
    b.at[i] = part(bytes[i]);
  }
  b.upload = off;
  b.scratch = part(scratch);
  b.device = off;
  b.staged = b.upload <= kStagedBytes;
  off = b.staged ? b.upload : 0;
  b.slots = part(slots);
  b.probe = part(probe);
  b.host = off;
  return b;
}

// ---------------------------------------------------------------------------------------
// level kernels
// ---------------------------------------------------------------------------------------

// A launch has less than 2^32 threads: the count wraps there, and the rest is left out without an error.
constexpr long long kMostThreads = 0xffffffffll;

// Levels that a workgroup of the index kernel takes one after the other, of `levels` in all.  units: groups of 8 batches
// x blocks of 64 nodes; blocks: workgroups that a launch has for each piece of the levels.  All levels, unless that leaves
// most of the chip idle; then one, or as many as it takes for the pieces to fit a launch (64 sources of 20000 nodes in
// a ring, 10001 levels: 1.3e10 threads with a level each).
inline int offset_levels(long long units, long long blocks, int threads, int levels) {
  if (units >= 2048) return levels;
  const long long pieces = std::max(1ll, kMostThreads / threads / blocks);
  return (int)((levels + pieces - 1) / pieces);
}

// ---------------------------------------------------------------------------------------
// topologies whose per-source state fits LDS
// ---------------------------------------------------------------------------------------

constexpr int kSmallWave = 64;
constexpr int kSmallThreads = 1024;   // largest workgroup
constexpr int kSmallUnseen = 255;     // level byte of a node not reached; levels go up to 253
constexpr int kSmallBatch = 32;       // most sources of a workgroup: they search together, a bit of a word each
constexpr int kSmallStripes = 16;     // most nodes a thread sorts with their ranks in registers
constexpr int kSmallChunk = 16;       // partial load rows that are added up before they meet the running sum
constexpr int kSmallCounters = 4;     // words per workgroup: sum of distances, reached pairs, inexact, demand x distance

// LDS that one workgroup may ask for (160 KB per compute unit, a little of it taken by fixed arrays).
constexpr size_t kSmallLds = 160 * 1024 - 1024;
constexpr int kComputeUnits = 256;

// The link tables hold 8 x id in 16 bits up to here, and ids beyond, up to the nodes that the single-path baseline's
// state for one source takes in LDS.
constexpr int kScaledNodes = 8191, kBothTables = 16384;

// Level bytes of one source.
constexpr size_t small_level_bytes(int N) { return ((size_t)N + 3) & ~(size_t)3; }

// LDS of a search by workgroups of up to `nodes` nodes a thread: two arrays of a word per node, the second one where an
// instruction's constant offset reaches it.
constexpr int small_search_apart(int nodes) { return nodes * kSmallThreads * 4; }
constexpr size_t small_search_bytes(int N, int nodes) { return (size_t)small_search_apart(nodes) + (size_t)N * 4; }
// The same with a workgroup's totals (four words of 8 bytes a wave) and sums of distances behind it.
constexpr size_t small_dist_bytes(int N, int nodes) {
  return (small_search_bytes(N, nodes) + 7) / 8 * 8 + kSmallThreads / 64 * 32 + kSmallBatch * 4;
}

// LDS of a workgroup, in this order: per-node state of its sources (kState... bytes per node and source), node queue
// (16-bit places, level by level), where each level starts in the queue, cursors, level bytes.  The search is done
// before any of it is written.
constexpr int kStateLoads = 16;  // coef, sigma
constexpr int kStateSigma = 8;   // sigma
constexpr int kStateSssp = 5;    // cost, chosen link
constexpr size_t small_state_bytes(int N, int per, int state) { return ((size_t)per * N * state + 7) & ~(size_t)7; }
// Counters per level that the sort of a source's nodes works with: lanes that count the same word wait for each other (an
// add takes 180 cycles with 64 lanes on a word, 85 with eight, 57 with one), and few levels mean full ones, so they are
// spread over groups of eight lanes there: single-path baseline of 16384 nodes 3.08 -> 2.60 ms, path counts of 2000 nodes
// 52 -> 44 us.
constexpr int small_spread(int depth) { return depth < 16 ? 8 : 1; }
constexpr size_t small_lds_bytes(int N, int per, int depth, int state) {
  const size_t nq = ((size_t)N + 1) & ~(size_t)1;
  return small_state_bytes(N, per, state) +
         (size_t)per * (nq * 2 + (size_t)(depth + 4) * 4 * (1 + small_spread(depth)) + small_level_bytes(N));
}

// Threads per source: a level of the sweeps has a few percent of the nodes, a lane each.  All sources of random topologies
// of degree 4, us with 64, 128, 256, 512 threads: path counts of 160 nodes 12.7, 11.8, 11.5, 12.0 and of 385 nodes 19.2, 16.3,
// 14.6, 14.8; loads of 700 nodes 40.9, 29.7, 29.0, 31.4 and of 4096 nodes 232, 232, 232, 188.
constexpr int small_threads(int N) { return N <= 96 ? 64 : N <= 384 ? 128 : N <= 1536 ? 256 : 512; }

// The loads of the links of a thread's nodes have to fit its registers: 40 doubles (36 with two words a node).
constexpr int small_max_nodes(int ell_words) { return ell_words == 2 ? 9 : 20 / ell_words; }

enum class SmallWhat { kLoads, kSigma, kDist, kSssp };

// Nodes that a thread may own: its registers hold the loads of their links, or the bit planes of their distances.
constexpr int small_most_nodes(SmallWhat what, int ell_words) {
  return what == SmallWhat::kLoads ? small_max_nodes(ell_words) : what == SmallWhat::kSssp ? 64 : 8;
}
// Threads that each of `per` sources of a workgroup can have at the most.
constexpr int small_source_threads(int per) { return kSmallThreads / per / kSmallWave * kSmallWave; }

// Single-path baseline in 32-bit integers: a link carries at most every commodity of the call and a path has at most
// `depth` links, so no cost reaches 2^32 - 1, which stands for "none".  (Commodities of a source handed on by a node, 28
// bits, are below N, at most 16384; those of a link, 32 bits, below N squared.)
constexpr bool sssp_costs_fit(int depth, int src_count, int N) {
  return (long long)depth * src_count * (N - 1) < 0xffffffffll;
}

struct SmallCut {
  int per, tg, ts;                 // as in SmallView
  int per_wg;
  int threads, workgroups, nodes;  // of a workgroup, of the whole call, nodes per thread
  size_t lds;
};

// How a call over src_count sources is cut up; depends on the topology and src_count only (so the results
// do not depend on the workspace).  As many sources per workgroup at a time as LDS and 1024 threads allow,
// up to one workgroup for every compute unit; as many rounds as it then takes to have one
// workgroup for each place on the chip, so that the rows of partial loads stay few.  (Sources that share a workgroup search
// together; with no more sharing than leaves at least 256 workgroups, a few units had two and the rest waited: link loads of 400
// nodes of degree 4 44.5 us, now 31.5; of 900 of degree 8 55.2, 45.7; 400 sources of 3000 nodes 124, 98; path counts of 600 nodes 15.0,
// 13.7; where both rules agree, from some 1200 sources on, the same.)
inline SmallCut small_cut(int N, int depth, int ell_words, int src_count, SmallWhat what) {
  const auto up = [](int x) { return (x + kSmallWave - 1) / kSmallWave * kSmallWave; };
  SmallCut c{};
  const int state = what == SmallWhat::kLoads ? kStateLoads : what == SmallWhat::kSigma ? kStateSigma : kStateSssp;
  const int most = small_most_nodes(what, ell_words);
  int tg = small_threads(N), per = 1;
  if (what == SmallWhat::kDist) {
    tg = std::min(kSmallThreads, up(N));
    c.lds = (size_t)N * 8;
  } else {
    const int want = std::max(1, std::min(kSmallThreads / kSmallWave, (src_count + kComputeUnits - 1) / kComputeUnits));
    // fewest threads of a source that shares its workgroup: 1537 nodes of degree 4 take 50.9 us for their loads with 256,
    // 57.9 with 128 and 59.4 with 512, a 40x40 torus 96, 93 and 129
    const int least = std::min(tg, 256);
    const int stripes = what == SmallWhat::kSssp ? kSmallStripes : N;  // nodes a thread of a source may sort
    while (per < want && (per + 1) * least <= kSmallThreads && small_lds_bytes(N, per + 1, depth, state) <= kSmallLds &&
           N <= stripes * small_source_threads(per + 1))
      ++per;
    // three sources leave 64 of the 1024 threads unused, which can be too few for the nodes
    while (per > 1 && N > most * per * small_source_threads(per)) --per;
    tg = std::min(tg, small_source_threads(per));
    while (N > stripes * tg) tg += kSmallWave;
    c.lds = small_lds_bytes(N, per, depth, state);
  }
  while (N > most * per * tg) tg += kSmallWave;
  c.per = per;
  c.tg = tg;
  c.threads = per * tg;
  const int resident = (int)std::max<size_t>(1, std::min<size_t>(kSmallThreads / c.threads, kSmallLds / c.lds));
  const long long at_once = (long long)per * kComputeUnits * resident;
  c.per_wg = (int)std::min<long long>((src_count + at_once - 1) / at_once, kSmallBatch / per) * per;
  c.workgroups = (src_count + c.per_wg - 1) / c.per_wg;
  c.nodes = (N + c.threads - 1) / c.threads;
  // 1.25 times an average level: most levels in one go
  c.ts = std::min(tg, up((int)((size_t)N * 5 / 4 / (size_t)std::max(depth, 1))));
  return c;
}

// Link loads with a thread per node (k_node_loads): LDS of four arrays of a double per node and source, a constant apart, and the waves'
// totals.  The constant is part of an instruction, but for the coefs of two nodes a thread and two sources: 64 KB on, each gather of
// theirs takes an addition.  With permuted places the arrays are not a power of two apart: the compiler made a constant that sets a bit of the
// place an operation of its own, and kept the results (2 nodes and 8 links: 100 bytes a lane spilled, now 16).  In order nothing spills either
// way, and a power of two is the faster one (us, 16 bytes more and this: 40x40 torus, 512 sources 42.8, 42.1, 12x13x13 41.1, 40.8, 1397 nodes
// of degree 5 45.1, 44.5, 1500 sources of 2000 of degree 4 51.7, 51.3, 2000 of a generalized Kautz topology of degree 6 47.6, 47.1).
constexpr int kNodeMost = 2;  // nodes a thread may have
constexpr bool node_permuted(int words, int sources) { return sources > 1 && words == 4; }  // (k_node_loads)
constexpr int node_apart(int nodes, int sources, int words) {
  return nodes * kSmallThreads * 8 * sources + (node_permuted(words, sources) ? 16 : 0);
}
constexpr int node_places(int N) { return (N + 15) / 16 * 16; }  // in whole blocks of 16
constexpr size_t node_lds_bytes(int N, int nodes, int sources, int words) {
  return 3 * (size_t)node_apart(nodes, sources, words) + (size_t)node_places(N) * 8 * sources + kSmallThreads / kSmallWave * 32;
}

// A thread has a node, or two where the registers allow it (link tables of 8 words spill: 1100 nodes 124 us, k_small_loads 52).  A
// workgroup for every compute unit, its sources one after the other: two workgroups at a time on a unit would leave twice the rows
// to add up (all of 512 nodes of degree 4 13.0 us, 15.4 then; of 300 11.7, 13.3).
struct NodeCut {
  int threads, nodes, per_wg, workgroups;  // of a workgroup, per thread, sources of a workgroup, of the whole call
};
inline NodeCut node_cut(int N, int src_count) {
  NodeCut c;
  c.nodes = N <= kSmallThreads ? 1 : 2;
  c.threads = ((N + c.nodes - 1) / c.nodes + kSmallWave - 1) / kSmallWave * kSmallWave;
  c.per_wg = (src_count + kComputeUnits - 1) / kComputeUnits;
  c.workgroups = (src_count + c.per_wg - 1) / c.per_wg;
  return c;
}
// Which calls take it.  k_small_loads goes over the levels of several sources at a time, and every level only over its own nodes; here
// each source has its levels to itself, and every node without a level looks at its links.  So it is the faster one up to so many
// levels, the fewer the more sources a workgroup has and where a thread has two nodes (us, k_small_loads and this, at the edges):
//   a node a thread.  One and two sources of a workgroup, any levels: 256 nodes of degree 8 12.7, 9.5; 8x128 torus (68 levels) 59.9,
//     47.1; bidirectional ring of 500 (250) 155, 121.  Three, 15 levels: 10x10x10 torus 31.8, 30.8; 22 and more not: 24x24 torus (24)
//     26.5, 28.8.  Four, 10: hypercube of 1024 38.7, 38.0, with a fifth of its links gone 39.1, 39.0, 5x5x6x6 torus 32.0, 32.4; 4x4x8x8
//     torus (12) 34.3, 35.1, 10x10x10 (15) 36.6, 39.1.
//   two nodes.  One source, any: 2000 of degree 8 37.0, 29.5; 44x46 torus (45) 48.9, 35.6.  Two: up to 1536 nodes any, 38x40 torus
//     (39) 49.7, 47.7, 5x300 (152) 134, 113; with more nodes 30, 4x16x32 torus (26) 46.7, 46.6, or levels of at most 35 nodes, 20x102
//     torus (61) 64.3, 62.1; not 40x40 (40) 47.4, 49.7, 45x45 (44) 54.9, 59.1, 24x74 (49) 53.2, 54.2.  Three, 11: 5x6x6x6 torus 34.4,
//     34.4, 4x4x4x4x6 47.6, 45.4; 6x6x6x6 (12) 38.9, 39.4, 11x11x11 (15) 38.1, 41.9.  Four, 7: 1300 of degree 5 34.2, 34.1, of degree 6
//     (6) 35.6, 34.0; 1536 of degree 4 (8) 32.5, 33.0, of degree 3 (9) 32.1, 33.4.  Five and six, which k_small_loads takes in two
//     rounds, 11: 5x6x6x6 torus 53.1, 47.7; 6x6x6x6 (12) 60.2, 62.8.  More: 2048 of degree 4 (8) 56.4, 64.1.
inline bool node_fits(int N, int ell_words, int depth, int src_count) {
  if (N > kNodeMost * kSmallThreads || (N > kSmallThreads && ell_words > 5)) return false;
  const int sources = node_cut(N, src_count).per_wg;
  if (N <= kSmallThreads) return sources <= 2 || depth <= (sources == 3 ? 15 : 10);
  const bool few = N <= kSmallThreads * 3 / 2;
  switch (sources) {
    case 1: return true;
    case 2: return few || depth <= 30 || N <= 35 * depth;
    case 3: return depth <= 11;
    case 4: return depth <= 7;
    default: return few && depth <= 11;
  }
}

// Which calls with unit demands take its sources two at a time, whether or not node_fits has them: 16 bytes a node and gather, a barrier a
// level for both.  An odd source has such a pass to itself; 10 links of two nodes have no registers for it, 8 spill 16 bytes.  A link's loads are
// added up in another order than one source at a time has them, so a call's last bits depend on which it takes; not on the
// workspace.  (us, the faster of k_small_loads and one at a time, and this.)
// A node a thread.  Two sources: 32x32 torus 31.3, 26.5, 10x10x10 24.9, 23.1, 1000 of degree 4 17.5, 16.5, of degree 8 21.9, 21.7, 1024 of a
// generalized Kautz topology of degree 8 19.0, 17.5, hypercube of 1024 27.6, 26.8.  Four, 16 levels: 1000 of degree 4 26.9, 25.4, of degree 8 31.4, 30.3,
// 8x8x16 torus 37.5, 36.8, 10x10x10 (15) 36.8, 35.8, hypercube of 1024 38.3, 36.7; not 32x32 (32) 41.0, 42.2.  Three not: 1000 of degree 4 20.7, 21.9,
// 10x10x10 30.8, 32.1.
// Two nodes.  Two sources, up to 6 links: 38x40 torus 47.9, 40.7, 12x13x13 42.0, 40.7, 2000 of degree 4 26.9, 26.1; not with 8: 1300 28.3, 28.9, 1800
// 31.8, 32.7.  Four, up to 6 links, 8 levels: 2000 of degree 4 (8) 38.1, 37.5, 1300 of degree 5 33.6, 32.2; not 6x6x6x6 torus (12) 42.4, 45.6, nor
// 8 links, 1800 44.2, 45.1 (but 1368 of a generalized Kautz topology 31.1, 28.0).  Five, above 1536 nodes (below, one at a time is the faster
// one: 1300 of degree 5 39.5, 40.6), and six, 11: 2000 of degree 4 54.2, 47.9 and 57.9, 51.2, of degree 8 71.1, 61.6 and 76.0, 65.0; not 11x11x11 (15) with
// six 59.4, 60.7.  Seven and eight, 5: 2000 of degree 8 76.1, 75.0 and 79.3, 78.5, of a generalized Kautz topology of degree 8 75.5, 45.4 and 74.9,
// 44.6, of degree 6 58.4, 43.6 and 61.9, 46.5; not of degree 4 (8) 55.8, 58.7.
inline bool node_pairs(int N, int ell_words, int depth, int src_count) {
  if (N > kNodeMost * kSmallThreads) return false;
  const int sources = node_cut(N, src_count).per_wg;
  if (N <= kSmallThreads) return ell_words <= 5 && (sources == 2 || (sources == 4 && depth <= 16));
  if (ell_words > 4) return false;
  switch (sources) {
    case 2: return ell_words <= 3;
    case 4: return ell_words <= 3 && depth <= 8;
    case 5: return N > kSmallThreads * 3 / 2 && depth <= 11;
    case 6: return depth <= 11;
    case 7:
    case 8: return depth <= 5;
    default: return false;
  }
}

// ---------------------------------------------------------------------------------------
// search with the frontier in LDS (a2a_wide_kernels.h)
// ---------------------------------------------------------------------------------------

// LDS of a search: a word per slot and thread, and a list of the new nodes of a sparse level, 16 bits each.  A level by the list costs
// some 7 thousand cycles for 65536 nodes and 20 for a full list of 8192 entries; by the links of all nodes 66 thousand with 8
// links a node, 33 with 4.  With 64 sources a word a node's links are gone over once for all of them, and the list is the longer
// one: sums alone, without and with it, 10000 nodes of degree 3 70, 72 us, torus 25x25x26 359, 362; with 32 or 16 sources, 20011 of
// degree 5 250, 221; 40000 of a generalized Kautz topology of degree 6 716, 548; 65536 of degree 3 3542, 2669; torus 40x40x40 16.0, 14.6 ms.
constexpr int kWideList = 8192;  // entries; a thread keeps some of them in registers
constexpr bool wide_sparse(int W) { return W != 64; }
constexpr size_t wide_words_bytes(int slots) { return (size_t)slots * kSmallThreads * 4; }
constexpr int wide_list(int N, int W) { return !wide_sparse(W) ? 0 : N / 8 < kWideList ? N / 8 : kWideList; }
static_assert(wide_words_bytes(32) + kWideList * 2 <= kSmallLds);

// Whether the waves of a workgroup store the same row of distances at a time, a barrier in front of each, and not each a slot of all its rows.
// What is under way then lies in few pages, and lines that two waves share are written soon after each other; but a wave waits for the others, and
// one without a slot stays.  So it is for calls of many rows that start within a line of 64 bytes; of rows of whole lines, for the longest, for
// large calls with little work from row to row (distances of 3 bits), and for many levels, where few workgroups would store at a time.
// (us, each by itself and together.  Within a line: all of 40001 nodes of degree 3 2037, 1512, 20011 of degree 5 565, 432, 45000 of degree 8 2201, 1863, 9001
// 139, 124; 190 MB, 8750 nodes of degree 8 91.8, 87.5, 20011 105, 98.6, 30001 131, 122, 25000 116, 117; 213, 44444 nodes of degree 3 158, 160, of degree 8 165,
// 156.  Not 144 MB, 900 sources of 44444 of degree 3 147, 154, nor 300 of 20011 70.8, 76.5, nor just above 8192 nodes, where the last slot is nearly empty: 8200 of
// degree 8 105, 109, 8260 119.7, 120.7, but 8488 118, 113.
// Whole lines: 65536 of degree 8 4000, 3756, 4096 sources 384, 351, of degree 3 403, 364, all 4034, 3848, of degree 4 3624, 3699, 63488 of degree 3 3842, 3625, 4096
// sources 332, 330, 62000 of degree 8 3348, 3172; 1024 of 65536 of degree 3 196, 208.  Fewer nodes: 50000 of degree 8 2200, 2112, 56000 2654, 2553, 53248 2361,
// 2301; not 32000 sources of 48000 1300, 1323, 44800 1664, 1710, 36000 1098, 1174, nor 60000 of degree 3 3134, 3281, nor where 64 sources share a word, 16384 of
// degree 3 284, 333, 8448 of degree 8 98.7, 103.3 (but 9600 124.8, 121.7).  Tori: 36x36x36 7.92, 7.68 ms, 32x32x32 3.22, 3.07, 10922 sources of it 1.36, 1.31;
// not 4665 of 36x36x36 1325, 1339 us, nor 64 sources a word, 24x24x24 449, 451.)
inline bool wide_together(int N, int src_count, int W, int depth) {
  const long long bytes = 4ll * N * src_count;
  if (N % 16 != 0) return N >= 8400 && src_count >= 1200 && bytes >= 190000000;
  if (W == 16 && (N >= 62000 ? bytes >= 500000000 : depth < 8 && bytes >= 9000000000)) return true;
  return W != 64 && depth >= 40 && bytes >= 1400000000;
}

// ---------------------------------------------------------------------------------------
// link loads by sources in LDS, links in registers (a2a_flow_kernels.h)
// ---------------------------------------------------------------------------------------

constexpr int kFlowWords = 5;           // words of level bytes a thread sorts: at most 20480 nodes
constexpr int kFlowFewestSources = 1024;
constexpr int kFlowDeepest = 11;
constexpr int flow_nodes(int ell_words) { return ell_words == 2 ? 6 : ell_words <= 4 ? 4 : 2; }  // a thread
constexpr int flow_stride(int N) { return (N + 63) / 64 * 64; }
// LDS of k_flow_sources: in its sort and forward sweep a word and a queue entry per node and positions per thread (one for each
// level of a word of counters, one for those without), and the demands; in its backward sweep 8 bytes a node, 16 with demands.
constexpr size_t flow_places(int depth) { return (size_t)(depth <= 8 ? 9 : 17) * 2 * kSmallThreads; }
constexpr size_t flow_sort_bytes(int N, int depth) { return (size_t)flow_stride(N) * 6 + 2 * 32 + flow_places(depth); }
constexpr size_t flow_demand_at(int N, int depth) {
  return flow_sort_bytes(N, depth) > (size_t)flow_stride(N) * 8 ? flow_sort_bytes(N, depth) : (size_t)flow_stride(N) * 8;
}
constexpr size_t kFlowTail = kSmallThreads / kSmallWave * (8 + 8 * 4);  // sums of the waves
// How k_flow_sources keeps the order of a source's nodes and their path counts from its forward sweep to its backward one, without demands: both
// in LDS, in that order (kRecords), behind the 8 bytes a node of the backward sweep; the order there, path counts by node in those 8 bytes
// (kQueue); the order in memory, path counts by node (kMemory; with demands, demand / path count in memory too).  Each where there is no room
// for the one before.  In the first two the positions of the sort lie between words and queue where they fit, or behind all that.
// (us, all sources, records through memory / kQueue / kRecords: 5200 nodes of degree 8 414 / 419 / 413, 9000 of degree 8 977 / 993 / 970, of degree 16
// 1414 / 1427 / 1394, of a generalized Kautz topology of degree 4 752 / 742 / 727; 11200 of degree 6 1265 / 1260 / 1234, of degree 12 2007 / 1948 / 1899.
// Records through memory / kMemory / kQueue: 13000 of degree 6 1763 / 1748 / 1703, 16200 of degree 12 3989 / 3871 / 3739, of degree 16 4013 / 4020 / 3955.)
enum class FlowKeep { kRecords, kQueue, kMemory };
constexpr bool flow_gap(int N, int depth) { return flow_places(depth) <= (size_t)flow_stride(N) * 4; }
constexpr size_t flow_keep_bytes(int N, int depth, FlowKeep keep) {
  return keep == FlowKeep::kMemory ? flow_demand_at(N, depth)
                                   : (size_t)flow_stride(N) * (keep == FlowKeep::kRecords ? 14 : 10) + 2 * 32 + (flow_gap(N, depth) ? 0 : flow_places(depth));
}
constexpr FlowKeep flow_keep(int N, int depth, bool demand) {
  if (!demand)
    for (const FlowKeep keep : {FlowKeep::kRecords, FlowKeep::kQueue})
      if (flow_keep_bytes(N, depth, keep) <= kSmallLds) return keep;
  return FlowKeep::kMemory;
}
constexpr size_t flow_tail_at(int N, int depth, FlowKeep keep, bool demand) {
  return flow_keep_bytes(N, depth, keep) + (demand ? (size_t)flow_stride(N) * 8 : 0);
}
constexpr size_t flow_source_lds(int N, int depth, bool demand) {
  return flow_tail_at(N, depth, flow_keep(N, depth, demand), demand) + kFlowTail;
}
// Of k_flow_links: the path counts of two sources.
constexpr size_t flow_link_lds(int N) { return (size_t)flow_stride(N) * 4 * 2; }
constexpr bool flow_lds_fits(int N, int depth, bool demand) {
  return N <= kFlowWords * 4 * kSmallThreads && flow_source_lds(N, depth, demand) <= kSmallLds + kFlowTail &&
         flow_link_lds(N) <= kSmallLds;
}
// Most nodes of a topology that may come this way.
constexpr int kFlowNodes = 20352;
static_assert(flow_lds_fits(kFlowNodes, kFlowDeepest, false) && !flow_lds_fits(kFlowNodes + 1, 1, false));

// LDS of k_flow_sssp: a word per node, a word per queue entry, sums, and the positions of the sort; those lie in the place of the
// first where there is no room for both.
constexpr size_t flow_sssp_places(int depth) { return (size_t)(depth <= 8 ? 9 : 17) * 2 * kSmallThreads; }
constexpr size_t flow_sssp_tail(int N) { return ((size_t)flow_stride(N) + 32) * 4 + 512; }  // from the queue on, without positions
constexpr bool flow_sssp_apart(int N, int depth) {
  return (size_t)flow_stride(N) * 4 + flow_sssp_tail(N) + flow_sssp_places(depth) <= kSmallLds;
}
constexpr size_t flow_sssp_queue(int N, int depth) {
  const size_t state = (size_t)flow_stride(N) * 4, places = flow_sssp_apart(N, depth) ? 0 : flow_sssp_places(depth);
  return state > places ? state : places;
}
constexpr size_t flow_sssp_lds(int N, int depth) {
  return flow_sssp_queue(N, depth) + flow_sssp_tail(N) + (flow_sssp_apart(N, depth) ? flow_sssp_places(depth) : 0);
}
// Which calls take it.  Below, k_small_sssp has more than two sources in a workgroup's LDS (us there and here: 4200 nodes of degree 6
// 580, 497; 5000 of degree 4 459, 435; 8191 of degree 4 1168, 1000).  Costs have 31 bits, the largest number of which
// stands for "none".
constexpr int kFlowSsspDeepest = 15;
constexpr bool flow_sssp_fits(int N, int depth, int src_count) {
  return N > 4096 && N <= kBothTables && depth <= kFlowSsspDeepest &&
         (long long)depth * src_count * (N - 1) < 0x7fffffffll && flow_sssp_lds(N, depth) <= kSmallLds;
}

// More nodes than that, by strips of nodes (k_strip_sources).  LDS, one after the other: queue and positions of the sort; 16-bit words
// of all nodes; coefs of a level, of one strip of nodes at a time, and of a level of few nodes (StripCut).  Behind all that sums of the
// waves and where strips start in the levels.
constexpr int kStripWords = 16;  // of level bytes a thread sorts: 65536 nodes
constexpr int kStripFewestSources = 2048;
constexpr int kStripDeepest = 15, kStripMost = 4;
constexpr size_t kStripState = kSmallLds;
constexpr size_t kStripTail = kSmallThreads / kSmallWave * 8 * 4 + kStripMost * 16 * 4 + 16;
constexpr int strip_levels(int depth) { return depth <= 8 ? 8 : depth <= 12 ? 12 : 16; }
constexpr size_t strip_sort_bytes(int N, int depth) { return (size_t)flow_stride(N) * 2 + (strip_levels(depth) + 1) * 2 * kSmallThreads; }
// Bits of a word that count paths; those above are the levels up to the deepest, counted down.  All ones: the count is elsewhere.
constexpr int strip_count_bits(int depth) { return depth < 8 ? 13 : 12; }
// Strips of whole threads of the sort.  LDS of the backward sweep: a double per node of a strip and a 0 behind them; a level of few nodes
// as a bit per node, the level's nodes before each word of bits, and a double for each of the level's nodes.
constexpr int kStripFew = 4096, kStripFewLeast = 2048;  // most of those; at least
struct StripCut {
  int count, threads, nodes;  // strips; of a strip
  int bits, before, few;      // places in LDS
  int most;                   // nodes of a level of few
};
constexpr StripCut strip_cut(int N) {
  const int words = (N + 4 * kSmallThreads - 1) / (4 * kSmallThreads), used = (N + 4 * words - 1) / (4 * words);
  const int bit_words = (N + 127) / 128 * 4;
  StripCut c{};
  for (c.count = 1;; ++c.count) {
    c.threads = (used + c.count - 1) / c.count;
    c.nodes = c.threads * 4 * words;
    c.bits = c.nodes * 8 + 16;
    c.before = c.bits + bit_words * 4;
    c.few = c.before + bit_words * 2;
    const int room = ((int)kStripState - c.few) / 8;
    c.most = room < kStripFew ? room : kStripFew;
    if (c.most >= kStripFewLeast) return c;
  }
}
constexpr bool strip_lds_fits(int N, int depth) {
  return N <= kStripWords * 4 * kSmallThreads && depth <= kStripDeepest && strip_sort_bytes(N, depth) <= kStripState &&
         strip_cut(N).count <= kStripMost;
}
static_assert(kStripState + kStripTail <= 160 * 1024 && strip_lds_fits(65536, 12));
// Of k_flow_links: two sources' words, or those of one where there is no more room.
constexpr bool strip_links_single(int N) { return (size_t)flow_stride(N) * 4 > kSmallLds; }
constexpr size_t strip_link_lds(int N) { return (size_t)flow_stride(N) * (strip_links_single(N) ? 2 : 4); }
// A workgroup's queue: nodes of 16 bits, then nodes with their path counts, 32 bits.
constexpr size_t strip_record_bytes(int stride) { return (size_t)stride * 6; }

// A workgroup's queue between the two sweeps: a 16-bit node per place, with demands 8 bytes more.
constexpr size_t flow_record_bytes(int stride, bool demand) { return (size_t)stride * (demand ? 10 : 2); }

// How the sources of a call are grouped: depends on the topology and their number only.  A workgroup of k_flow_links keeps the
// loads of a block of links over a group, and the groups are added up in order; about one workgroup per compute unit.
struct FlowGroups {
  int blocks, group, groups;  // blocks of nodes, sources per group, groups
};
inline FlowGroups flow_groups(int N, int ell_words, int src_count, bool strips = false) {
  FlowGroups g;
  g.blocks = (N + flow_nodes(ell_words) * kSmallThreads - 1) / (flow_nodes(ell_words) * kSmallThreads);
  const int most = std::max(8, kComputeUnits / g.blocks / 8 * 8);
  g.group = (src_count + most - 1) / most;
  // By strips a source takes up to a megabyte of workspace, and what of a call fits it may be few groups, so they are smaller, at the price of
  // as many partial loads (65536 nodes of degree 8, with groups as above and these: 4096 sources in 1 GB 8.33, 6.42 ms; groups of 128 for all
  // 65536 sources 71.9, of 256 71.3 ms, in 1 GB 100 and 125, in 4 GB 76.6 and 76.7; of 50000 of a generalized Kautz topology of degree 5, groups as above 29.6,
  // of 128 30.6, these 30.9 ms).
  if (strips) g.group = std::min(g.group, std::min(256, std::max(128, src_count / 128)));
  g.groups = (src_count + g.group - 1) / g.group;
  return g;
}

// Whether k_flow_links after k_strip_sources has two nodes a thread for its usual four or six: where all workgroups of the groups at hand then still
// run at once.  A group's workgroups share an XCD, so that is a matter of the XCD with the most groups.  A link's load is the same sum.
// (16384 sources, ms, usual and two nodes, and workgroups of that XCD with two: 65536 nodes of degree 8, 7 groups 27.2, 25.1 (32), 8 groups 24.3, 22.6 (32),
// 11 groups 22.4, 24.7 (64), of degree 4, 8 groups 26.6, 24.6 (32), 9 groups 26.9, 28.5 (64); 50000 of a generalized Kautz topology of degree 5, 8 groups 14.0,
// 12.7 (25), 10 groups 12.7, 14.8 (50); 45000 of degree 3, 8 groups 19.8, 17.4 (22), 11 groups 18.3, 19.5 (44); 24000 of degree 8, 16 groups 8.40, 7.67 (24),
// 21 groups 8.08, 8.71 (36); 20353 of degree 6, 25 groups 6.73, 7.18 (40); 4096 of 33000 of degree 7, 7 groups 4.09, 3.72 (17), 11 groups 3.19, 3.67 (34).)
inline bool strip_links_narrow(int N, int ell_words, int groups) {
  constexpr int kXcds = 8, kNarrow = 2 * kSmallThreads;
  return flow_nodes(ell_words) > 2 && (groups + kXcds - 1) / kXcds * ((N + kNarrow - 1) / kNarrow) <= kComputeUnits / kXcds;
}

// Where things lie in the workspace: `rows` sources at a time, partial loads of `parts` groups.  rows: all, or as many whole
// groups as fit, or a part of one.
struct FlowLayout {
  int rows = 0, parts = 0;
  size_t counters = 0, weighted = 0, record = 0, part = 0, level = 0, count = 0, coef = 0, total = 0;
  size_t escaped = 0, exact = 0;  // by strips only
};
inline FlowLayout flow_layout_for(int N, int ell_words, int src_count, bool demand, int rows, int parts, bool strips = false) {
  FlowLayout l;
  l.rows = rows;
  l.parts = parts;
  size_t off = 256;
  const auto take = [&off](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) / 256 * 256;
    return at;
  };
  const size_t stride = (size_t)flow_stride(N);
  l.counters = take((size_t)kComputeUnits * kSmallCounters * 8);
  l.weighted = take((size_t)src_count * 8);
  l.record = take((size_t)std::min(rows, kComputeUnits) * (strips ? strip_record_bytes((int)stride) : flow_record_bytes((int)stride, demand)));
  l.part = take((size_t)parts * N * ell_words * 2 * 8);
  l.level = take((size_t)rows * small_level_bytes(N));
  if (strips) {
    l.escaped = take((size_t)rows * 4);
    l.exact = take((size_t)rows * stride * 4);
  }
  l.count = take((size_t)rows * stride * (strips ? 2 : 4));
  l.coef = take((size_t)rows * stride * 8);
  l.total = off;
  return l;
}
inline FlowLayout flow_layout(int N, int ell_words, int src_count, bool demand, size_t bytes, bool strips = false) {
  const FlowGroups g = flow_groups(N, ell_words, src_count, strips);
  const auto most = [bytes](int hi, auto&& at) {  // largest k in 0..hi with at(k) that fits
    int lo = 0;
    while (lo < hi) {
      const int mid = lo + (hi - lo + 1) / 2;
      if (at(mid).total <= bytes)
        lo = mid;
      else
        hi = mid - 1;
    }
    return lo;
  };
  const auto groups = [&](int k) { return flow_layout_for(N, ell_words, src_count, demand, std::min(k * g.group, src_count), k, strips); };
  const auto rows = [&](int k) { return flow_layout_for(N, ell_words, src_count, demand, k, 1, strips); };
  const int k = most(g.groups, groups);
  if (k == 0) return rows(most(g.group, rows));
  if (strips) return groups(k);
  // Of the ways to as many pieces, the one whose sources take the fewest rounds over the chip: 780 and 652 sources take seven rounds, 756 and 676
  // six (2682 nodes of degree 12, 1432 sources, 215, 206 us).
  const int pieces = (g.groups + k - 1) / k;
  const auto rounds = [&](int each) {
    const int size = each * g.group, last = src_count - (pieces - 1) * size;
    return (pieces - 1) * ((size + kComputeUnits - 1) / kComputeUnits) + (last + kComputeUnits - 1) / kComputeUnits;
  };
  int best = k;
  for (int each = k - 1; each * pieces >= g.groups; --each)
    if (rounds(each) < rounds(best)) best = each;
  return groups(best);
}

}  // namespace a2a_dev
