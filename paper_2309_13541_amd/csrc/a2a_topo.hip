// a2a_topo host side: the C ABI of include/a2a_topo.h.  All-pairs hop distances, shortest-path
// counts and EwSP link loads of a direct-connect topology (Sec. 2.2, 5.2, 5.3, 5.4 of the paper)
// on one MI355X.  A call goes one of four ways, by what fits where (small_..._fit, flow_fits, strips_fit, wide_..._fit):
//   - topologies of up to 8191 nodes and 16 links a node: one kernel takes a workgroup's sources from the search to
//     their results with all state in LDS, a second adds up (a2a_small_kernels.h; single-path baseline up to 16384 nodes)
//   - link loads of up to 65536 nodes and 16 links a node from many sources: a source at a time in LDS, as a whole or by strips of nodes, and
//     a second kernel with the links' loads in registers (a2a_flow_kernels.h)
//   - up to 65536 nodes and 16 links a node: the levels come from a search with the frontier in LDS
//     (a2a_wide_kernels.h); distances straight from it, path counts of up to 16384 nodes a source at a time in LDS, link
//     loads (of those topologies of more than 4096 nodes that do not go the other ways) by the level kernels
//   - everything else: the level kernels alone (a2a_kernels.h, where their data model is described)
//
// Level kernels.  A "group" of G source batches (64 sources each) advances level by level together, one kernel
// launch per level and pass, as many batches as the caller's workspace holds:
//   bfs    levels 1 .. deepest (the handle knows the deepest level any source reaches), or the search in LDS
//   offs   row offsets of the level-compact value array
//   fwd    levels 1 .. deepest: sigma
//   bwd    levels deepest .. 0: coef and per-batch link loads
//   sum    load += per-batch loads, in ascending batch order
// Nothing in a2a_distances / a2a_link_loads waits for the device or reads anything back: the
// launch sequence is fixed by the handle, and what depends on the data (which levels a batch
// has, how full they are) is decided inside the kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "a2a_kernels.h"
#include "a2a_launch.h"
#include "a2a_sssp_kernels.h"
#include "a2a_topo.h"

using namespace a2a_dev;

// Workspace of a2a_link_loads_static.  One copy per GPU, held until the process ends; in host
// code this name only stands for the symbol: its address on a device is taken once, in
// a2a_topo_create with that device current, and kept in the handle.
static __device__ __align__(256) unsigned char scratch[A2A_STATIC_WORKSPACE_BYTES];

struct a2a_topo {
  int32_t N = 0;
  int64_t E = 0;
  int32_t dmax = 0;
  int32_t dmax_in = 0;  // largest in-degree
  int32_t level_bound = 0;  // largest finite D(s,t), found by the level probe at create
  // The handle's memory: one device block and one pinned host block (HandleBlocks).
  struct Arena {
    int device = -1;
    size_t device_bytes = 0, host_bytes = 0;
    char* d = nullptr;
    char* h = nullptr;
  };
  Arena mem;
  int32_t* d_out_ptr = nullptr;
  int32_t* d_out_col = nullptr;
  int32_t* d_in_ptr = nullptr;
  int32_t* d_in_col = nullptr;
  int32_t* d_in_link = nullptr;  // link id (position in the out-CSR) of every in-CSR entry
  // Slots of a2a_schedule_bound / _cap: kSlots x kSlotWords int64 of pinned host memory that the kernels write their
  // results to, scratch and an arrival counter on the device; every call takes the next slot, so calls on
  // different streams or threads do not share one.
  static constexpr unsigned kSlots = 64, kSlotWords = 8;
  int64_t* h_slots = nullptr;
  long long* d_scratch_slots = nullptr;  // [kSlots][kExtremaGroups][kExtremaWords]
  unsigned* d_arrived = nullptr;         // [kSlots], 0 between calls
  mutable std::atomic<unsigned> next_slot{0};
  // Topologies whose per-source state fits LDS (a2a_small_kernels.h): link tables of `ell_words` words per
  // node, 0 if there are none; which calls use them; smallest workspaces of the calls.
  uint32_t *d_ell_out = nullptr, *d_ell_in = nullptr;
  int ell_words = 0;
  bool small_loads = false, small_sigma = false, small_dist = false, wide_dist = false, wide_sigma = false;
  size_t min_loads_bytes = 0, min_sigma_bytes = 0, min_dist_bytes = 0;
  void* d_scratch = nullptr;    // device address of `scratch` on the handle's GPU
  // Whether all work that uses the handle is known to be over (then a2a_topo_destroy need not wait for the device,
  // 25 us): calls begun, calls now inside, the number begun when a call last waited for everything before it.
  struct Uses {
    std::atomic<uint64_t> begun{0}, inside{0}, settled{0};
    std::atomic<void*> stream{this};  // of the first call; before that no stream's handle
    std::atomic<bool> several{false};  // streams, or recorded in a graph: only the device knows
  };
  mutable Uses uses;
  // optional per-kernel timing (a2a_profile_enable); events are created per launch while it is on
  struct ProfRec {
    int cls, level;
    hipEvent_t beg, end;
  };
  mutable int prof_mode = 0;  // 0 off, 1 events, 2 events + shortest-path link count (level kernels)
  bool level_kernels_only() const { return prof_mode == 2; }
  mutable std::vector<ProfRec> prof_recs;
  mutable int64_t prof_pairs_level[A2A_PROF_MAX_LEVELS] = {};
  mutable int64_t prof_dag_level[A2A_PROF_MAX_LEVELS] = {};
  mutable int64_t prof_calls = 0;
  mutable int32_t prof_depth = 0;
  mutable int32_t prof_groups = 0;
  mutable uint64_t prof_narrow = 0;
  mutable uint64_t prof_fwd_flavours = 0, prof_bwd_flavours = 0;
};

namespace {

// A call that enqueues work with the handle.
class Use {
 public:
  Use(const a2a_topo* t, hipStream_t st) : u_(t->uses) {
    u_.inside.fetch_add(1);
    u_.begun.fetch_add(1);
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (st != nullptr && hipStreamIsCapturing(st, &capture) != hipSuccess) u_.several = true;
    void* first = &u_;
    const bool other = !u_.stream.compare_exchange_strong(first, st) && first != (void*)st;
    if (capture != hipStreamCaptureStatusNone || other || st == hipStreamPerThread) u_.several = true;
  }
  ~Use() { u_.inside.fetch_sub(1); }
  Use(const Use&) = delete;
  Use& operator=(const Use&) = delete;
  // Before a launch: what a wait for it will cover, 0 if that is not everything begun so far.
  uint64_t covered() const {
    const uint64_t n = u_.begun.load();
    return u_.inside.load() == 1 && !u_.several.load() ? n : 0;
  }
  void waited(uint64_t n) const {
    if (n != 0) u_.settled = n;
  }

 private:
  a2a_topo::Uses& u_;
};

// Blocks of destroyed handles, kept for the next ones: a program that evaluates one small topology after the other
// would spend most of its time in hipMalloc, hipHostMalloc and hipFree otherwise.  At most kKept blocks of at most
// kPooledBytes each are kept (an idle program holds 8 MiB of each kind of memory at the most); they are given back
// when an allocation fails.  A block comes here only when the device has finished all work that may use it.
class ArenaPool {
 public:
  using Arena = a2a_topo::Arena;
  static constexpr size_t kKept = 4, kGrain = 64u << 10;

  bool take(size_t device_bytes, size_t host_bytes, Arena* out) {
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return false;
    {
      std::lock_guard<std::mutex> lock(mutex_);
      for (size_t i = 0; i < kept_.size(); ++i)
        if (kept_[i].device == device && kept_[i].device_bytes >= device_bytes && kept_[i].host_bytes >= host_bytes) {
          *out = kept_[i];
          kept_.erase(kept_.begin() + (long)i);
          return true;
        }
    }
    Arena a;
    a.device = device;
    a.device_bytes = align_up_to(device_bytes);
    a.host_bytes = align_up_to(host_bytes);
    if (allocate(&a)) {
      *out = a;
      return true;
    }
    give_back();
    if (!allocate(&a)) return false;
    *out = a;
    return true;
  }

  // settled: no work that uses the block is left.
  void put(const Arena& a, bool settled) {
    if (a.d == nullptr && a.h == nullptr) return;
    int device = a.device;
    const bool other = hipGetDevice(&device) == hipSuccess && device != a.device;
    if (other) (void)hipSetDevice(a.device);
    const bool idle = settled || hipDeviceSynchronize() == hipSuccess;  // as hipFree would wait
    bool keep = idle && a.d != nullptr && a.h != nullptr && a.device_bytes <= kPooledBytes && a.host_bytes <= kPooledBytes;
    if (keep) {
      std::lock_guard<std::mutex> lock(mutex_);
      keep = kept_.size() < kKept;
      if (keep) {
        try {
          kept_.push_back(a);
        } catch (const std::bad_alloc&) {
          keep = false;
        }
      }
    }
    if (!keep) release(a);
    if (other) (void)hipSetDevice(device);
    (void)hipGetLastError();
  }

 private:
  static size_t align_up_to(size_t x) { return (x + kGrain - 1) / kGrain * kGrain; }
  static bool allocate(Arena* a) {
    if (hipMalloc((void**)&a->d, a->device_bytes) == hipSuccess) {
      if (hipHostMalloc((void**)&a->h, a->host_bytes, hipHostMallocDefault) == hipSuccess) return true;
      (void)hipFree(a->d);
    }
    (void)hipGetLastError();
    a->d = a->h = nullptr;
    return false;
  }
  static void release(const Arena& a) {
    if (a.d) (void)hipFree(a.d);
    if (a.h) (void)hipHostFree(a.h);
  }
  void give_back() {
    std::vector<Arena> all;
    {
      std::lock_guard<std::mutex> lock(mutex_);
      all.swap(kept_);
    }
    for (const Arena& a : all) release(a);
  }
  std::mutex mutex_;
  std::vector<Arena> kept_;
};

ArenaPool& arena_pool() {
  alignas(ArenaPool) static unsigned char place[sizeof(ArenaPool)];
  static ArenaPool* const pool = new (place) ArenaPool;  // never destroyed: the runtime may be gone by then
  return *pool;
}

enum {
  PROF_INIT = A2A_K_INIT, PROF_BFS = A2A_K_BFS, PROF_OFFSETS = A2A_K_OFFSETS, PROF_FWD = A2A_K_FWD_ROWS,
  PROF_FWD_FEW = A2A_K_FWD_FEW, PROF_FWD_SPREAD = A2A_K_FWD_SPREAD, PROF_BWD = A2A_K_BWD_ROWS,
  PROF_BWD_FEW = A2A_K_BWD_FEW, PROF_BWD_SPREAD = A2A_K_BWD_SPREAD, PROF_REDUCE = A2A_K_REDUCE, PROF_EXTRACT = A2A_K_EXTRACT,
  PROF_SEARCH = A2A_K_SEARCH, PROF_SOURCES = A2A_K_SOURCES,
  PROF_CLASSES = A2A_K_COUNT
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Workspace layout for G batches.  All arrays are 256-byte aligned.
struct Layout {
  int G = 0;     // batches per group
  int Lcap = 0;  // level slots per batch (levels 0 .. Lcap-1)
  int Npad = 0;  // N rounded up to a multiple of 256
  int bpb = 0;   // 256-node blocks per batch
  int nb64 = 0;  // 64-node blocks per batch
  int SB = 0;    // super-batches of kSub batches (BFS arrays)
  bool values = false, loads = false, sssp = false;
  size_t Epad = 0;
  size_t off_misc = 0;       // int64 [8]: 0 sigma-inexact flag, 1 dist_sum, 2 reached pairs, 3 DAG links
  size_t off_ltot = 0;       // int64 [G][Lcap]
  size_t off_dag = 0;        // int64 [G][Lcap]
  size_t off_bsum = 0;       // int32 [SB*kSub][Lcap][nb64]
  size_t off_seen = 0;       // uint64 [SB][Npad][kSub]
  size_t off_bm = 0;         // uint64 [SB][Lcap][Npad][kSub]
  size_t off_idxb = 0;       // NodeIdx [G][Lcap][Npad]        (with sigma / loads)
  size_t off_dat = 0;        // [G][Npad*64] x 8 bytes: sigma.  Entry e of a level kept in double precision is
                             // the e-th double, that of a level kept in single precision the e-th float of
                             // the same array: the single-precision levels come first, so the two never meet
  size_t off_coef = 0;       // double [G][Npad*64]  coef (link loads only)
  size_t off_part = 0;       // double [G][Epad]
  size_t off_wpart = 0;      // double [G][nb64]  demand x distance per (batch, 64-node block)
  size_t off_cost = 0;       // int64 [G][Npad][64]   single-path baseline: cost, chosen link, paths through
  size_t off_pick = 0;       // int32 [G][Npad][64]
  size_t off_sub = 0;        // int32 [G][Npad][64]
  size_t off_iload = 0;      // uint64 [Epad]
  size_t total = 0;
};

// recommend: size for all batches (or one, if minimal); otherwise fit as many batches as
// ws_bytes holds (G = 0: not even one).
Layout make_layout(const a2a_topo* t, int32_t src_count, int flags, size_t ws_bytes, bool recommend,
                   bool minimal) {
  Layout L;
  L.values = (flags & (A2A_WS_SIGMA | A2A_WS_LOADS)) != 0;
  L.loads = (flags & A2A_WS_LOADS) != 0;
  L.sssp = (flags & A2A_WS_SSSP) != 0;
  L.Npad = (int)align_up((size_t)t->N, kBlock);
  L.bpb = L.Npad / kBlock;
  L.nb64 = L.Npad / kBfsNodes;
  L.Lcap = t->level_bound + 2;
  L.Epad = align_up((size_t)(t->E > 0 ? t->E : 1), 32);
  const int nb = (src_count + 63) / 64;
  auto total_for = [&](int G, Layout* out) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
      const size_t at = off;
      off += align_up(bytes, 256);
      return at;
    };
    const size_t o_misc = take(64);
    const size_t SB = (size_t)(G + kSub - 1) / kSub;
    const size_t o_ltot = take(SB * kSub * L.Lcap * 8);
    const size_t o_dag = take((size_t)G * L.Lcap * 8);
    const size_t o_bsum = take(SB * kSub * L.Lcap * L.nb64 * 4);
    const size_t o_seen = take(SB * L.Npad * kSub * 8);
    const size_t o_bm = take(SB * L.Lcap * L.Npad * kSub * 8);
    const size_t o_idxb = L.values ? take((size_t)G * L.Lcap * L.Npad * sizeof(NodeIdx)) : 0;
    // + 256: rows are read in aligned 16-byte pairs, the last of which may reach one entry past the end
    const size_t o_dat = L.values ? take((size_t)G * L.Npad * 64 * 8 + 256) : 0;
    const size_t o_coef = L.loads ? take((size_t)G * L.Npad * 64 * 8 + 256) : 0;
    const size_t o_part = L.loads ? take((size_t)G * L.Epad * 8) : 0;
    const size_t o_wpart = L.loads ? take((size_t)G * L.nb64 * 8) : 0;
    const size_t o_cost = L.sssp ? take((size_t)G * L.Npad * 64 * 8) : 0;
    const size_t o_pick = L.sssp ? take((size_t)G * L.Npad * 64 * 4) : 0;
    const size_t o_sub = L.sssp ? take((size_t)G * L.Npad * 64 * 4) : 0;
    const size_t o_iload = L.sssp ? take(L.Epad * 8) : 0;
    if (out) {
      out->off_misc = o_misc;
      out->off_ltot = o_ltot;
      out->off_dag = o_dag;
      out->off_bsum = o_bsum;
      out->off_seen = o_seen;
      out->off_bm = o_bm;
      out->SB = (int)SB;
      out->off_idxb = o_idxb;
      out->off_dat = o_dat;
      out->off_coef = o_coef;
      out->off_part = o_part;
      out->off_wpart = o_wpart;
      out->off_cost = o_cost;
      out->off_pick = o_pick;
      out->off_sub = o_sub;
      out->off_iload = o_iload;
      out->total = off;
      out->G = G;
    }
    return off;
  };
  int G;
  if (recommend) {
    G = minimal ? 1 : nb;
  } else {
    if (total_for(1, nullptr) > ws_bytes) return L;  // G = 0
    int lo = 1, hi = nb;  // largest G that fits
    while (lo < hi) {
      const int mid = lo + (hi - lo + 1) / 2;
      if (total_for(mid, nullptr) <= ws_bytes)
        lo = mid;
      else
        hi = mid - 1;
    }
    G = lo;
  }
  total_for(G, &L);
  return L;
}

#define HIP_TRY(expr)           \
  do {                          \
    if ((expr) != hipSuccess) { \
      (void)hipGetLastError();  \
      return A2A_ERR_HIP;       \
    }                           \
  } while (0)

// Waits until done(), which looks at host memory that a kernel on the stream writes to at its end, or until the stream
// has finished.  The kernel's word is there before the runtime learns of the kernel's end: 5 to 8 us per wait.  Looks
// for about 100 us; what takes longer is left to the runtime, which does not keep the processor busy.
template <typename Done>
hipError_t wait_for(hipStream_t st, Done&& done) {
  const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(100);
  do {
    for (int k = 0; k < 64; ++k) {
      if (done()) return hipSuccess;
      __builtin_ia32_pause();
    }
  } while (std::chrono::steady_clock::now() < until);
  return hipStreamSynchronize(st);
}
template <typename T>
T seen(const T* p) {
  return __atomic_load_n(p, __ATOMIC_ACQUIRE);
}

// Zeroes `bytes` bytes (rounded up to a multiple of 8; every array it is used on has that room) at
// the 8-byte aligned device address p with a kernel on the stream.
inline hipError_t zero_async(void* p, size_t bytes, hipStream_t st) {
  const size_t n = (bytes + 7) / 8;
  if (n == 0) return hipSuccess;
  const size_t blocks = (n + kBlock - 1) / kBlock;
  k_zero<<<(unsigned)(blocks < 16384 ? blocks : 16384), kBlock, 0, st>>>((unsigned long long*)p, n);
  return hipGetLastError();
}

// Brackets one kernel launch with two events while profiling is on (t_ nullptr: not this one).
struct ProfScope {
  const a2a_topo* t;
  hipStream_t st;
  a2a_topo::ProfRec rec{};
  bool live = false;
  ProfScope(const a2a_topo* t_, int cls, hipStream_t st_, int level = 0) : t(t_), st(st_) {
    if (t == nullptr || t->prof_mode == 0) return;
    rec.cls = cls;
    rec.level = level;
    if (hipEventCreate(&rec.beg) != hipSuccess) return;
    if (hipEventCreate(&rec.end) != hipSuccess) {
      (void)hipEventDestroy(rec.beg);
      return;
    }
    live = hipEventRecord(rec.beg, st) == hipSuccess;
  }
  ~ProfScope() {
    if (!live) return;
    (void)hipEventRecord(rec.end, st);
    try {
      t->prof_recs.push_back(rec);
    } catch (const std::bad_alloc&) {  // the launch is missing from the profile
      (void)hipEventDestroy(rec.beg);
      (void)hipEventDestroy(rec.end);
    }
  }
};

inline unsigned grid_for(int G, int blocks_per_batch, int inflight = kXcd) {
  return (unsigned)((G + inflight - 1) / inflight * inflight * blocks_per_batch);
}

// Largest topology: a batch's value array (N * 64 entries of 8 bytes) is addressed with 32-bit
// byte offsets.
constexpr int32_t kMaxNodes = 4 * 1024 * 1024;

constexpr int32_t kPaddedRows = 4096;  // nodes above which the in-link table has whole slots of the wide search

// Nominal lane layout of a level for the profile's kernel classes (the kernels pick per batch,
// from the same rule applied to the batch's own counts).
constexpr double kNominalRows = 8.0;

struct Run {
  const a2a_topo* t;
  Layout L;
  char* ws;
  hipStream_t st;
  int src_begin, src_count;
  const double* demand = nullptr;  // [N][src_count] by target, or nullptr: every pair has demand 1
  int inflight = kXcd;  // batches in flight = XCDs: one batch's node blocks per XCD at a time
  int split = 1;        // waves per block of 64 nodes in the forward / backward kernels (pick_split)
  mutable bool indexed = false;  // run_index has written the group's index entries
  bool timed = true;             // its launches are part of the profile
  mutable std::vector<double> lanes_per_node;  // profiling only: per level of the current group, pairs / (G*N)
  bool few(int level) const {
    return level >= 0 && level < (int)lanes_per_node.size() && lanes_per_node[level] > 0.0 &&
           lanes_per_node[level] < kNominalRows;
  }
  // Path counts on `level` are at most (largest in-degree)^level: while that is below 2^24 the level
  // keeps sigma in single precision (exact: whole numbers a float holds), which halves what the
  // forward pass writes and gathers and what the backward pass reads of it.  If a level is narrow,
  // so are all before it.
  bool narrow(int level) const { return (double)level * std::log2((double)std::max(t->dmax_in, 2)) < 24.0; }
  int f32_levels() const {
    int n = 1;
    while (n < L.Lcap && narrow(n)) ++n;
    return n;
  }
  long long* misc() const { return (long long*)(ws + L.off_misc); }
  GroupView view(int batch0, int G) const {
    GroupView gv;
    gv.bm = (uint64_t*)(ws + L.off_bm);
    gv.idxb = L.values ? (NodeIdx*)(ws + L.off_idxb) : nullptr;
    gv.seen = (uint64_t*)(ws + L.off_seen);
    gv.dat = L.values ? (double*)(ws + L.off_dat) : nullptr;
    gv.datf = L.values ? (float*)(ws + L.off_dat) : nullptr;
    gv.coef = L.loads ? (double*)(ws + L.off_coef) : nullptr;
    gv.bsum = (int*)(ws + L.off_bsum);
    gv.ltot = (long long*)(ws + L.off_ltot);
    gv.dag = (long long*)(ws + L.off_dag);
    gv.part = L.loads ? (double*)(ws + L.off_part) : nullptr;
    gv.Epad = L.Epad;
    gv.N = t->N;
    gv.Npad = L.Npad;
    gv.Lcap = L.Lcap;
    gv.G = G;
    gv.SB = (G + kSub - 1) / kSub;
    gv.bpb = L.bpb;
    gv.nb64 = L.nb64;
    gv.inflight = inflight;
    gv.split = split;
    gv.src_begin = src_begin;
    gv.src_count = src_count;
    gv.batch0 = batch0;
    gv.f32_levels = f32_levels();
    gv.dem = demand;
    gv.dem_ld = src_count;
    gv.wpart = L.loads ? (double*)(ws + L.off_wpart) : nullptr;
    return gv;
  }
};

// A group that cannot fill the chip with one wave per 64 nodes lets 2, 4 or 8 waves share each block of
// 64 nodes (a tile of eight nodes is the unit): a wave's chain of dependent memory requests, which
// is what a launch of a small group costs, gets that much shorter.  Not with demands, not while
// shortest-path links are counted (see GroupView).  The line: us of link loads with sharing up to 0, 4096, 8192, 16384 and
// 32768 waves: 512 sources of 20011 nodes of degree 5 531, 531, 420, 419, 440; 512 of 16384 nodes of degree 4 497, 384, 380, 401,
// 401; 1000 of a 25x25x26 torus 1613, 1615, 1397, 1371, 1575.  (Where every level is dense a later line is better: 2501 of
// 4500 nodes of degree 10 637, 637, 570, 510, 489; and for a single source none at all: 65536 nodes 380, 457, 598, 597, 597.)
constexpr int kSplitWaves = 8192;
int pick_split(const a2a_topo* t, int G, int nb64, bool demand) {
  if (demand || t->prof_mode == 2) return 1;
  int split = 1;
  while (split < 8 && (long long)G * nb64 * split * 2 <= kSplitWaves) split *= 2;
  return split;
}

// While profiling is on: how full each level of a finished search is, by what it left in gv.ltot (this waits), and which
// lane layouts the level kernels pick for that.
int profile_group(const Run& r, const GroupView& gv) {
  const a2a_topo* t = r.t;
  const Layout& L = r.L;
  r.lanes_per_node.clear();
  if (t->prof_mode == 0) return A2A_OK;
  try {
    std::vector<long long> lt((size_t)gv.G * L.Lcap);
    HIP_TRY(hipMemcpyAsync(lt.data(), gv.ltot, lt.size() * 8, hipMemcpyDeviceToHost, r.st));
    HIP_TRY(hipStreamSynchronize(r.st));
    r.lanes_per_node.assign((size_t)L.Lcap, 0.0);
    int d = 0;
    for (int g = 0; g < gv.G; ++g)
      for (int k = 0; k < L.Lcap; ++k) {
        const long long n = lt[(size_t)g * L.Lcap + k];
        r.lanes_per_node[k] += (double)n;
        if (n > 0 && k > d) d = k;
      }
    for (int k = 0; k <= d; ++k)
      t->prof_pairs_level[k < A2A_PROF_MAX_LEVELS ? k : A2A_PROF_MAX_LEVELS - 1] += (int64_t)r.lanes_per_node[k];
    // which lane layout and precision each batch's kernels pick on each level (the kernels' own rule)
    for (int g = 0; g < gv.G; ++g)
      for (int k = 0; k + 1 < L.Lcap; ++k) {
        const long long* row = &lt[(size_t)g * L.Lcap];
        const long long here = row[k], after = row[k + 1], before = k > 0 ? row[k - 1] : 0;
        if (here == 0) continue;
        if (k >= 1 && L.values)
          t->prof_fwd_flavours |= 1ull << (3 * pick_flavour(here, before, t->N) + (r.narrow(k) ? 0 : (r.narrow(k - 1) ? 1 : 2)));
        if (L.loads && (r.demand != nullptr || after > 0))
          t->prof_bwd_flavours |= 1ull << (2 * pick_flavour(here, after, t->N) + (r.narrow(k) ? 0 : 1));
      }
    for (auto& x : r.lanes_per_node) x /= (double)gv.G * (double)t->N;
    if (d > t->prof_depth) t->prof_depth = d;
    t->prof_groups++;
  } catch (const std::bad_alloc&) {
    return A2A_ERR_NO_MEMORY;
  }
  return A2A_OK;
}

// BFS of one group: levels 1 .. top (the handle's deepest level, one more when the backward pass
// will look at the empty level after a batch's last one).
int run_bfs(const Run& r, const GroupView& gv, int top) {
  const a2a_topo* t = r.t;
  const Layout& L = r.L;
  HIP_TRY(zero_async(gv.ltot, (size_t)gv.SB * kSub * L.Lcap * 8, r.st));
  {
    ProfScope ps(r.timed ? t : nullptr, PROF_INIT, r.st);
    k_init_group<<<grid_for(gv.SB, L.nb64), kBfsBlock, 0, r.st>>>(gv);
  }
  for (int l = 1; l <= top; ++l) {
    ProfScope ps(r.timed ? t : nullptr, PROF_BFS, r.st, l);
    k_bfs_level<<<grid_for(gv.SB, L.nb64), kBfsBlock, 0, r.st>>>(t->d_in_ptr, t->d_in_col, gv, l);
  }
  HIP_TRY(hipGetLastError());
  return profile_group(r, gv);
}

// Row offsets, then sigma for levels 1 .. depth.
int run_fwd(const Run& r, const GroupView& gv, int depth) {
  const a2a_topo* t = r.t;
  const Layout& L = r.L;
  if (!r.indexed) {
    // With demands the backward pass also visits a batch's deepest level and looks at the (empty)
    // level after it, which the BFS has computed: its index entries are written too.
    const int idx_depth = gv.dem != nullptr ? depth + 1 : depth;
    ProfScope ps(t, PROF_OFFSETS, r.st);
    if (idx_depth >= 1) k_scan_blocks<<<(unsigned)(gv.G * idx_depth), kWave, 0, r.st>>>(gv, idx_depth);
    const int levels = offset_levels((long long)gv.SB * L.nb64, grid_for(gv.SB, L.nb64), kBfsBlock, idx_depth + 1);
    const int chunks = (idx_depth + levels) / levels;
    k_write_offsets<<<grid_for(gv.SB, L.nb64 * chunks), kBfsBlock, 0, r.st>>>(gv, idx_depth, levels);
  }
  const unsigned grid = grid_for(gv.G, L.bpb * gv.split, r.inflight);
  for (int l = 1; l <= depth; ++l) {
    const int cls = r.few(l) ? PROF_FWD_FEW : (r.few(l - 1) ? PROF_FWD_SPREAD : PROF_FWD);
    ProfScope ps(t, cls, r.st, l);
    const bool count = t->prof_mode == 2;
    auto launch = [&](auto kernel) {
      kernel<<<grid, kBlock, 0, r.st>>>(t->d_in_ptr, t->d_in_col, gv, l, r.misc());
    };
    // precision of the level gathered from and of the one written; waves sharing blocks of nodes or not
    const bool shared = gv.split > 1;  // never while counting
    if (r.narrow(l))
      count    ? launch(k_fwd<true, float, float>)
      : shared ? launch(k_fwd<false, float, float, true>)
               : launch(k_fwd<false, float, float>);
    else if (r.narrow(l - 1))
      count    ? launch(k_fwd<true, float, double>)
      : shared ? launch(k_fwd<false, float, double, true>)
               : launch(k_fwd<false, float, double>);
    else
      count    ? launch(k_fwd<true, double, double>)
      : shared ? launch(k_fwd<false, double, double, true>)
               : launch(k_fwd<false, double, double>);
    if (t->prof_mode != 0 && l < 64 && r.narrow(l - 1)) t->prof_narrow |= 1ull << l;
  }
  HIP_TRY(hipGetLastError());
  if (t->prof_mode == 2) {  // shortest-path links into each level, for the roofline accounting
    try {
      std::vector<long long> dg((size_t)gv.G * L.Lcap);
      HIP_TRY(hipMemcpyAsync(dg.data(), gv.dag, dg.size() * 8, hipMemcpyDeviceToHost, r.st));
      HIP_TRY(hipStreamSynchronize(r.st));
      for (int g = 0; g < gv.G; ++g)
        for (int l = 0; l <= depth; ++l)
          t->prof_dag_level[l < A2A_PROF_MAX_LEVELS ? l : A2A_PROF_MAX_LEVELS - 1] += dg[(size_t)g * L.Lcap + l];
    } catch (const std::bad_alloc&) {
      return A2A_ERR_NO_MEMORY;
    }
  }
  return A2A_OK;
}

// Level totals of the finished group go into the call's running totals.
int run_fold(const Run& r, const GroupView& gv, int depth) {
  k_fold_counters<<<1, kBlock, 0, r.st>>>(gv, depth, r.misc());
  HIP_TRY(hipGetLastError());
  return A2A_OK;
}

// While profiling is on: the levels of a call that other kernels have served, by a level search in its workspace, which
// is not timed.
int profile_levels(const a2a_topo* t, int32_t src_begin, int32_t src_count, const double* demand, int ws_flags, char* ws,
                   size_t ws_bytes, hipStream_t st) {
  if (t->prof_mode == 0) return A2A_OK;
  Run r;
  r.t = t;
  r.L = make_layout(t, src_count, ws_flags, ws_bytes, false, false);
  if (r.L.G < 1) return A2A_ERR_WORKSPACE_TOO_SMALL;
  r.ws = ws;
  r.st = st;
  r.src_begin = src_begin;
  r.src_count = src_count;
  r.demand = demand;
  r.timed = false;
  const int nb = (src_count + 63) / 64;
  for (int b0 = 0; b0 < nb; b0 += r.L.G) {
    const int rc = run_bfs(r, r.view(b0, std::min(nb - b0, r.L.G)), t->level_bound);
    if (rc != A2A_OK) return rc;
  }
  t->prof_calls++;
  return A2A_OK;
}

// Largest finite hop distance of the topology: the BFS from every node, 64 sources per mask, as
// many super-batches at a time as about 1 GiB of temporary device memory holds.  Runs on the
// default stream and waits (this is a2a_topo_create).  Topologies with link tables need one launch and leave the
// results in `deepest_of`, pinned host memory.
int probe_depth(const a2a_topo* t, int* deepest_of, int32_t* depth_out) {
  const int N = t->N;
  if (t->ell_words > 0 && N <= kScaledNodes) {
    const int groups = (N + kSmallBatch - 1) / kSmallBatch;
    const unsigned threads = (unsigned)std::min<size_t>(kSmallThreads, align_up((size_t)N, kWave));
    std::fill_n(deepest_of, groups, -1);
    k_small_probe<<<(unsigned)groups, threads, (size_t)N * 3 * sizeof(uint32_t), nullptr>>>(t->d_ell_out, t->ell_words, N,
                                                                                        deepest_of);
    HIP_TRY(hipGetLastError());
    HIP_TRY(wait_for(nullptr, [&, k = 0]() mutable {
      while (k < groups && seen(&deepest_of[k]) >= 0) ++k;
      return k == groups;
    }));
    *depth_out = *std::max_element(deepest_of, deepest_of + groups);
    return A2A_OK;
  }
  const int Npad = (int)align_up((size_t)N, kBlock);
  const int nb64 = Npad / kBfsNodes;
  const int sb_all = ((N + 63) / 64 + kSub - 1) / kSub;
  const size_t per_sb = (size_t)Npad * kSub * 8;  // one mask array of one super-batch
  const int sb_grp = (int)std::max<size_t>(1, std::min<size_t>((size_t)sb_all, ((size_t)1 << 30) / (3 * per_sb)));
  constexpr int kChunk = 16;  // levels between two looks at the "anything new" flags
  uint64_t* buf = nullptr;
  int* d_flags = nullptr;
  int h_flags[kChunk];
  int rc = A2A_OK, deepest = 0;
  if (hipMalloc((void**)&buf, 3 * per_sb * sb_grp) != hipSuccess ||
      hipMalloc((void**)&d_flags, kChunk * sizeof(int)) != hipSuccess) {
    (void)hipGetLastError();
    if (buf) (void)hipFree(buf);
    return A2A_ERR_HIP;
  }
  uint64_t* ring[2] = {buf, buf + per_sb / 8 * sb_grp};
  uint64_t* seen = buf + 2 * (per_sb / 8) * sb_grp;
  for (int sb0 = 0; sb0 < sb_all && rc == A2A_OK; sb0 += sb_grp) {
    const int SB = std::min(sb_grp, sb_all - sb0);
    k_probe_init<<<grid_for(SB, nb64), kBfsBlock, 0, nullptr>>>(ring[0], seen, N, Npad, SB, sb0 * kSub * 64);
    int level = 1;
    bool done = false;
    while (!done && rc == A2A_OK) {
      rc = zero_async(d_flags, sizeof(h_flags), nullptr) == hipSuccess ? A2A_OK : A2A_ERR_HIP;
      for (int k = 0; k < kChunk && rc == A2A_OK; ++k)
        k_probe_level<<<grid_for(SB, nb64), kBfsBlock, 0, nullptr>>>(t->d_in_ptr, t->d_in_col, ring[(level + k + 1) & 1],
                                                                   ring[(level + k) & 1], seen, N, Npad, SB, d_flags + k);
      if (rc == A2A_OK && (hipGetLastError() != hipSuccess ||
                           hipMemcpy(h_flags, d_flags, sizeof(h_flags), hipMemcpyDeviceToHost) != hipSuccess))
        rc = A2A_ERR_HIP;
      for (int k = 0; k < kChunk && rc == A2A_OK && !done; ++k) {
        if (h_flags[k] == 0)
          done = true;  // level + k reached nothing new: every later level is empty too
        else
          deepest = std::max(deepest, level + k);
      }
      level += kChunk;
      if (level > N) done = true;  // a shortest path has at most N - 1 links
    }
  }
  (void)hipFree(buf);
  (void)hipFree(d_flags);
  if (rc != A2A_OK) (void)hipGetLastError();
  *depth_out = deepest;
  return rc;
}

// --- topologies whose per-source state fits LDS ------------------------------------------------------

// Words per node of the link tables (two links a word) for a largest in- or out-degree, 0: no tables.
int ell_words_for(int32_t N, int32_t degree) {
  if (N > kWideMost || degree > 16 || degree < 1) return 0;
  for (int w : {2, 3, 4, 5})
    if (degree <= 2 * w) return w;
  return 8;
}

// Link table of a CSR: the neighbours of a node in list order, then the node itself.  `rows` >= N: rows past the last
// node are zero (the wide search reads whole slots).
std::vector<uint32_t> make_ell(int32_t N, const int32_t* ptr, const int32_t* col, int words, size_t rows) {
  std::vector<uint32_t> ell(rows * words);
  const uint32_t scale = N <= kScaledNodes ? 8 : 1;
  for (int32_t u = 0; u < N && words > 0; ++u) {
    const int32_t p0 = ptr[u], deg = ptr[u + 1] - p0;
    for (int k = 0; k < words; ++k) {
      const uint32_t a = (uint32_t)(2 * k < deg ? col[p0 + 2 * k] : u);
      const uint32_t b = (uint32_t)(2 * k + 1 < deg ? col[p0 + 2 * k + 1] : u);
      ell[(size_t)u * words + k] = scale * a | (scale * b << 16);
    }
  }
  return ell;
}

SmallPlan small_plan(const a2a_topo* t, int32_t src_count, SmallWhat what) {
  const SmallCut c = small_cut(t->N, t->level_bound, t->ell_words, src_count, what);
  SmallPlan p;
  p.T = c.threads;
  p.workgroups = c.workgroups;
  p.nodes = c.nodes;
  p.lds = c.lds;
  p.sv.out = t->d_ell_out;
  p.sv.in = t->d_ell_in;
  p.sv.N = t->N;
  p.sv.per = c.per;
  p.sv.tg = c.tg;
  p.sv.ts = c.ts;
  p.sv.per_wg = c.per_wg;
  p.sv.qshift = t->N <= kScaledNodes ? 3 : 0;
  p.sv.depth = t->level_bound;
  p.sv.src_count = src_count;
  return p;
}

// The same for link loads, with a thread per node where that is faster.
SmallPlan small_loads_plan(const a2a_topo* t, int32_t src_count, bool demand) {
  SmallPlan p = small_plan(t, src_count, SmallWhat::kLoads);
  const bool pairs = !demand && node_pairs(t->N, t->ell_words, t->level_bound, src_count);
  if (pairs || node_fits(t->N, t->ell_words, t->level_bound, src_count)) {
    const NodeCut c = node_cut(t->N, src_count);
    p.T = c.threads;
    p.nodes = c.nodes;
    p.workgroups = c.workgroups;
    p.at_a_time = pairs ? 2 : 1;
    p.lds = node_lds_bytes(t->N, c.nodes, p.at_a_time, t->ell_words);
    p.sv.per = 1;
    p.sv.per_wg = c.per_wg;
  }
  return p;
}

// Bytes of workspace per workgroup: its row of partial loads, its counters and level bytes.
size_t small_row_bytes(const a2a_topo* t, int per_wg) {
  return (size_t)t->N * t->ell_words * 2 * sizeof(double) + kSmallCounters * sizeof(long long) +
         (size_t)per_wg * small_level_bytes(t->N);
}

// Whether link loads take the one-workgroup-per-source kernel: everything fits, and so do the rows of one
// chunk of partial loads into the smallest workspace that a caller may bring.
bool small_loads_fit(const a2a_topo* t) {
  return t->ell_words > 0 && t->N <= kScaledNodes && t->level_bound < kSmallUnseen - 1 &&
         t->N <= small_max_nodes(t->ell_words) * kSmallThreads &&
         small_lds_bytes(t->N, 1, t->level_bound, kStateLoads) <= kSmallLds &&
         256 + kSmallChunk * small_row_bytes(t, kSmallBatch) <= t->min_loads_bytes;
}

// Workspace for all rows at once of a call over src_count sources or fewer.  (256 sources of 256 nodes of degree 8 have 4.2 MB of
// rows; 1.2 MB are what the level kernels take, and in those the rows went in four launches, and as many to add them up: 40.6 us,
// 13.0 in one.  256 sources of 1000 nodes 70.3, 23.6.)
size_t small_loads_bytes(const a2a_topo* t, int32_t src_count) {
  size_t most = 0;
  for (const bool demand : {false, true}) {
    const SmallPlan p = small_loads_plan(t, src_count, demand);
    const int rows = std::max(p.workgroups, std::min(src_count, kComputeUnits));
    most = std::max(most, 256 + (size_t)rows * small_row_bytes(t, p.sv.per_wg));
  }
  return most;
}

int small_link_loads(const a2a_topo* t, int32_t src_begin, int32_t src_count, const double* demand, double* load,
                     double* weighted_dist, int64_t* dist_sum_total, int64_t* flags, char* ws, size_t ws_bytes,
                     hipStream_t st) {
  if (ws_bytes < t->min_loads_bytes) return A2A_ERR_WORKSPACE_TOO_SMALL;
  SmallPlan p = small_loads_plan(t, src_count, demand != nullptr);
  const bool by_node = p.at_a_time > 0;
  p.sv.src_begin = src_begin;
  p.sv.dem = demand;
  p.sv.dem_ld = src_count;
  long long rows = (long long)((ws_bytes - 256) / small_row_bytes(t, p.sv.per_wg));  // at least kSmallChunk
  rows = rows >= p.workgroups ? p.workgroups : rows / kSmallChunk * kSmallChunk;
  p.sv.part = (double*)(ws + 256);
  p.sv.counters = (long long*)(p.sv.part + (size_t)rows * t->N * t->ell_words * 2);
  p.sv.level = (unsigned char*)(p.sv.counters + (size_t)rows * kSmallCounters);
  const SmallTotals tot{(long long)src_count * (t->N - 1), (long long*)dist_sum_total, nullptr,
                        (long long*)flags, weighted_dist};
  const unsigned blocks = (unsigned)((t->N * t->ell_words * 2 + 31) / 32 + 1);
  for (int w0 = 0; w0 < p.workgroups; w0 += (int)rows) {
    const int n = std::min(p.workgroups - w0, (int)rows);
    p.sv.wg0 = w0;
    {
      ProfScope ps(t, PROF_SOURCES, st);
      by_words(t->ell_words, [&](auto ks) { by_node ? launch_node_loads<decltype(ks)::value>(p, demand != nullptr, n, st)
                                                      : launch_small_loads<decltype(ks)::value>(p, demand != nullptr, n, st); });
    }
    ProfScope ps(t, PROF_REDUCE, st);
    k_small_reduce<<<blocks, kBlock, 0, st>>>(p.sv, t->ell_words, n, w0 == 0 ? 1 : 0, w0 + n == p.workgroups ? 1 : 0,
                                              t->d_out_ptr, load, (long long*)ws, tot);
  }
  HIP_TRY(hipGetLastError());
  return A2A_OK;
}

// Whether distances (and path counts) take the small kernels: their level bytes and counters fit the smallest
// workspace that a caller may bring, for one workgroup at least.
bool small_distances_fit(const a2a_topo* t, bool sigma) {
  return t->ell_words > 0 && t->N <= kScaledNodes && t->level_bound < kSmallUnseen - 1 &&
         small_lds_bytes(t->N, 1, t->level_bound, kStateSigma) <= kSmallLds &&
         256 + kSmallBatch * small_level_bytes(t->N) + kSmallCounters * sizeof(long long) <=
             (sigma ? t->min_sigma_bytes : t->min_dist_bytes);
}

int small_distances(const a2a_topo* t, int32_t src_begin, int32_t src_count, const SmallOut& out, int64_t* unreachable,
                    int64_t* flags, char* ws, size_t ws_bytes, hipStream_t st) {
  const bool sigma = out.sigma != nullptr;
  if (ws_bytes < (sigma ? t->min_sigma_bytes : t->min_dist_bytes)) return A2A_ERR_WORKSPACE_TOO_SMALL;
  SmallPlan p = small_plan(t, src_count, sigma ? SmallWhat::kSigma : SmallWhat::kDist);
  p.sv.src_begin = src_begin;
  const size_t row = kSmallCounters * sizeof(long long) + (sigma ? p.sv.per_wg * small_level_bytes(t->N) : 0);
  const int rows = (int)std::min<size_t>((size_t)p.workgroups, (ws_bytes - 256) / row);
  p.sv.counters = (long long*)(ws + 256);
  p.sv.level = (unsigned char*)(p.sv.counters + (size_t)rows * kSmallCounters);
  const SmallTotals tot{(long long)src_count * (t->N - 1), nullptr, (long long*)unreachable, (long long*)flags, nullptr};
  for (int w0 = 0; w0 < p.workgroups; w0 += rows) {
    const int n = std::min(p.workgroups - w0, rows);
    p.sv.wg0 = w0;
    {
      ProfScope ps(t, PROF_SOURCES, st);
      by_words(t->ell_words, [&](auto ks) { launch_small_outputs<decltype(ks)::value>(p, out, n, st); });
    }
    ProfScope ps(t, PROF_REDUCE, st);
    // a single workgroup: the counters only
    k_small_reduce<<<1, kBlock, 0, st>>>(p.sv, t->ell_words, n, w0 == 0 ? 1 : 0, w0 + n == p.workgroups ? 1 : 0,
                                         t->d_out_ptr, nullptr, (long long*)ws, tot);
  }
  HIP_TRY(hipGetLastError());
  return A2A_OK;
}

// Whether distances take the wide search: link table there, levels few enough.
bool wide_distances_fit(const a2a_topo* t) {
  return t->ell_words > 0 && t->N > kScaledNodes && t->level_bound < kWideDepth;
}
// Path counts with a source's state in LDS: 10 bytes a node have to fit, and a level per lane.
bool wide_sigma_fits(const a2a_topo* t) {
  return wide_distances_fit(t) && t->N <= kWideStateNodes && t->level_bound <= kWideStateDepth;
}

// The wide search over the sources of wv, its memory at `ws`, of which it may use ws_bytes (at least what the smallest
// workspace of a call leaves).  Sets *workgroups, each of which has counters at wv->counters.
int wide_search(const a2a_topo* t, WideView* wv, int out, char* ws, size_t ws_bytes, int* workgroups, hipStream_t st) {
  // sources per workgroup: as few as the fewest rounds over the chip allow (a level takes the same time)
  const int n = wv->src_count;
  int W = 16;
  const auto rounds = [&](int w) { return ((n + w - 1) / w + kComputeUnits - 1) / kComputeUnits; };
  for (int w = out == kWideBytes ? 64 : 32; w <= 64 && (size_t)t->N * w <= (size_t)kWideMost * 16; w *= 2)
    if (rounds(w) < rounds(W)) W = w;
  wv->in = t->d_ell_in;
  wv->N = t->N;
  wv->depth = t->level_bound;
  wv->slots = W == 16 ? (t->N + 2 * kWideThreads - 1) / (2 * kWideThreads) : (t->N + kWideThreads - 1) / kWideThreads * (W / 32);
  wv->out = t->d_ell_out;
  wv->list = wide_list(t->N, W);
  wv->together = wv->dist != nullptr && wide_together(t->N, n, W, t->level_bound);
  const size_t masks = (size_t)(wv->depth / 2 + 1) * wv->slots * kWideThreads * sizeof(uint32_t);
  const size_t room = ws_bytes / (masks + kSmallCounters * sizeof(long long));
  if (room < 1) return A2A_ERR_WORKSPACE_TOO_SMALL;
  *workgroups = (int)std::min<size_t>({(size_t)(n + W - 1) / W, (size_t)kComputeUnits, room});
  wv->masks = (uint32_t*)ws;
  wv->counters = (long long*)(ws + *workgroups * masks);
  ProfScope ps(t, PROF_SEARCH, st);
  by_words(t->ell_words, [&](auto ks) { launch_wide_search<decltype(ks)::value>(*wv, W, out, *workgroups, st); });
  return A2A_OK;
}

// Link loads by the level kernels: whether the levels of a group of G batches come from the wide search (link table
// there, whole slots of rows in it, masks of all levels fit the memory of the level search's).  Search and index entries
// before and after: 16384 nodes of degree 4 433 -> 223 us, 2501 sources of 20011 nodes 190 -> 103 us, 65536 nodes of
// degree 8 9.4 -> 5.9 ms; with many levels the whole call: torus 128x128 (128 levels) 34.8 -> 32.0 ms, 4x2000 (1002)
// 47.0 -> 40.6 ms, ring of 8000 (4000) 286 -> 233 ms, so there is no limit on them.  The table of up
// to 8191 nodes has 8 x id, which is the place of a 64-bit word.
int wide_masks_sources(const a2a_topo* t) { return t->N <= kBothTables ? 64 : 16; }  // a word
int wide_masks_slots(const a2a_topo* t) {
  return wide_masks_sources(t) == 16 ? (t->N + 2 * kWideThreads - 1) / (2 * kWideThreads)
                                     : (t->N + kWideThreads - 1) / kWideThreads * 2;
}
bool wide_masks_fit(const a2a_topo* t, const Layout& L, int G) {
  const size_t room = L.off_bm - L.off_seen + (size_t)L.SB * L.Lcap * L.Npad * kSub * 8;
  const size_t groups = (size_t)G * (64 / wide_masks_sources(t));
  return t->ell_words > 0 && t->N > kPaddedRows && t->level_bound >= 1 && !t->level_kernels_only() &&
         groups * t->level_bound * wide_masks_slots(t) * kWideThreads * sizeof(uint32_t) <= room;
}

// Search and index entries of a group, levels 0 .. top.
int run_index(const Run& r, const GroupView& gv, int top) {
  const a2a_topo* t = r.t;
  WideView wv{};
  wv.in = t->d_ell_in;
  wv.masks = (uint32_t*)(r.ws + r.L.off_seen);
  wv.N = t->N;
  wv.depth = t->level_bound;
  wv.src_begin = r.src_begin + gv.batch0 * 64;
  wv.src_count = std::min(gv.G * 64, r.src_count - gv.batch0 * 64);
  wv.slots = wide_masks_slots(t);
  wv.ltot = gv.ltot;
  wv.Lcap = gv.Lcap;
  HIP_TRY(zero_async(gv.ltot, (size_t)gv.SB * kSub * r.L.Lcap * 8, r.st));
  const int W = wide_masks_sources(t);
  const int workgroups = std::min((wv.src_count + W - 1) / W, kComputeUnits);
  {
    ProfScope ps(t, PROF_SEARCH, r.st);
    by_words(t->ell_words, [&](auto ks) { launch_wide_masks<decltype(ks)::value>(wv, W, workgroups, r.st); });
  }
  const unsigned blocks = (unsigned)(gv.G * (top + 1));  // 2^32 threads: the entries alone would take 290 GB
  {
    ProfScope ps(t, PROF_OFFSETS, r.st);
    W == 16 ? k_wide_index<16><<<blocks, kWideThreads, 0, r.st>>>(wv, gv) : k_wide_index<64><<<blocks, kWideThreads, 0, r.st>>>(wv, gv);
  }
  HIP_TRY(hipGetLastError());
  return profile_group(r, gv);
}

// The call's totals from the counters of its workgroups (see k_small_reduce); misc: 64 bytes for the running ones.
void wide_totals(const a2a_topo* t, long long* counters, int workgroups, bool first, bool last, const SmallTotals& tot,
                 long long* misc, hipStream_t st) {
  SmallView sv{};
  sv.N = t->N;
  sv.counters = counters;
  ProfScope ps(t, PROF_REDUCE, st);
  k_small_reduce<<<1, kBlock, 0, st>>>(sv, t->ell_words, workgroups, first ? 1 : 0, last ? 1 : 0, t->d_out_ptr, nullptr, misc, tot);
}

int wide_distances(const a2a_topo* t, int32_t src_begin, int32_t src_count, int32_t* dist, int64_t* dist_sum,
                   int64_t* unreachable, int64_t* flags, char* ws, size_t ws_bytes, hipStream_t st) {
  if (ws_bytes < t->min_dist_bytes) return A2A_ERR_WORKSPACE_TOO_SMALL;
  WideView wv{};
  wv.src_begin = src_begin;
  wv.src_count = src_count;
  wv.dist = dist;
  wv.sums = (long long*)dist_sum;
  int workgroups = 0;
  const int rc = wide_search(t, &wv, kWideDist, ws + 256, ws_bytes - 256, &workgroups, st);
  if (rc != A2A_OK) return rc;
  const SmallTotals tot{(long long)src_count * (t->N - 1), nullptr, (long long*)unreachable, (long long*)flags, nullptr};
  wide_totals(t, wv.counters, workgroups, true, true, tot, (long long*)ws, st);
  HIP_TRY(hipGetLastError());
  return A2A_OK;
}

int wide_sigma(const a2a_topo* t, int32_t src_begin, int32_t src_count, const SmallOut& out, int64_t* unreachable,
               int64_t* flags, char* ws, size_t ws_bytes, hipStream_t st) {
  if (ws_bytes < t->min_sigma_bytes) return A2A_ERR_WORKSPACE_TOO_SMALL;
  // a quarter of the workspace for level bytes, for all sources if they fit it
  const size_t level_bytes = small_level_bytes(t->N);
  const int chunk = (int)std::min<size_t>((size_t)src_count, std::max<size_t>(1, ws_bytes / 4 / level_bytes));
  unsigned char* const level = (unsigned char*)(ws + 256);
  char* const rest = ws + 256 + align_up(chunk * level_bytes, 256);
  long long* const counters = (long long*)rest;
  char* const search = rest + align_up(kComputeUnits * kSmallCounters * sizeof(long long), 256);
  const SmallTotals tot{(long long)src_count * (t->N - 1), nullptr, (long long*)unreachable, (long long*)flags, nullptr};
  for (int c0 = 0; c0 < src_count; c0 += chunk) {
    WideView wv{};
    wv.src_begin = src_begin + c0;
    wv.src_count = std::min(chunk, src_count - c0);
    wv.level = level;
    int groups = 0;
    const int rc = wide_search(t, &wv, kWideBytes, search, (size_t)(ws + ws_bytes - search), &groups, st);
    if (rc != A2A_OK) return rc;
    WideSigma wsig;
    wsig.in = t->d_ell_in;
    wsig.level = level;
    wsig.counters = counters;
    wsig.N = t->N;
    wsig.depth = t->level_bound;
    wsig.src_count = wv.src_count;
    const size_t row = (size_t)c0 * t->N;
    wsig.out = SmallOut{out.dist ? out.dist + row : nullptr, out.sigma + row, out.sums ? out.sums + c0 : nullptr};
    const int workgroups = std::min(wv.src_count, kComputeUnits);
    {
      ProfScope ps(t, PROF_SOURCES, st);
      by_words(t->ell_words, [&](auto ks) { launch_wide_sigma<decltype(ks)::value>(wsig, workgroups, st); });
    }
    wide_totals(t, counters, workgroups, c0 == 0, c0 + chunk >= src_count, tot, (long long*)ws, st);
  }
  HIP_TRY(hipGetLastError());
  return A2A_OK;
}

// Whether link loads of src_count sources go by sources in LDS and links in registers: path counts of all levels below 2^24 (a
// word holds a count and its level), LDS large enough, and for one source and group at least the smallest workspace that a caller may
// bring.  us of level kernels and of this, random topologies, all sources, 1024 and 256 of them: 8192 nodes of degree 5 1680, 760; 313,
// 162; 214, 177.  16384 of degree 4 6520, 2638; 590, 250; 396, 242.  20011 of degree 5 9944, 4165; 690, 309; 411, 290.  6000 of degree 8
// 954, 488; 242, 220; 163, 228.  It would win for fewer sources too (from 8192 nodes on) and with more levels (20011 of degree 3, 12
// levels, 10853, 4175): there the level kernels stay, whose results the tests hold bit for bit.
bool flow_fits(const a2a_topo* t, int32_t src_count, bool demand) {
  const double bits = (double)t->level_bound * std::log2((double)std::max(t->dmax_in, 2));  // as Run::narrow
  return t->ell_words > 0 && t->N <= kFlowNodes && !t->small_loads && src_count >= kFlowFewestSources && t->level_bound >= 1 &&
         t->level_bound <= kFlowDeepest && bits < 24.0 && flow_lds_fits(t->N, t->level_bound, demand) &&
         flow_layout_for(t->N, t->ell_words, src_count, demand, kSmallBatch, 1).total <= t->min_loads_bytes;
}

// The same for unit demands of topologies of more nodes, by strips (k_strip_sources): path counts of all levels below 2^32.  ms of
// level kernels and of this, all sources and 2048 of them: random topologies, 20353 nodes of degree 6 9.49, 6.68; 1.09, 0.74; 30000 of degree 4
// 20.7, 12.4; 1.60, 0.99; 45000 of degree 3 (13 levels) 59.6, 34.4; 3.02, 1.84; 65536 of degree 8 106.3, 75.2; 3.58, 2.64; 24000 of degree 16 2048
// sources 2.41, 1.25; generalized Kautz topologies, 40000 of degree 5 24.6, 18.8; 1.42, 1.04; 65535 of degree 3 76.5, 61.6; 60000 of degree 8
// 64.8, 57.4.  With demands it was not the faster one everywhere (16384 nodes of degree 4 5.23, 5.82; 32768 of degree 3 33.2, 28.8).  Fewer
// sources stay with the level kernels, whose results the tests hold bit for bit.
bool strips_fit(const a2a_topo* t, int32_t src_count) {
  const double bits = (double)t->level_bound * std::log2((double)std::max(t->dmax_in, 2));
  return t->ell_words > 0 && t->N > kFlowNodes && src_count >= kStripFewestSources && t->level_bound >= 1 && bits < 32.0 &&
         strip_lds_fits(t->N, t->level_bound) &&
         flow_layout_for(t->N, t->ell_words, src_count, false, kSmallBatch, 1, true).total <= t->min_loads_bytes;
}

int flow_link_loads(const a2a_topo* t, bool strips, int32_t src_begin, int32_t src_count, const double* demand, double* load,
                    double* weighted_dist, int64_t* dist_sum_total, int64_t* flags, char* ws, size_t ws_bytes, hipStream_t st) {
  if (ws_bytes < t->min_loads_bytes) return A2A_ERR_WORKSPACE_TOO_SMALL;
  const FlowGroups g = flow_groups(t->N, t->ell_words, src_count, strips);
  const FlowLayout l = flow_layout(t->N, t->ell_words, src_count, demand != nullptr, ws_bytes, strips);
  FlowView fv{};
  fv.in = t->d_ell_in;
  fv.out = t->d_ell_out;
  fv.level = (unsigned char*)(ws + l.level);
  fv.record = ws + l.record;
  fv.count = (uint32_t*)(ws + l.count);
  fv.exact = strips ? (uint32_t*)(ws + l.exact) : nullptr;
  fv.escaped = (int*)(ws + l.escaped);
  fv.coef = (double*)(ws + l.coef);
  fv.counters = (long long*)(ws + l.counters);
  fv.part = (double*)(ws + l.part);
  fv.N = t->N;
  fv.stride = flow_stride(t->N);
  fv.depth = t->level_bound;
  fv.group = g.group;
  const int places = 2 * t->ell_words;
  const SmallTotals tot{(long long)src_count * (t->N - 1), (long long*)dist_sum_total, nullptr, (long long*)flags, nullptr};
  // pieces of whole groups, or one group in several
  const bool whole = l.parts > 1 || l.rows >= g.group;
  int piece = 0;
  bool added = false;
  for (int s0 = 0; s0 < src_count; s0 += piece) {
    const int left = whole ? src_count - s0 : std::min(src_count, (s0 / g.group + 1) * g.group) - s0;  // of the call, or the group
    piece = std::min(l.rows, left);
    fv.source0 = src_begin + s0;
    fv.sources = piece;
    fv.groups = (piece + g.group - 1) / g.group;
    fv.resume = !whole && s0 % g.group != 0;
    fv.weighted = (double*)(ws + l.weighted) + s0;
    if (t->N <= kScaledNodes) {
      SmallPlan lp = small_plan(t, piece, SmallWhat::kSssp);
      lp.sv.src_begin = fv.source0;
      lp.sv.per_wg = kSmallBatch;
      lp.sv.level = (unsigned char*)(ws + l.level);
      ProfScope ps(t, PROF_SEARCH, st);
      by_words(t->ell_words, [&](auto ks) { launch_small_levels<decltype(ks)::value>(lp, (piece + kSmallBatch - 1) / kSmallBatch, st); });
    } else {
      WideView wv{};
      wv.src_begin = fv.source0;
      wv.src_count = piece;
      wv.level = (unsigned char*)(ws + l.level);
      int groups = 0;
      const int rc = wide_search(t, &wv, kWideBytes, ws + l.coef, l.total - l.coef, &groups, st);
      if (rc != A2A_OK) return rc;
    }
    const int workgroups = std::min(piece, kComputeUnits);
    {
      ProfScope ps(t, PROF_SOURCES, st);
      if (demand) {
        const unsigned tiles = (unsigned)((t->N + kWave - 1) / kWave) * (unsigned)((piece + kWave - 1) / kWave);
        k_flow_demand<<<tiles, kBlock, 0, st>>>(fv, demand + s0, src_count);
      }
      by_words(t->ell_words, [&](auto ks) {
        strips ? launch_strip_sources<decltype(ks)::value>(fv, workgroups, st)
               : launch_flow_sources<decltype(ks)::value>(fv, demand != nullptr, workgroups, st);
      });
      by_words(t->ell_words, [&](auto ks) { launch_flow_links<decltype(ks)::value>(fv, demand != nullptr, st); });
    }
    const bool last = s0 + piece == src_count;
    if (whole || last || (s0 + piece) % g.group == 0) {
      ProfScope ps(t, PROF_REDUCE, st);
      k_flow_reduce<<<(unsigned)(((size_t)t->N * places + kBlock - 1) / kBlock), kBlock, 0, st>>>(
          fv.part, fv.groups, places, t->N, added ? 0 : 1, t->d_in_ptr, t->d_in_link, load);
      added = true;
    }
    wide_totals(t, fv.counters, workgroups, s0 == 0, last, tot, (long long*)ws, st);
  }
  if (weighted_dist) {
    if (demand)
      k_flow_weighted<<<1, kWideThreads, 0, st>>>((double*)(ws + l.weighted), src_count, weighted_dist);
    else
      HIP_TRY(zero_async(weighted_dist, 8, st));
  }
  HIP_TRY(hipGetLastError());
  return A2A_OK;
}

// Whether a call of the single-path baseline takes the small kernels: its state for one source fits LDS, levels fit a
// byte (and, with more than 8191 nodes, the search's four bit planes), and costs fit 32 bits.
bool small_sssp_fits(const a2a_topo* t, int32_t src_count) {
  return t->ell_words > 0 && t->N <= kBothTables && t->level_bound < (t->N <= kScaledNodes ? kSmallUnseen - 1 : 16) &&
         small_lds_bytes(t->N, 1, t->level_bound, kStateSssp) <= kSmallLds &&
         sssp_costs_fit(t->level_bound, src_count, t->N);
}

// ws: at least what a2a_workspace_bytes says for the iteration (with dense rows of 1 KB per batch and node, far
// more than one iteration takes here).
int small_sssp(const a2a_topo* t, int32_t src_begin, int32_t src_count, int32_t per_iter, double* load,
               int64_t* dist_sum_total, int64_t* flags, char* ws, size_t ws_bytes, hipStream_t st) {
  const int places = 2 * t->ell_words;
  const int iterations = (src_count + per_iter - 1) / per_iter;
  const SmallPlan whole = small_plan(t, std::min(per_iter, src_count), SmallWhat::kSssp);
  const bool flow = flow_sssp_fits(t->N, t->level_bound, src_count);
  size_t off = 256;
  const auto part = [&off](size_t bytes) {
    const size_t at = off;
    off += align_up(bytes, 256);
    return at;
  };
  SmallSssp ss;
  ss.weight = (uint32_t*)(ws + part((size_t)t->N * places * 4));
  ss.handed = (uint32_t*)(ws + part((size_t)per_iter * t->N * 4));
  long long* const counters = (long long*)(ws + part((size_t)src_count * kSmallCounters * 8));  // at most one workgroup per source
  unsigned char* const level = (unsigned char*)(ws + off);
  // iterations whose levels fit what is left
  const size_t level_bytes = small_level_bytes(t->N);
  const long long room = off < ws_bytes ? (long long)((ws_bytes - off) / (level_bytes * per_iter)) : 0;
  if (room < 1) return A2A_ERR_WORKSPACE_TOO_SMALL;
  HIP_TRY(zero_async(ss.weight, (size_t)t->N * places * 4, st));
  int rows = 0;
  for (int i0 = 0; i0 < iterations; i0 += (int)room) {
    const int i1 = (int)std::min<long long>(iterations, i0 + room);
    SmallPlan lp = whole;
    lp.sv.src_begin = src_begin + i0 * per_iter;
    lp.sv.src_count = std::min(src_count, i1 * per_iter) - i0 * per_iter;
    lp.sv.per_wg = kSmallBatch;
    lp.sv.level = level;
    const int groups = (lp.sv.src_count + kSmallBatch - 1) / kSmallBatch;
    {
      ProfScope ps(t, PROF_SEARCH, st);
      by_words(t->ell_words, [&](auto ks) { launch_small_levels<decltype(ks)::value>(lp, groups, st); });
    }
    for (int i = i0; i < i1; ++i) {
      SmallPlan p = small_plan(t, std::min(per_iter, src_count - i * per_iter), SmallWhat::kSssp);
      p.sv.src_begin = src_begin + i * per_iter;
      p.sv.level = level + (size_t)(i - i0) * per_iter * level_bytes;
      p.sv.counters = counters + (size_t)rows * kSmallCounters;
      const int workgroups = flow ? std::min(p.sv.src_count, kComputeUnits) : p.workgroups;
      rows += workgroups;
      {
        ProfScope ps(t, PROF_SOURCES, st);
        by_words(t->ell_words, [&](auto ks) {
          constexpr int KS = decltype(ks)::value;
          flow ? launch_flow_sssp<KS>(p, ss, workgroups, st) : launch_small_sssp<KS>(p, ss, st);
        });
      }
      ProfScope ps(t, PROF_REDUCE, st);
      by_words(t->ell_words, [&](auto ks) { launch_small_sssp_add<decltype(ks)::value>(p, ss, st); });
    }
  }
  k_small_sssp_output<<<(unsigned)(((size_t)t->N * places + kBlock - 1) / kBlock), kBlock, 0, st>>>(
      ss.weight, places, t->d_in_ptr, t->d_in_link, t->N, load);
  SmallView sv = whole.sv;
  sv.counters = counters;
  const SmallTotals tot{(long long)src_count * (t->N - 1), (long long*)dist_sum_total, nullptr, (long long*)flags, nullptr};
  k_small_reduce<<<1, kBlock, 0, st>>>(sv, t->ell_words, rows, 1, 1, t->d_out_ptr, nullptr, (long long*)ws, tot);
  HIP_TRY(hipGetLastError());
  return A2A_OK;
}

int check_common(const a2a_topo* t, int32_t src_begin, int32_t src_count, void* ws) {
  if (!t || src_begin < 0 || src_count < 0 || (int64_t)src_begin + src_count > t->N) return A2A_ERR_INVALID_ARG;
  if (src_count > 0 && (!ws || ((uintptr_t)ws & 255u))) return A2A_ERR_INVALID_ARG;
  return A2A_OK;
}

}  // namespace

extern "C" {

const char* a2a_status_string(int status) {
  switch (status) {
    case A2A_OK: return "ok";
    case A2A_ERR_INVALID_ARG: return "invalid argument";
    case A2A_ERR_SELF_LOOP: return "self-loop in topology";
    case A2A_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
    case A2A_ERR_HIP: return "HIP runtime error";
    case A2A_ERR_NOT_IMPLEMENTED: return "not implemented";
    case A2A_ERR_DISCONNECTED: return "topology is not strongly connected";
    case A2A_ERR_NO_MEMORY: return "out of host memory";
    case A2A_ERR_LEVEL_OVERFLOW: return "BFS exceeded the level bound";
    default: return "unknown status";
  }
}

int a2a_topo_create(int32_t N, const int32_t* row_ptr, const int32_t* col_idx, a2a_topo** out) {
  if (!out) return A2A_ERR_INVALID_ARG;
  *out = nullptr;
  if (N <= 0 || !row_ptr || row_ptr[0] != 0) return A2A_ERR_INVALID_ARG;
  if (N > kMaxNodes) return A2A_ERR_NOT_IMPLEMENTED;
  int32_t dmax = 0;
  for (int32_t u = 0; u < N; ++u) {
    if (row_ptr[u + 1] < row_ptr[u]) return A2A_ERR_INVALID_ARG;
    if (row_ptr[u + 1] - row_ptr[u] > dmax) dmax = row_ptr[u + 1] - row_ptr[u];
  }
  const int64_t E = row_ptr[N];
  if (E > 0 && !col_idx) return A2A_ERR_INVALID_ARG;
  for (int32_t u = 0; u < N; ++u)
    for (int32_t p = row_ptr[u]; p < row_ptr[u + 1]; ++p) {
      if (col_idx[p] < 0 || col_idx[p] >= N) return A2A_ERR_INVALID_ARG;
      if (col_idx[p] == u) return A2A_ERR_SELF_LOOP;
    }
  a2a_topo* t = new (std::nothrow) a2a_topo();
  if (!t) return A2A_ERR_NO_MEMORY;
  std::vector<int32_t> in_ptr, in_col, in_link;
  std::vector<uint32_t> ell_out, ell_in;  // link tables of small topologies, see SmallView
  try {
    in_ptr.assign((size_t)N + 1, 0);
    in_col.resize((size_t)(E > 0 ? E : 1));
    in_link.resize((size_t)(E > 0 ? E : 1));
    for (int64_t p = 0; p < E; ++p) in_ptr[(size_t)col_idx[p] + 1]++;
    for (int32_t v = 0; v < N; ++v) in_ptr[(size_t)v + 1] += in_ptr[v];
    std::vector<int32_t> fill(in_ptr.begin(), in_ptr.end() - 1);
    for (int32_t u = 0; u < N; ++u)  // ascending link id => in-lists are stable in link order
      for (int32_t p = row_ptr[u]; p < row_ptr[u + 1]; ++p) {
        const size_t at = (size_t)fill[col_idx[p]]++;
        in_col[at] = u;
        in_link[at] = p;
      }
    for (int32_t v = 0; v < N; ++v) t->dmax_in = std::max(t->dmax_in, in_ptr[(size_t)v + 1] - in_ptr[v]);
    t->ell_words = ell_words_for(N, std::max(dmax, t->dmax_in));
    ell_out = make_ell(N, row_ptr, col_idx, t->ell_words, N);
    ell_in = make_ell(N, in_ptr.data(), in_col.data(), t->ell_words,
                      N <= kPaddedRows ? N : align_up((size_t)N, 2 * kWideThreads));
  } catch (const std::bad_alloc&) {
    delete t;
    return A2A_ERR_NO_MEMORY;
  }
  t->N = N;
  t->E = E;
  t->dmax = dmax;
  const HandleBlocks m = handle_blocks(N, E, ell_out.size() * sizeof(uint32_t), ell_in.size() * sizeof(uint32_t),
                                       a2a_topo::kSlots * sizeof(unsigned),
                                       (size_t)a2a_topo::kSlots * kExtremaGroups * kExtremaWords * sizeof(long long),
                                       (size_t)a2a_topo::kSlots * a2a_topo::kSlotWords * sizeof(int64_t),
                                       (size_t)((std::min(N, kScaledNodes) + kSmallBatch - 1) / kSmallBatch) * sizeof(int));
  bool ok = arena_pool().take(m.device, m.host, &t->mem);
  ok = ok && hipGetSymbolAddress(&t->d_scratch, HIP_SYMBOL(scratch)) == hipSuccess && t->d_scratch != nullptr;
  if (ok) {
    char *const d = t->mem.d, *const h = t->mem.h;
    t->d_out_ptr = (int32_t*)(d + m.at[kOutPtr]);
    t->d_out_col = (int32_t*)(d + m.at[kOutCol]);
    t->d_in_ptr = (int32_t*)(d + m.at[kInPtr]);
    t->d_in_col = (int32_t*)(d + m.at[kInCol]);
    t->d_in_link = (int32_t*)(d + m.at[kInLink]);
    t->d_ell_out = (uint32_t*)(d + m.at[kEllOut]);
    t->d_ell_in = (uint32_t*)(d + m.at[kEllIn]);
    t->d_arrived = (unsigned*)(d + m.at[kArrived]);
    t->d_scratch_slots = (long long*)(d + m.scratch);
    t->h_slots = (int64_t*)(h + m.slots);
    const unsigned arrived[a2a_topo::kSlots] = {};
    const void* const from[kHandleParts] = {row_ptr, E > 0 ? col_idx : in_col.data(), in_ptr.data(), in_col.data(),
                                            in_link.data(), ell_out.data(), ell_in.data(), arrived};
    for (int i = 0; i < kHandleParts && ok; ++i) {
      if (m.bytes[i] == 0) continue;
      if (m.staged)
        std::memcpy(h + m.at[i], from[i], m.bytes[i]);
      else
        ok = hipMemcpy(d + m.at[i], from[i], m.bytes[i], hipMemcpyHostToDevice) == hipSuccess;
    }
    if (ok && m.staged) ok = hipMemcpyAsync(d, h, m.upload, hipMemcpyHostToDevice, nullptr) == hipSuccess;
  }
  // the probe runs after the upload and is waited for
  if (ok) ok = E > 0 ? probe_depth(t, (int*)(t->mem.h + m.probe), &t->level_bound) == A2A_OK : hipStreamSynchronize(nullptr) == hipSuccess;
  if (ok) {
    t->min_loads_bytes = make_layout(t, 64, A2A_WS_LOADS, 0, true, true).total;
    t->min_sigma_bytes = make_layout(t, 64, A2A_WS_SIGMA, 0, true, true).total;
    t->min_dist_bytes = make_layout(t, 64, A2A_WS_DISTANCES, 0, true, true).total;
    t->small_loads = small_loads_fit(t);
    t->small_sigma = small_distances_fit(t, true);
    t->small_dist = small_distances_fit(t, false);
    t->wide_dist = wide_distances_fit(t);
    t->wide_sigma = wide_sigma_fits(t);
  }
  if (!ok) {
    (void)hipGetLastError();
    t->uses.several = true;  // whatever got as far as the device
    a2a_topo_destroy(t);
    return A2A_ERR_HIP;
  }
  *out = t;
  return A2A_OK;
}

void a2a_topo_destroy(a2a_topo* t) {
  if (!t) return;
  for (auto& rec : t->prof_recs) {
    (void)hipEventDestroy(rec.beg);
    (void)hipEventDestroy(rec.end);
  }
  arena_pool().put(t->mem, t->uses.several.load() ? false : t->uses.begun.load() == t->uses.settled.load());
  delete t;
}

int a2a_topo_info(const a2a_topo* t, int32_t* N, int64_t* E, int32_t* dmax, int32_t* level_bound) {
  if (!t) return A2A_ERR_INVALID_ARG;
  if (N) *N = t->N;
  if (E) *E = t->E;
  if (dmax) *dmax = t->dmax;
  if (level_bound) *level_bound = t->level_bound;
  return A2A_OK;
}

size_t a2a_workspace_bytes(const a2a_topo* t, int32_t src_count, int flags) {
  if (!t || src_count < 0 || (size_t)src_count > align_up((size_t)t->N, 64)) return 0;
  if (src_count == 0) return 256;
  const bool minimal = (flags & A2A_WS_MINIMAL) != 0;
  const Layout L = make_layout(t, src_count, flags & 0xff, 0, true, minimal);
  return minimal || !(flags & A2A_WS_LOADS) || !t->small_loads ? L.total : std::max(L.total, small_loads_bytes(t, src_count));
}

int a2a_distances(const a2a_topo* t, int32_t src_begin, int32_t src_count, int32_t* dist, double* sigma,
                  int64_t* dist_sum, int64_t* unreachable, int64_t* flags, void* workspace,
                  size_t workspace_bytes, void* hip_stream) {
  int rc = check_common(t, src_begin, src_count, workspace);
  if (rc != A2A_OK) return rc;
  hipStream_t st = (hipStream_t)hip_stream;
  const Use use(t, st);
  if (src_count == 0) {
    if (unreachable) HIP_TRY(zero_async(unreachable, 8, st));
    if (flags) HIP_TRY(zero_async(flags, 8, st));
    return A2A_OK;
  }
  const bool small = sigma ? t->small_sigma : t->small_dist;
  if ((small || (sigma ? t->wide_sigma : t->wide_dist)) && !t->level_kernels_only()) {
    const SmallOut out{dist, sigma, (long long*)dist_sum};
    char* const ws = (char*)workspace;
    if (small)
      rc = small_distances(t, src_begin, src_count, out, unreachable, flags, ws, workspace_bytes, st);
    else if (sigma)
      rc = wide_sigma(t, src_begin, src_count, out, unreachable, flags, ws, workspace_bytes, st);
    else
      rc = wide_distances(t, src_begin, src_count, dist, dist_sum, unreachable, flags, ws, workspace_bytes, st);
    if (rc != A2A_OK) return rc;
    return profile_levels(t, src_begin, src_count, nullptr, sigma ? A2A_WS_SIGMA : A2A_WS_DISTANCES, ws, workspace_bytes, st);
  }
  Run r;
  r.t = t;
  r.L = make_layout(t, src_count, sigma ? A2A_WS_SIGMA : A2A_WS_DISTANCES, workspace_bytes, false, false);
  if (r.L.G < 1) return A2A_ERR_WORKSPACE_TOO_SMALL;
  r.ws = (char*)workspace;
  r.st = st;
  r.src_begin = src_begin;
  r.src_count = src_count;
  const Layout& L = r.L;
  HIP_TRY(zero_async(r.misc(), 64, st));
  if (dist_sum) HIP_TRY(zero_async(dist_sum, (size_t)src_count * 8, st));
  const int nb = (src_count + 63) / 64;
  const int tiles = L.Npad / kWave;
  for (int b0 = 0; b0 < nb; b0 += L.G) {
    r.split = pick_split(t, nb - b0 < L.G ? nb - b0 : L.G, L.nb64, false);
    const GroupView gv = r.view(b0, nb - b0 < L.G ? nb - b0 : L.G);
    const int depth = t->level_bound;
    rc = run_bfs(r, gv, depth);
    if (rc != A2A_OK) return rc;
    if (sigma) {
      rc = run_fwd(r, gv, depth);
      if (rc != A2A_OK) return rc;
      ProfScope ps(t, PROF_EXTRACT, st);
      k_extract_sigma<<<grid_for(gv.G, tiles), kWave, 0, st>>>(gv, tiles, depth, sigma);
    }
    if (dist || dist_sum) {
      ProfScope ps(t, PROF_EXTRACT, st);
      if (depth < 128) {  // eight sources at a time, the number of bit planes fixed at compile time
        const unsigned grid = grid_for(gv.SB, L.bpb * kSub);
        auto launch = [&](auto kernel) { kernel<<<grid, kBlock, 0, st>>>(gv, depth, dist, (long long*)dist_sum); };
        if (depth < 8)
          dist_sum ? launch(k_extract_dist_packed<3, true>) : launch(k_extract_dist_packed<3, false>);
        else if (depth < 32)
          dist_sum ? launch(k_extract_dist_packed<5, true>) : launch(k_extract_dist_packed<5, false>);
        else
          dist_sum ? launch(k_extract_dist_packed<7, true>) : launch(k_extract_dist_packed<7, false>);
      } else if (depth < 256) {
        int planes = 0;
        while ((depth >> planes) != 0) ++planes;
        k_extract_dist_planes<<<grid_for(gv.SB, L.bpb * kSub), kBlock, 0, st>>>(gv, depth, planes, dist,
                                                                                (long long*)dist_sum);
      } else {
        k_extract_dist<<<grid_for(gv.G, tiles), kWave, 0, st>>>(gv, tiles, depth, dist, (long long*)dist_sum);
      }
    }
    rc = run_fold(r, gv, depth);
    if (rc != A2A_OK) return rc;
  }
  k_finish<<<1, 64, 0, st>>>(r.misc(), (long long)src_count * (t->N - 1), nullptr, (long long*)unreachable,
                             (long long*)flags);
  HIP_TRY(hipGetLastError());
  if (t->prof_mode) t->prof_calls++;
  return A2A_OK;
}

namespace {

// a2a_link_loads (demand == nullptr) and a2a_link_loads_demand.
int link_loads(const a2a_topo* t, int32_t src_begin, int32_t src_count, const double* demand, double* load,
               double* weighted_dist, int64_t* dist_sum_total, int64_t* flags, void* workspace,
               size_t workspace_bytes, void* hip_stream) {
  int rc = check_common(t, src_begin, src_count, workspace);
  if (rc != A2A_OK) return rc;
  if (!load && t->E > 0) return A2A_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  const Use use(t, st);
  if (t->small_loads && src_count > 0 && !t->level_kernels_only()) {
    rc = small_link_loads(t, src_begin, src_count, demand, load, weighted_dist, dist_sum_total, flags, (char*)workspace,
                          workspace_bytes, st);
    if (rc != A2A_OK) return rc;
    return profile_levels(t, src_begin, src_count, demand, A2A_WS_LOADS, (char*)workspace, workspace_bytes, st);
  }
  const bool whole = flow_fits(t, src_count, demand != nullptr);
  if ((whole || (demand == nullptr && strips_fit(t, src_count))) && !t->level_kernels_only()) {
    rc = flow_link_loads(t, !whole, src_begin, src_count, demand, load, weighted_dist, dist_sum_total, flags, (char*)workspace,
                         workspace_bytes, st);
    if (rc != A2A_OK) return rc;
    return profile_levels(t, src_begin, src_count, demand, A2A_WS_LOADS, (char*)workspace, workspace_bytes, st);
  }
  if (weighted_dist) HIP_TRY(zero_async(weighted_dist, 8, st));
  if (src_count == 0) {
    if (t->E > 0) HIP_TRY(zero_async(load, (size_t)t->E * 8, st));
    if (dist_sum_total) HIP_TRY(zero_async(dist_sum_total, 8, st));
    if (flags) HIP_TRY(zero_async(flags, 8, st));
    return A2A_OK;
  }
  Run r;
  r.t = t;
  r.L = make_layout(t, src_count, A2A_WS_LOADS, workspace_bytes, false, false);
  if (r.L.G < 1) return A2A_ERR_WORKSPACE_TOO_SMALL;
  r.ws = (char*)workspace;
  r.st = st;
  r.src_begin = src_begin;
  r.src_count = src_count;
  r.demand = demand;
  const Layout& L = r.L;
  HIP_TRY(zero_async(r.misc(), 64, st));
  const int nb = (src_count + 63) / 64;
  for (int b0 = 0; b0 < nb; b0 += L.G) {
    r.split = pick_split(t, nb - b0 < L.G ? nb - b0 : L.G, L.nb64, demand != nullptr);
    const GroupView gv = r.view(b0, nb - b0 < L.G ? nb - b0 : L.G);
    const int depth = t->level_bound;
    r.indexed = wide_masks_fit(t, L, gv.G);
    rc = r.indexed ? run_index(r, gv, demand ? depth + 1 : depth) : run_bfs(r, gv, demand ? depth + 1 : depth);
    if (rc != A2A_OK) return rc;
    rc = run_fwd(r, gv, depth);
    if (rc != A2A_OK) return rc;
    if (t->E > 0) {
      HIP_TRY(zero_async(gv.part, (size_t)gv.G * L.Epad * 8, st));
      if (demand) HIP_TRY(zero_async(gv.wpart, (size_t)gv.G * L.nb64 * 8, st));
      const unsigned grid = grid_for(gv.G, L.bpb * gv.split, r.inflight);
      // Unit demands: a batch's deepest level has no successors and its coef = 1/sigma was left by
      // the forward pass, nothing to add (the kernel skips it).  With demands it is visited like the others.
      for (int l = demand ? depth : depth - 1; l >= 0; --l) {
        const int cls = r.few(l) ? PROF_BWD_FEW : (r.few(l + 1) ? PROF_BWD_SPREAD : PROF_BWD);
        ProfScope ps(t, cls, st, l);
        auto launch = [&](auto kernel) { kernel<<<grid, kBlock, 0, st>>>(t->d_out_ptr, t->d_out_col, gv, l); };
        if (demand)  // precision of this level's sigma
          r.narrow(l) ? launch(k_bwd<float, true>) : launch(k_bwd<double, true>);
        else if (gv.split > 1)
          r.narrow(l) ? launch(k_bwd<float, false, true>) : launch(k_bwd<double, false, true>);
        else
          r.narrow(l) ? launch(k_bwd<float, false>) : launch(k_bwd<double, false>);
      }
      if (demand && weighted_dist) {
        k_fold_weighted_batch<<<(unsigned)gv.G, kBlock, 0, st>>>(gv.wpart, L.nb64);
        k_fold_weighted<<<1, 64, 0, st>>>(gv.wpart, gv.G, L.nb64, weighted_dist);
      }
      ProfScope ps(t, PROF_REDUCE, st);
      k_reduce_part<<<(unsigned)((t->E + kBlock - 1) / kBlock), kBlock, 0, st>>>(
          gv.part, L.Epad, gv.G, (long long)t->E, b0 == 0 ? 1 : 0, load);
    }
    rc = run_fold(r, gv, depth);
    if (rc != A2A_OK) return rc;
  }
  k_finish<<<1, 64, 0, st>>>(r.misc(), (long long)src_count * (t->N - 1), (long long*)dist_sum_total,
                             nullptr, (long long*)flags);
  HIP_TRY(hipGetLastError());
  if (t->prof_mode) t->prof_calls++;
  return A2A_OK;
}

}  // namespace

int a2a_link_loads(const a2a_topo* t, int32_t src_begin, int32_t src_count, double* load,
                   int64_t* dist_sum_total, int64_t* flags, void* workspace, size_t workspace_bytes,
                   void* hip_stream) {
  return link_loads(t, src_begin, src_count, nullptr, load, nullptr, dist_sum_total, flags, workspace,
                    workspace_bytes, hip_stream);
}

int a2a_link_loads_static(const a2a_topo* t, int32_t src_begin, int32_t src_count, double* load,
                          int64_t* dist_sum_total, int64_t* flags, void* hip_stream) {
  if (!t) return A2A_ERR_INVALID_ARG;
  if (src_count > 0 && src_count <= t->N) {
    // refuse before anything is enqueued: the array must hold at least one batch of this topology
    const Layout L = make_layout(t, src_count, A2A_WS_LOADS, A2A_STATIC_WORKSPACE_BYTES, false, false);
    if (L.G < 1) return A2A_ERR_WORKSPACE_TOO_SMALL;
  }
  return link_loads(t, src_begin, src_count, nullptr, load, nullptr, dist_sum_total, flags, t->d_scratch,
                    A2A_STATIC_WORKSPACE_BYTES, hip_stream);
}

int a2a_link_loads_demand(const a2a_topo* t, int32_t src_begin, int32_t src_count, const double* demand,
                          double* load, double* weighted_dist, int64_t* dist_sum_total, int64_t* flags,
                          void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!demand) return A2A_ERR_INVALID_ARG;
  return link_loads(t, src_begin, src_count, demand, load, weighted_dist, dist_sum_total, flags, workspace,
                    workspace_bytes, hip_stream);
}

int a2a_sssp_loads(const a2a_topo* t, int32_t src_begin, int32_t src_count, int32_t iter_sources, double* load,
                   int64_t* dist_sum_total, int64_t* flags, void* workspace, size_t workspace_bytes,
                   void* hip_stream) {
  int rc = check_common(t, src_begin, src_count, workspace);
  if (rc != A2A_OK) return rc;
  if (!load && t->E > 0) return A2A_ERR_INVALID_ARG;
  if (iter_sources <= 0 || iter_sources % 64 != 0) return A2A_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  const Use use(t, st);
  if (src_count == 0) {
    if (t->E > 0) HIP_TRY(zero_async(load, (size_t)t->E * 8, st));
    if (dist_sum_total) HIP_TRY(zero_async(dist_sum_total, 8, st));
    if (flags) HIP_TRY(zero_async(flags, 8, st));
    return A2A_OK;
  }
  // one iteration = one group: the workspace has to hold all its batches
  const int nb = (src_count + 63) / 64;
  const int per_iter = std::min(iter_sources / 64, nb);
  Run r;
  r.t = t;
  r.L = make_layout(t, per_iter * 64, A2A_WS_SSSP, workspace_bytes, false, false);
  if (r.L.G < per_iter) return A2A_ERR_WORKSPACE_TOO_SMALL;
  if (t->E > 0 && small_sssp_fits(t, src_count))
    return small_sssp(t, src_begin, src_count, std::min(per_iter * 64, src_count), load, dist_sum_total, flags,
                      (char*)workspace, workspace_bytes, st);
  r.ws = (char*)workspace;
  r.st = st;
  r.src_begin = src_begin;
  r.src_count = src_count;
  const Layout& L = r.L;
  SsspView sv;
  sv.cost = (long long*)(r.ws + L.off_cost);
  sv.pick = (int*)(r.ws + L.off_pick);
  sv.sub = (int*)(r.ws + L.off_sub);
  sv.iload = (unsigned long long*)(r.ws + L.off_iload);
  HIP_TRY(zero_async(r.misc(), 64, st));
  HIP_TRY(zero_async(sv.iload, L.Epad * 8, st));
  const int depth = t->level_bound;
  for (int b0 = 0; b0 < nb; b0 += per_iter) {
    const GroupView gv = r.view(b0, nb - b0 < per_iter ? nb - b0 : per_iter);
    rc = run_bfs(r, gv, depth);
    if (rc != A2A_OK) return rc;
    // nodes per wave: 64, or 8 when the iteration has too few batches to give every SIMD a wave otherwise
    const int npw = (long long)gv.G * L.Npad >= 64ll * 4096 ? 64 : 8;
    const unsigned grid = grid_for(gv.G, L.bpb * (kWave / npw), r.inflight);
    for (int l = 1; l <= depth; ++l) {
      ProfScope ps(t, PROF_FWD, st, l);
      k_sssp_fwd<<<grid, kBlock, 0, st>>>(t->d_in_ptr, t->d_in_col, t->d_in_link, gv, sv, l, npw);
    }
    for (int l = depth; l >= 0; --l) {
      ProfScope ps(t, PROF_BWD, st, l);
      k_sssp_bwd<<<grid, kBlock, 0, st>>>(t->d_out_ptr, t->d_out_col, gv, sv, l, npw);
    }
    rc = run_fold(r, gv, depth);
    if (rc != A2A_OK) return rc;
  }
  if (t->E > 0)
    k_sssp_output<<<(unsigned)((t->E + kBlock - 1) / kBlock), kBlock, 0, st>>>(sv.iload, (long long)t->E, load);
  k_finish<<<1, 64, 0, st>>>(r.misc(), (long long)src_count * (t->N - 1), (long long*)dist_sum_total,
                             nullptr, (long long*)flags);
  HIP_TRY(hipGetLastError());
  return A2A_OK;
}

int a2a_schedule_bound(const a2a_topo* t, const double* load, int64_t sum_dist, int64_t flags,
                       double m_bytes, double b_bytes_per_s, a2a_bound* out, void* hip_stream) {
  if (!t || !out || !load || t->E <= 0 || !(m_bytes > 0.0) || !(b_bytes_per_s > 0.0) || sum_dist < 0)
    return A2A_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  const unsigned slot = t->next_slot.fetch_add(1) % a2a_topo::kSlots;
  int64_t* const h_res = t->h_slots + slot * a2a_topo::kSlotWords;
  const Use use(t, st);
  const uint64_t covered = use.covered();
  h_res[kExtremaDone] = 0;
  k_load_extrema<<<extrema_groups(t->E, 32 * kExtremaThreads, 4 * kExtremaThreads), kExtremaThreads, 0, st>>>(
      load, (int)t->E, t->d_scratch_slots + slot * (kExtremaGroups * kExtremaWords), t->d_arrived + slot,
      (long long*)h_res);
  HIP_TRY(hipGetLastError());
  HIP_TRY(wait_for(st, [&] { return seen(&h_res[kExtremaDone]) != 0; }));
  use.waited(covered);
  double lmax, lmin;
  std::memcpy(&lmax, &h_res[0], 8);
  std::memcpy(&lmin, &h_res[2], 8);
  const double m = m_bytes, b = b_bytes_per_s;
  out->max_load = lmax;
  out->argmax_arc = h_res[1];
  out->min_load = lmin;
  out->sum_dist = sum_dist;
  out->n_links = t->E;
  out->n_nodes = t->N;
  out->dmax = t->dmax;
  out->t_sched = lmax * m / b;
  out->t_lb_nd = (double)sum_dist * m / ((double)t->N * (double)t->dmax * b);
  out->t_lb_links = (double)sum_dist * m / ((double)t->E * b);
  out->ratio = out->t_sched / out->t_lb_nd;
  out->throughput = (double)(t->N - 1) * m / out->t_sched;
  out->flow_value = 1.0 / lmax;
  out->throughput_upper = (double)(t->N - 1) * out->flow_value * b;
  return (flags & A2A_FLAG_UNREACHABLE) ? A2A_ERR_DISCONNECTED : A2A_OK;
}

int a2a_schedule_bound_cap(const a2a_topo* t, const double* load, const double* cap, int64_t sum_dist,
                           int64_t flags, double m_bytes, double b_bytes_per_s, a2a_bound_cap* out,
                           void* hip_stream) {
  if (!t || !out || !load || !cap || t->E <= 0 || !(m_bytes > 0.0) || !(b_bytes_per_s > 0.0) || sum_dist < 0)
    return A2A_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  const unsigned slot = t->next_slot.fetch_add(1) % a2a_topo::kSlots;
  int64_t* const h_res = t->h_slots + slot * a2a_topo::kSlotWords;
  const Use use(t, st);
  const uint64_t covered = use.covered();
  h_res[kExtremaDone] = 0;
  const int groups = extrema_groups(t->N, kExtremaThreads, kBlock);
  k_util_extrema<<<groups, groups == 1 ? kExtremaThreads : kBlock, 0, st>>>(
      t->d_out_ptr, load, cap, t->N, t->d_scratch_slots + slot * (kExtremaGroups * kExtremaWords), t->d_arrived + slot,
      (long long*)h_res);
  HIP_TRY(hipGetLastError());
  HIP_TRY(wait_for(st, [&] { return seen(&h_res[kExtremaDone]) != 0; }));
  use.waited(covered);
  if (h_res[5] != 0) return A2A_ERR_INVALID_ARG;  // a capacity that is not positive and finite
  double umax, umin, total, cmax;
  std::memcpy(&umax, &h_res[0], 8);
  std::memcpy(&umin, &h_res[2], 8);
  std::memcpy(&total, &h_res[3], 8);
  std::memcpy(&cmax, &h_res[4], 8);
  const double m = m_bytes, b = b_bytes_per_s;
  out->max_util = umax;
  out->argmax_arc = h_res[1];
  out->min_util = umin;
  out->sum_dist = sum_dist;
  out->n_links = t->E;
  out->n_nodes = t->N;
  out->total_capacity = total;
  out->max_node_capacity = cmax;
  out->t_sched = umax * m / b;
  out->t_lb_nd = (double)sum_dist * m / ((double)t->N * cmax * b);
  out->t_lb_links = (double)sum_dist * m / (total * b);
  out->ratio = out->t_sched / out->t_lb_nd;
  out->throughput = (double)(t->N - 1) * m / out->t_sched;
  out->flow_value = 1.0 / umax;
  out->throughput_upper = (double)(t->N - 1) * out->flow_value * b;
  return (flags & A2A_FLAG_UNREACHABLE) ? A2A_ERR_DISCONNECTED : A2A_OK;
}

int a2a_tree_lower_bound(int32_t N, int32_t d, double m_bytes, double b_bytes_per_s, a2a_tree_bound* out) {
  if (!out || N < 1 || d < 1 || !(m_bytes > 0.0) || !(b_bytes_per_s > 0.0)) return A2A_ERR_INVALID_ARG;
  int64_t left = (int64_t)N - 1, width = 1, sum = 0;
  int32_t level = 0;
  bool full = true;
  while (left > 0) {
    ++level;
    // d^level hosts fit on this level; stop multiplying once it exceeds what is left
    width = width > left / d ? left + 1 : width * d;
    const int64_t take = width < left ? width : left;
    full = take == width;
    sum += take * level;
    left -= take;
  }
  out->s_min = sum;
  out->height = level;
  out->full = full ? 1 : 0;
  out->t_lb = (double)sum * m_bytes / ((double)d * b_bytes_per_s);
  out->throughput_ub = N > 1 ? (double)(N - 1) * m_bytes / out->t_lb : 0.0;
  return A2A_OK;
}

int a2a_profile_enable(a2a_topo* t, int mode) {
  if (!t || mode < 0 || mode > 2) return A2A_ERR_INVALID_ARG;
  for (auto& rec : t->prof_recs) {
    (void)hipEventDestroy(rec.beg);
    (void)hipEventDestroy(rec.end);
  }
  t->prof_recs.clear();
  t->prof_calls = 0;
  t->prof_depth = 0;
  t->prof_groups = 0;
  t->prof_narrow = 0;
  t->prof_fwd_flavours = t->prof_bwd_flavours = 0;
  t->prof_mode = mode;
  std::memset(t->prof_pairs_level, 0, sizeof(t->prof_pairs_level));
  std::memset(t->prof_dag_level, 0, sizeof(t->prof_dag_level));
  return A2A_OK;
}

int a2a_profile_read(a2a_topo* t, a2a_profile* out) {
  if (!t || !out) return A2A_ERR_INVALID_ARG;
  std::memset(out, 0, sizeof(*out));
  HIP_TRY(hipDeviceSynchronize());
  for (auto& rec : t->prof_recs) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, rec.beg, rec.end) == hipSuccess && rec.cls >= 0 && rec.cls < PROF_CLASSES) {
      out->ms[rec.cls] += ms;
      out->launches[rec.cls] += 1;
      const int l = rec.level < A2A_PROF_MAX_LEVELS ? rec.level : A2A_PROF_MAX_LEVELS - 1;
      out->ms_level[rec.cls][l] += ms;
    }
  }
  int64_t dag = 0;
  for (int l = 0; l < A2A_PROF_MAX_LEVELS; ++l) {
    out->pairs_level[l] = t->prof_pairs_level[l];
    out->dag_level[l] = t->prof_dag_level[l];
    dag += t->prof_dag_level[l];
  }
  out->dag_links = dag;
  out->calls = t->prof_calls;
  out->depth = t->prof_depth;
  out->groups = t->prof_groups;
  out->narrow_levels = t->prof_narrow;
  out->fwd_flavours = t->prof_fwd_flavours;
  out->bwd_flavours = t->prof_bwd_flavours;
  return A2A_OK;
}

}  // extern "C"
