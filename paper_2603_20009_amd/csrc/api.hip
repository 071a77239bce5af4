// C ABI of libskm and the host-side driver of Algorithm 1 (SuperKMeans): every arithmetic step on the
// points runs in the HIP kernels of this library; the host keeps scalars only (d', prune fraction,
// recall history, the list of empty clusters and the integer PRNG that re-seeds them).
#include "../../include/skm.h"
#include "skm_internal.h"

#include <algorithm>
#include <atomic>
#include <chrono>
#include <mutex>
#include <thread>
#include <system_error>
#include <functional>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <string>
#include <vector>

using namespace skm;

namespace {

thread_local std::string g_last_error;

int fail(int rc, const char *what) {
  g_last_error = what;
  return rc;
}
int fail_hip(hipError_t e, const char *where) {
  g_last_error = std::string(where) + ": " + hipGetErrorString(e);
  return e == hipErrorOutOfMemory ? SKM_ENOMEM : SKM_EHIP;
}
#define HIPCHK(expr)                                              \
  do {                                                            \
    hipError_t e__ = (expr);                                      \
    if (e__ != hipSuccess) return fail_hip(e__, #expr);           \
  } while (0)

// Device blocks that calls without a lent workspace have finished with, for the next such call: hipMalloc and hipFree of a
// few buffers cost a step call 0.2 to 0.3 ms, several times its kernels, and hipFree of gigabytes 10 ms for each.  Every
// call waits for its stream before it gives a block back, so the next one may use it on any stream; a call that fails
// frees its block instead.  Bounded (kMost bytes over all devices), safe between threads, emptied by
// skm_release_memory() and by a hipMalloc of the library that fails.
struct BlockCache {
  struct Block {
    void *p;
    size_t bytes;
    int dev;
  };
  static constexpr size_t kMost = (size_t)4 << 30;
  std::mutex mu;
  std::vector<Block> idle;
  size_t held = 0;
  static int device() {
    int dev = 0;
    (void)hipGetDevice(&dev);
    return dev;
  }
  // the smallest idle block of the current device that holds `bytes`
  void *take(size_t bytes, size_t *cap) {
    const int dev = device();
    std::lock_guard<std::mutex> lock(mu);
    size_t best = idle.size();
    for (size_t i = 0; i < idle.size(); ++i)
      if (idle[i].dev == dev && idle[i].bytes >= bytes && (best == idle.size() || idle[i].bytes < idle[best].bytes)) best = i;
    if (best == idle.size()) return nullptr;
    void *p = idle[best].p;
    *cap = idle[best].bytes;
    held -= idle[best].bytes;
    idle.erase(idle.begin() + (std::ptrdiff_t)best);
    return p;
  }
  // keeps the block if the bound allows it, dropping older ones for it; frees it otherwise
  void give(void *p, size_t bytes) {
    std::vector<Block> drop;
    {
      const int dev = device();
      std::lock_guard<std::mutex> lock(mu);
      if (bytes <= kMost) {
        while (held + bytes > kMost || idle.size() >= 16) {
          drop.push_back(idle.front());
          held -= idle.front().bytes;
          idle.erase(idle.begin());
        }
        idle.push_back({p, bytes, dev});
        held += bytes;
        p = nullptr;
      }
    }
    for (const Block &b : drop) (void)hipFree(b.p);
    if (p) (void)hipFree(p);
  }
  size_t idle_bytes() {   // of the current device
    const int dev = device();
    std::lock_guard<std::mutex> lock(mu);
    size_t sum = 0;
    for (const Block &b : idle)
      if (b.dev == dev) sum += b.bytes;
    return sum;
  }
  void release() {
    std::vector<Block> drop;
    {
      std::lock_guard<std::mutex> lock(mu);
      drop.swap(idle);
      held = 0;
    }
    for (const Block &b : drop) (void)hipFree(b.p);
  }
};
BlockCache &block_cache() {
  static BlockCache *c = new BlockCache;   // (never destroyed: the process's end takes the blocks)
  return *c;
}
hipError_t device_malloc(void **p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    block_cache().release();
    e = hipMalloc(p, bytes);
  }
  return e;
}

// device allocations released when the call ends, whichever way it ends
// A preallocated slab that Pools of nested calls carve their buffers from (the hierarchical fit runs hundreds of small
// fits; a hipMalloc per buffer would dominate them).  A Pool constructed while an arena is current takes memory from it
// and gives it back, stack-like, when it is destroyed; what does not fit falls back to hipMalloc.
struct Arena {
  char *base = nullptr;
  size_t cap = 0, off = 0;
  bool owned = true;     // false: the caller's memory (params->workspace)
  bool strict = false;   // true: what does not fit is an error, never a hipMalloc
  bool keep = false;     // the call has waited for its stream: an owned block goes to the cache
  ~Arena() {
    if (!base || !owned) return;
    if (keep) block_cache().give(base, cap);
    else (void)hipFree(base);
  }
  hipError_t init(size_t bytes) {
    bytes = (bytes + ((size_t)2 << 20) - 1) & ~(((size_t)2 << 20) - 1);
    base = static_cast<char *>(block_cache().take(bytes, &cap));
    if (base) return hipSuccess;
    cap = bytes;
    return device_malloc(reinterpret_cast<void **>(&base), bytes);
  }
  void lend(void *mem, size_t bytes) {
    base = static_cast<char *>(mem);
    cap = bytes;
    owned = false;
    strict = true;
  }
};
thread_local Arena *tl_arena = nullptr;
struct ArenaScope {
  Arena *saved;
  explicit ArenaScope(Arena *a) : saved(tl_arena) { tl_arena = a; }
  ~ArenaScope() { tl_arena = saved; }
};

struct Pool {
  std::vector<void *> ptrs;
  Arena *arena = tl_arena;
  size_t mark = tl_arena ? tl_arena->off : 0;
  bool count_only = false;   // plan mode: add up what would be taken (256-byte granules), hand out nothing
  size_t counted = 0;
  ~Pool() {
    for (void *p : ptrs) (void)hipFree(p);
    if (arena) arena->off = mark;
  }
  template <typename T>
  hipError_t get(T **out, size_t count) {
    void *p = nullptr;
    size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
    if (count_only) {
      counted += (bytes + 255) & ~(size_t)255;
      *out = nullptr;
      return hipSuccess;
    }
    if (arena) {
      const size_t at = (arena->off + 255) & ~(size_t)255;
      if (at + bytes <= arena->cap) {
        arena->off = at + bytes;
        *out = reinterpret_cast<T *>(arena->base + at);
        return hipSuccess;
      }
      if (arena->strict) {   // a caller-owned workspace: the call allocates nothing
        *out = nullptr;
        return hipErrorOutOfMemory;
      }
    }
    hipError_t e = device_malloc(&p, bytes);
    if (e != hipSuccess) {
      *out = nullptr;
      return e;
    }
    ptrs.push_back(p);
    *out = static_cast<T *>(p);
    return hipSuccess;
  }
  // gives back what has been taken since `m` (nothing launched may use it)
  struct Mark {
    size_t nptrs, off;
  };
  Mark taken() const { return {ptrs.size(), arena ? arena->off : 0}; }
  void give_back(const Mark &m) {
    for (size_t i = m.nptrs; i < ptrs.size(); ++i) (void)hipFree(ptrs[i]);
    ptrs.resize(m.nptrs);
    if (arena) arena->off = m.off;
  }
};

// Page-locked host memory for the few numbers that every step reports to the host: copies into it are asynchronous,
// so one wait per step covers all of them (a copy into pageable memory waits for its own staging).  Blocks are kept
// in a per-thread cache and reused by later calls on that thread (the hierarchical fit runs hundreds of small fits);
// worker threads release their cache before they end, that of a caller's thread stays until the process ends.
// Whoever gives a block back has waited for every kernel that may write into it: the next call on the thread, on whatever
// stream, takes it at once.
struct PinnedCache {
  std::vector<std::pair<void *, size_t>> idle;
  void *take(size_t bytes, size_t *cap) {
    for (size_t i = 0; i < idle.size(); ++i)
      if (idle[i].second >= bytes) {
        void *p = idle[i].first;
        *cap = idle[i].second;
        idle.erase(idle.begin() + (std::ptrdiff_t)i);
        return p;
      }
    void *p = nullptr;
    const size_t want = std::max<size_t>(bytes, (size_t)1 << 16);
    if (hipHostMalloc(&p, want, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    *cap = want;
    return p;
  }
  void give(void *p, size_t cap) { idle.emplace_back(p, cap); }
  void release() {
    for (auto &b : idle) (void)hipHostFree(b.first);
    idle.clear();
  }
};
thread_local PinnedCache tl_pinned;

// one page-locked word that a kernel on the stream writes and the host reads once it has waited for the stream
struct PinnedWord {
  volatile unsigned int *host = nullptr;
  unsigned int *dev = nullptr;
  void *block = nullptr;
  size_t cap = 0;
  hipStream_t st;
  bool waited = false;   // (left false by a call that returns on the way: the destructor waits)
  explicit PinnedWord(hipStream_t stream) : st(stream) {
    block = tl_pinned.take(sizeof(unsigned int), &cap);
    void *dv = nullptr;
    if (!block || hipHostGetDevicePointer(&dv, block, 0) != hipSuccess) return;
    host = static_cast<volatile unsigned int *>(block);
    dev = static_cast<unsigned int *>(dv);
  }
  ~PinnedWord() {
    if (!block) return;
    if (!waited) (void)hipStreamSynchronize(st);
    tl_pinned.give(block, cap);
  }
  int wait() {
    HIPCHK(hipStreamSynchronize(st));
    waited = true;
    return SKM_OK;
  }
  PinnedWord(const PinnedWord &) = delete;
  PinnedWord &operator=(const PinnedWord &) = delete;
};

struct Events {
  std::vector<hipEvent_t> ev;
  ~Events() {
    for (hipEvent_t e : ev) (void)hipEventDestroy(e);
  }
  hipEvent_t next() {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    ev.push_back(e);
    return e;
  }
};

// Stage times of a call: stamps that kernels at the stages' borders write into page-locked memory (put_stamp).  The time
// between two consecutive marks of a step is charged to the stage of the later mark; all of them are read once the
// stream has been waited for.
enum Stage { ST_NONE = 0, ST_TAU, ST_GEMM, ST_PRUNE, ST_UPDATE, ST_ETR, ST_COUNT };
struct StageTimer {
  bool on;
  void *block = nullptr;
  size_t block_bytes = 0, cap = 0, used = 0;
  volatile stamp_t *host = nullptr;
  stamp_t *dev = nullptr;
  double ms_per_tick = 1e-5;
  std::vector<std::pair<int, size_t>> marks;   // (stage, stamp)
  std::vector<size_t> first;                   // first mark of every step
  hipStream_t st;
  bool waited = false;   // the call has waited for its stream behind the last stamp (left false by one that returns on the way)
  StageTimer(bool enable, hipStream_t stream) : on(enable), st(stream) {}
  StageTimer(const StageTimer &) = delete;
  StageTimer &operator=(const StageTimer &) = delete;
  ~StageTimer() {
    if (!block) return;
    if (!waited) (void)hipStreamSynchronize(st);
    tl_pinned.give(block, block_bytes);
  }
  // room for so many stamps (further ones are not taken)
  int init(size_t stamps) {
    if (!on) return SKM_OK;
    static const double tick = []() {
      int dev_id = 0, khz = 0;
      (void)hipGetDevice(&dev_id);
      if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev_id) != hipSuccess || khz <= 0) khz = 100000;
      return 1.0 / khz;
    }();
    ms_per_tick = tick;
    cap = std::min<size_t>(stamps, (size_t)1 << 17);
    block = tl_pinned.take(cap * sizeof(stamp_t), &block_bytes);
    void *dv = nullptr;
    if (!block || hipHostGetDevicePointer(&dv, block, 0) != hipSuccess) return fail(SKM_EHIP, "hipHostMalloc failed for the stage times");
    host = static_cast<volatile stamp_t *>(block);
    dev = static_cast<stamp_t *>(dv);
    std::memset(block, 0, cap * sizeof(stamp_t));
    return SKM_OK;
  }
  // a stamp on its own (*at = its number)
  stamp_t *point(size_t *at) {
    *at = next();
    return on && *at < cap ? dev + *at : nullptr;
  }
  // The border lies where the next kernel that carries a stamp starts: that stamp serves for both.
  static constexpr size_t kNone = ~(size_t)0;
  size_t waiting = kNone;
  size_t next() {
    const size_t at = waiting != kNone ? waiting : used++;
    waiting = kNone;
    return at;
  }
  void mark_next(int stage) {
    if (!on || used >= cap) return;
    waiting = used++;
    marks.push_back({stage, waiting});
  }
  void begin_step() { first.push_back(marks.size()); }
  // the border that ends a stretch of `stage` (and starts the next)
  stamp_t *mark(int stage) {
    const size_t at = next();
    if (!on || at >= cap) return nullptr;
    marks.push_back({stage, at});
    return dev + at;
  }
  // (call these after the stream has been waited for)
  float between(size_t a, size_t b) const {
    if (!on || a >= cap || b >= cap || host[a] == 0 || host[b] <= host[a]) return 0.f;
    return (float)((double)(host[b] - host[a]) * ms_per_tick);
  }
  void collect(size_t q, float ms[ST_COUNT], float *total) const {
    for (int s = 0; s < ST_COUNT; ++s) ms[s] = 0.f;
    *total = 0.f;
    if (q >= first.size()) return;
    const size_t end = q + 1 < first.size() ? first[q + 1] : marks.size();
    for (size_t i = first[q] + 1; i < end; ++i) {
      const float t = between(marks[i - 1].second, marks[i].second);
      ms[marks[i].first] += t;
      *total += t;
    }
  }
  void reset() {   // the stamps are used again
    marks.clear();
    first.clear();
    if (block) std::memset(block, 0, std::min(used, cap) * sizeof(stamp_t));
    used = 0;
    waiting = kNone;
  }
};

// ---------------------------------------------------------------- integer PRNG (splitmix64)
struct Rng {
  uint64_t s;
  uint64_t next() {
    s += 0x9E3779B97F4A7C15ULL;
    uint64_t z = s;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
  }
  double uniform() { return (double)(next() >> 11) * (1.0 / 9007199254740992.0); }
};
Rng rng_stream(uint64_t seed, uint64_t stream) { return Rng{seed + stream * 0xD1342543DE82EF95ULL}; }
enum { STREAM_INIT = 0, STREAM_SPLIT = 1, STREAM_QUERIES = 2, STREAM_ROTATION = 3, STREAM_SAMPLE = 4 };

// k distinct indices of [0, n): the first k steps of a Fisher-Yates shuffle of the identity
void sample_rows(uint64_t seed, uint64_t stream, int64_t n, int32_t k, int64_t *out) {
  Rng r = rng_stream(seed, stream);
  if ((int64_t)k * 8 >= n) {
    std::vector<int64_t> perm((size_t)n);
    for (int64_t i = 0; i < n; ++i) perm[(size_t)i] = i;
    for (int32_t i = 0; i < k; ++i) {
      const int64_t j = i + (int64_t)(r.next() % (uint64_t)(n - i));
      std::swap(perm[(size_t)i], perm[(size_t)j]);
      out[i] = perm[(size_t)i];
    }
    return;
  }
  // few draws from many rows: the same shuffle, keeping only the entries that no longer hold their own index (step i
  // reads positions i and j >= i and never looks at a position below i again, so position i itself need not be kept).  They are kept
  // in one table, at most half full: with an allocation a row the draw was as long as the rotation that it runs beside, and longer
  // again where the runtime gives back what finished launches held, on a thread of its own, at the same time (3000 of 100 000
  // rows in a fit: 98 us where the host waits for the stream after every step, 163 to 280 where it watches the report).
  int bits = 4;
  while ((int64_t)1 << bits < 2 * (int64_t)k) ++bits;
  struct Moved {
    int64_t at = -1, holds = 0;
  };
  std::vector<Moved> moved((size_t)1 << bits);
  const size_t mask = moved.size() - 1;
  auto find = [&](int64_t at) -> Moved & {   // its entry, or the free one that it would take
    size_t h = (size_t)(((uint64_t)at * 0x9E3779B97F4A7C15ULL) >> (64 - bits));
    while (moved[h].at >= 0 && moved[h].at != at) h = (h + 1) & mask;
    return moved[h];
  };
  for (int32_t i = 0; i < k; ++i) {
    const int64_t j = i + (int64_t)(r.next() % (uint64_t)(n - i));
    const Moved &mi = find(i);
    const int64_t vi = mi.at < 0 ? (int64_t)i : mi.holds;
    Moved &mj = find(j);
    out[i] = mj.at < 0 ? j : mj.holds;
    mj.at = j;
    mj.holds = vi;
  }
}

// ---------------------------------------------------------------- scalar rules
double theta_ratio(int32_t d, int32_t t, double eps0) {
  if (t >= d) return 1.0;
  if (t <= 0) return 0.0;
  const double s = 1.0 + eps0 / std::sqrt((double)t);
  const double r = (double)t / (double)d * s * s;
  return r < 1.0 ? r : 1.0;
}
int32_t snap16(double v, int32_t d) {
  int32_t top = d / 16 * 16;
  if (top < 16) top = 16;
  int32_t r = (int32_t)std::floor(v / 16.0 + 0.5) * 16;
  return std::min(std::max(r, 16), top);
}
int32_t dprime_init(int32_t d, double frac) { return snap16(std::floor((double)d * frac), d); }
int32_t dprime_adjust(int32_t d, int32_t dp, double f, double lo, double hi, double step) {
  // nearest multiple of 16, but at least one step of 16 in the chosen direction
  if (f > hi) return std::min(snap16((double)dp - step * (double)dp, d), snap16((double)dp - 16.0, d));
  if (f < lo) return std::max(snap16((double)dp + step * (double)dp, d), snap16((double)dp + 16.0, d));
  return dp;
}
// Section 6: sqrt(k) meso-clusters; the k fine clusters are shared out in proportion to sqrt(n_i), one to every
// non-empty meso-cluster first, floors of the quotas next, the rest by largest fractional part (lowest index on ties),
// never more clusters than points.
int32_t hier_meso_count(int32_t k) {
  const int32_t km = (int32_t)std::floor(std::sqrt((double)k) + 0.5);
  return std::min(std::max(km, 1), k);
}
void hier_alloc(const int64_t *sizes, int32_t km, int32_t k, int32_t *counts) {
  std::vector<double> root((size_t)km), frac((size_t)km);
  double W = 0.0;
  int64_t given = 0;
  for (int32_t i = 0; i < km; ++i) {
    root[(size_t)i] = std::sqrt((double)sizes[i]);
    W += root[(size_t)i];
    counts[i] = sizes[i] > 0 ? 1 : 0;
    given += counts[i];
  }
  const int64_t r = std::max<int64_t>((int64_t)k - given, 0);
  for (int32_t i = 0; i < km; ++i) {
    const double q = W > 0.0 ? (double)r * root[(size_t)i] / W : 0.0;
    const double whole = std::floor(q);
    const int64_t g = std::min<int64_t>((int64_t)whole, sizes[i] - counts[i]);
    counts[i] += (int32_t)g;
    given += g;
    frac[(size_t)i] = q - whole;
  }
  std::vector<int32_t> order((size_t)km);
  for (int32_t i = 0; i < km; ++i) order[(size_t)i] = i;
  std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return frac[(size_t)a] > frac[(size_t)b]; });
  int64_t left = (int64_t)k - given;
  while (left > 0) {
    bool progress = false;
    for (int32_t a = 0; a < km && left > 0; ++a) {
      const int32_t i = order[(size_t)a];
      if ((int64_t)counts[i] < sizes[i]) {
        ++counts[i];
        --left;
        progress = true;
      }
    }
    if (!progress) break;
  }
}
int32_t nprobe_of(int32_t k, double frac) {
  int32_t np = (int32_t)std::floor(frac * (double)k + 0.5);
  return std::min(std::max(np, 1), k);
}

// ---------------------------------------------------------------- rotation matrix (device, fp64)
int make_rotation_dev(Pool &pool, int32_t d, uint64_t seed, hipStream_t st, float *R_out) {
  double *Qw = nullptr, *Cw = nullptr, *Ww = nullptr;
  HIPCHK(pool.get(&Qw, (size_t)d * d + 2));
  HIPCHK(pool.get(&Cw, rotation_cwork(d)));
  HIPCHK(pool.get(&Ww, (size_t)((d + 63) / 64) * 64 * d));
  HIPCHK(launch_make_rotation(d, rng_stream(seed, STREAM_ROTATION).s, Qw, Cw, Ww, R_out, st));
  return SKM_OK;
}

inline int32_t round_up(int32_t v, int32_t m) { return (v + m - 1) / m * m; }

// *slot = bit pattern of max |A| (the bound the split-fp16 GEMMs scale their operands by)
int measure_absmax(const float *A, int64_t lda, int64_t rows, int32_t cols, unsigned int *slot, hipStream_t st,
                   int max_blocks = 0) {
  HIPCHK(launch_fill_u32(slot, 1, 0u, st));
  HIPCHK(launch_absmax(A, lda, rows, cols, slot, st, max_blocks));
  return SKM_OK;
}
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// fit = false: an assignment of n points to k given centroids, where k may exceed n
int check_shape(const void *X, int64_t n, int32_t d, int32_t k, bool fit = true) {
  if (!X) return fail(SKM_EINVAL, "null input pointer");
  if (n < 1 || n >= (int64_t)1 << 31) return fail(SKM_EINVAL, "n out of range [1, 2^31)");
  if (d < 16 || d > 16384) return fail(SKM_EINVAL, "d out of range [16, 16384]");
  if (k < 1 || (fit && k > n) || k > (1 << 24)) return fail(SKM_EINVAL, "k out of range [1, min(n, 2^24)]");
  return SKM_OK;
}

// the caller's initial rows, if there are any (checked before anything is enqueued)
int check_init_idx(const skm_params &p, int64_t n, int32_t k) {
  for (int32_t i = 0; p.init_idx && i < k; ++i)
    if (p.init_idx[i] < 0 || p.init_idx[i] >= n) return fail(SKM_EINVAL, "init_idx out of range");
  return SKM_OK;
}

// ---------------------------------------------------------------- one fit / assign context
struct Ctx {
  hipStream_t st = nullptr;
  Pool pool;
  int64_t n = 0;
  int32_t d = 0, ds = 0, k = 0;
  const float *Xr = nullptr;  // rotated (or original) points, row stride ldx, padded to ds
  int64_t ldx = 0;
  float *Y = nullptr;         // centroids k x ds (rotated space)
  float *Ypdx = nullptr;
  uint32_t *Xs = nullptr;     // split-fp16 copy of Xr for the progressive kernel, made with xnp
  uint32_t *Ys = nullptr;     // the same of Y, remade in every pruned step
  float *xnp = nullptr;       // [ds / 16][n] prefix norms of the points at every multiple of 16 dims, written by the
  bool xnp_valid = false;     // first pruned step (the points of a context never change)
  bool xh_valid = false;      // Xh likewise: left out of a pass that a regrouping pass will repeat
  // Regrouping (a fit with several steps left): once the tables exist, a threshold pass rewrites the points, their split
  // copy, their tables and every per-point array in the order of their clusters (step_pruned).  Row tiles then hold points
  // of one or two clusters, whose challengers are the same few centroids: the alive pairs of a step gather in few tiles, the
  // others end at the first test, and the rows and centroid blocks the gather kernel fetches are shared by neighbouring pairs.
  float *Xr2 = nullptr;          // [n][ds] the points in the new order (NULL: no regrouping in this context)
  int32_t *pos_to_id = nullptr;  // [n] point of every position
  unsigned char *subkey = nullptr;   // [n] scratch: the key that orders the points inside a cluster
  float *Xr_own = nullptr;       // Xr where its rows are the library's own: once regrouped they are room for the next regrouping
  int32_t regroup_left = 0;      // assignment steps of the fit from this one on (0: its points are not regrouped)
  int64_t moved = 0;             // changes of a label since the points were last grouped by it
  int32_t max_cluster = -1;      // size of the largest cluster at the last update (-1: none yet)
  bool single_step = false;      // an assignment on its own, with incumbents of the caller's or none
  bool group_now = false;        // a single step that groups the points by their incumbents itself (assign_impl)
  int32_t *grp_cnt = nullptr;    // [k + 1] sizes of those groups, and how many of a sample of the thresholds are in a tail
  int32_t *class_ws = nullptr;   // [threshold_class_words(n)] scratch of their order by threshold
  bool order_fresh = false;      // up.order groups the points by the labels now in `prev`
  bool permuted = false;
  unsigned long long *point_keys = nullptr;   // keys that name points (ETR ground truth): renumbered with the points
  int64_t n_point_keys = 0;
  float *ynp = nullptr;       // [nb + 1][k] prefix norms of the centroids at the checkpoints of the current step
  float *ynorm = nullptr;
  float *tau = nullptr, *dist = nullptr;
  unsigned long long *best = nullptr;
  int32_t *assign = nullptr, *prev = nullptr;
  Pair *pairs = nullptr;
  int64_t pair_cap = 0, sub_cap = 0, chunk_rows = 0;
  int32_t nchunks = 0;
  unsigned int emit_max = 0;         // a tile with at most this many alive pairs goes to the gather kernel
  unsigned int *counters = nullptr;  // per chunk the fill counters of the sub-lists, then the tile counters
  size_t ncounters = 0;              // words in `counters`
  float *ratio_dev = nullptr;        // [kMaxBlocks + 1]
  unsigned long long *scal = nullptr;  // [SC_COUNT]
  double *obj_partial = nullptr;
  UpdateWs up{};
  IncUpdateWs inc{};                 // workspace of the incremental update
  double *S = nullptr;               // [k][ds] cluster sums of the last update (fp64), valid once S_valid
  bool S_valid = false;
  bool split_last = false;           // the last update re-seeded empty clusters (their donors' rows are perturbed)
  // thresholds that the last step left in tau and that still hold: of no point, of those in untouched clusters, of all
  enum { KEPT_NONE = 0, KEPT_UNTOUCHED = 1, KEPT_ALL = 2 };
  int tau_kept = KEPT_NONE;
  uint32_t *touched = nullptr;       // [k] clusters that the last (incremental) update changed
  int32_t inc_updates = 0;           // update steps that took the incremental path
  int32_t *split_dev = nullptr;
  bool block_stats = false;
  // low-precision first filter (screen.hip): mode as params->screen; buffers for one chunk of rows
  int32_t screen_mode = 0;
  double last_prune_frac = -1.0;     // of the previous pruned step of this context (-1: none yet)
  double last_listed = 1.0;          // share of the 128 x 128 tiles that it worked on (1 where it listed none)
  uint32_t *colmask = nullptr;
  float *scr_arow = nullptr, *scr_ycol = nullptr;
  uint32_t *Xh = nullptr, *Yh = nullptr;   // the hi halves of Xs, Ys as planes of their own
  uint32_t *Yd = nullptr;                  // ... of Ys from d' on, for the listed tiles
  int32_t pruned_steps = 0;                // pruned steps this context has completed
  bool exact_filter_off = false;           // iteration 1 takes the full GEMM (set after a candidate-list overflow)
  float2 *scr_widen = nullptr;
  int32_t *scr_cnt = nullptr, *scr_first = nullptr, *scr_ntiles = nullptr, *scr_cols = nullptr, *scr_pos = nullptr;
  int2 *scr_tile_rt = nullptr;
  unsigned int *amax = nullptr;      // [AM_COUNT] magnitude bounds of the GEMM operands
  enum { AM_XR = 0, AM_Y = 1, AM_X = 2, AM_Q = 3, AM_QR = 4, AM_COUNT = 8, AM_ROTATION = 8 };   // (the last: Rot's words, behind the others)
  unsigned int *xr_bound = nullptr;  // that of Xr: amax[AM_XR], or a word that is kept with the rows (fit_host_impl)

  // What a step reports: the finalize kernel writes it straight into this page-locked block (see PinnedCache), so the
  // host waits for the stream once per step and copies nothing.  Behind it lies room for the initial row numbers.
  void *rb_block = nullptr;
  size_t rb_cap = 0;
  Ctx() = default;
  Ctx(const Ctx &) = delete;
  Ctx &operator=(const Ctx &) = delete;
  ~Ctx() {
    if (pending) (void)hipStreamSynchronize(st);      // (an error on the way: the block is not reused under a kernel)
    if (rb_block) tl_pinned.give(rb_block, rb_cap);   // a context lives and dies on one thread
  }
  bool pending = false;                    // a kernel that writes the report has been launched and not been waited for
  StepReport *report = nullptr;            // host address ...
  StepReport *report_dev = nullptr;        // ... and the same block as kernels see it
  int64_t *idx_host = nullptr;             // [k], page-locked, for at most kPinnedIdx clusters (NULL above)
  const int64_t *idx_dev_view = nullptr;
  bool sizes_known = false;                // report holds the empty clusters and the largest size of c.assign's clusters
  const int32_t *prev_in = nullptr;        // the caller's labels, checked and copied to prev when the step starts
  char *zblock = nullptr;                  // device: counters | flag | done | scal | cluster sizes (see alloc_common)
  size_t zbytes = 0;
  unsigned int *flag = nullptr, *done = nullptr;
  int32_t *change_start = nullptr;         // [finalize_blocks(n)]
  static constexpr int32_t kPinnedIdx = 65536;
  int alloc_readback() {
    const size_t off_idx = (sizeof(StepReport) + 63) & ~(size_t)63;
    const size_t want = off_idx + (k <= kPinnedIdx ? (size_t)k * sizeof(int64_t) : 0);
    rb_block = tl_pinned.take(want, &rb_cap);
    char *h = static_cast<char *>(rb_block);
    if (!h) return fail(SKM_EHIP, "hipHostMalloc failed for the step report");
    void *dv = nullptr;
    HIPCHK(hipHostGetDevicePointer(&dv, h, 0));
    report = reinterpret_cast<StepReport *>(h);
    report->seq = 0;
    report_dev = static_cast<StepReport *>(dv);
    if (k <= kPinnedIdx) {
      idx_host = reinterpret_cast<int64_t *>(h + off_idx);
      idx_dev_view = reinterpret_cast<const int64_t *>(static_cast<char *>(dv) + off_idx);
    }
    return SKM_OK;
  }
  // the last kernel of a step, and the wait for it (a step whose flag is set by then leaves labels and distances, which may
  // be the caller's arrays, as they are)
  int close_step(stamp_t *start = nullptr, stamp_t *end = nullptr) {
    FinalizeArgs f{best, prev_counts ? prev : nullptr, n, assign, dist, up.cnt, k, flag};
    f.seq = ++seq;
    f.done = done; f.obj_partial = obj_partial; f.change_start = change_start; f.scal = scal; f.report = report_dev;
    f.stamp = start; f.stamp_end = end;
    f.nscal = block_stats ? SC_COUNT : SC_ENTER;   // (the counters per block are zero otherwise)
    HIPCHK(launch_finalize_assign(f, st));
    pending = true;
    return SKM_OK;
  }
  // With `watch` the report is waited for, not the stream: what a fit does next is ordered behind the step on the stream, and the
  // runtime notices the end of a kernel 3 to 4 us after its last word has arrived (a fit of 20 000 x 128, eleven steps, 897 -> 866 us,
  // of 120 001 x 200, seven steps, 2200 -> 2170).  For half a millisecond: then the stream is asked, which also reports a failure.
  int wait_step() {
    if (watch) {
      const volatile unsigned int *word = &report->seq;
      const auto t0 = std::chrono::steady_clock::now();
      for (;;) {
        for (int i = 0; i < 64; ++i) {
          if (*word == seq) {
            std::atomic_thread_fence(std::memory_order_acquire);
            sizes_known = true;
            return SKM_OK;
          }
          __builtin_ia32_pause();
        }
        if (std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(500)) break;   // (`pending` stays: see the destructor)
      }
    }
    return wait_stream();
  }
  int wait_stream() {
    HIPCHK(hipStreamSynchronize(st));
    pending = false;
    sizes_known = true;
    return SKM_OK;
  }
  bool watch = false;                      // (set in a call that has its thread to itself, where waits spin)
  bool update_ahead = false;               // an update follows this step, and a small one may follow before its report is read
  int64_t ahead_most = 0;                  // it has, if at most this many labels changed (and any did)
  int64_t last_changed = 0;                // of the step before
  unsigned int seq = 0;                    // number of the last report asked for
  bool prev_counts = true;                 // changed points are counted against prev (false in the exact step)

  int alloc_bounds(stamp_t *stamp = nullptr) {
    HIPCHK(pool.get(&amax, (size_t)AM_COUNT + AM_ROTATION));
    if (!pool.count_only) HIPCHK(launch_fill_u32(amax, AM_COUNT + AM_ROTATION, 0u, st, stamp));
    xr_bound = amax + AM_XR;
    return SKM_OK;
  }
  int measure_xr() { return measure_absmax(Xr, ldx, n, ds, xr_bound, st); }
  // the words that a step counts into, cleared by the pass over the centroids that starts it
  void clear_with(CentroidPrep &a) const {
    a.clear = reinterpret_cast<unsigned int *>(zblock);
    a.clear_words = (int64_t)(zbytes / sizeof(unsigned int));
  }
  bool best_filled = false;    // best holds ~0 throughout (see launch_opening)
  int fill_best() {
    if (!best_filled) HIPCHK(launch_fill_u64(best, n, ~0ull, st));
    best_filled = false;
    return SKM_OK;
  }
  bool y_amax_valid = false;   // amax[AM_Y] bounds the current Y (the update writes it; other changes of Y clear this)
  int measure_y() {
    if (y_amax_valid) return SKM_OK;
    y_amax_valid = true;
    return measure_absmax(Y, ds, k, ds, amax + AM_Y, st);
  }

  int alloc_common(int64_t pair_budget, float dense_frac, bool need_update) {
    HIPCHK(pool.get(&Y, (size_t)k * ds));
    const int32_t nbmax = (ds - 16 + kBlockDims - 1) / kBlockDims + 1;
    HIPCHK(pool.get(&Ypdx, (size_t)nbmax * k * kBlockDims));
    HIPCHK(pool.get(&xnp, (size_t)(ds / 16) * n));
    HIPCHK(pool.get(&Xs, split_words(n, ds)));
    HIPCHK(pool.get(&Ys, split_words(k, ds)));
    HIPCHK(pool.get(&ynp, (size_t)nbmax * k));
    HIPCHK(pool.get(&ynorm, (size_t)k));
    HIPCHK(pool.get(&tau, (size_t)n));
    HIPCHK(pool.get(&dist, (size_t)n));
    HIPCHK(pool.get(&best, (size_t)n));
    HIPCHK(pool.get(&assign, (size_t)n));
    HIPCHK(pool.get(&prev, (size_t)n));
    // Every tile hands over at most emit_max pairs, so a chunk of rows needs tiles * emit_max slots.
    const int64_t tile_pairs = progressive_tile_pairs();
    if (!(dense_frac >= 0.f)) dense_frac = 0.f;
    if (dense_frac > 1.f) dense_frac = 1.f;
    emit_max = (unsigned int)std::llround((double)dense_frac * (double)tile_pairs);
    const int64_t per_tile = std::max<int64_t>(emit_max, 1);
    if (pair_budget <= 0) pair_budget = (int64_t)1 << 29;
    const int64_t col_tiles = progressive_tiles(1, k);
    int64_t row_tiles = std::max<int64_t>(pair_budget / (per_tile * col_tiles), 1);
    row_tiles = std::min<int64_t>(row_tiles, std::max<int64_t>(((1 << 24) - 1) / col_tiles, 1));  // launch size limit
    chunk_rows = std::min<int64_t>(row_tiles * 128, (n + 127) / 128 * 128);
    nchunks = (int32_t)((n + chunk_rows - 1) / chunk_rows);
    // each of the kSubLists parts must hold what the tiles of one XCD can hand over
    const int64_t tiles_chunk = progressive_tiles(std::min<int64_t>(chunk_rows, n), k);
    sub_cap = ((tiles_chunk + kSubLists - 1) / kSubLists) * per_tile;
    // the filtered iteration 1 lists a few candidates per point in the same list (if it ever overflows, the step is
    // redone with the full GEMM): room for 16 per point of a chunk in each of the eight parts
    // (the kernels behind the filter address a listed centroid's row with 32-bit byte offsets: not for a centroid table
    // of 2^30 words or more, where the steps simply run unfiltered)
    const bool may_screen = (screen_mode > 0 || (screen_mode == 0 && k >= 256)) &&
                            ((int64_t)k + 1) * split_ld(ds) < ((int64_t)1 << 30);
    if (may_screen) sub_cap = std::max<int64_t>(sub_cap, 16 * std::min<int64_t>(chunk_rows, n));
    pair_cap = sub_cap * kSubLists;
    if (pair_cap >= ((int64_t)1 << 32)) return fail(SKM_EINVAL, "pair_budget too large (must stay below 2^32 pairs)");
    HIPCHK(pool.get(&pairs, (size_t)pair_cap));
    ncounters = (size_t)nchunks * (kSubLists + 8) * kSubListStride;   // list fill counters, tile counters
    if (may_screen) {   // (unless forced: of no use with few centroids)
      // one bit per (row tile, centroid); at most one tile of listed columns per (row tile, column tile) of the chunk
      const int64_t nrt_chunk = (std::min<int64_t>(chunk_rows, n) + 127) / 128;
      HIPCHK(pool.get(&colmask, (size_t)nrt_chunk * 4 * (size_t)((k + 127) / 128)));
      HIPCHK(pool.get(&scr_cnt, (size_t)nrt_chunk));
      HIPCHK(pool.get(&scr_first, (size_t)nrt_chunk));
      HIPCHK(pool.get(&scr_ntiles, 2));   // the tile count, then a float scalar of the filter
      HIPCHK(pool.get(&scr_arow, (size_t)std::min<int64_t>(chunk_rows, n)));
      HIPCHK(pool.get(&scr_ycol, (size_t)k));
      HIPCHK(pool.get(&Xh, split_words(n, ds) / 2));
      HIPCHK(pool.get(&Yh, split_words(k, ds) / 2));
      HIPCHK(pool.get(&Yd, split_words(k, ds)));
      HIPCHK(pool.get(&scr_cols, (size_t)tiles_chunk * kListCols));
      HIPCHK(pool.get(&scr_widen, (size_t)kMaxBlocks + 1));
      HIPCHK(pool.get(&scr_tile_rt, (size_t)tiles_chunk));
      HIPCHK(pool.get(&scr_pos, (size_t)n));
    }
    // everything a step clears at its start is one block: counters | flag | ticket | step scalars | cluster sizes
    {
      const size_t nscal = (size_t)SC_COUNT * kStatReplicas;
      const size_t off_flag = ncounters * sizeof(unsigned int);
      const size_t off_scal = (off_flag + 2 * sizeof(unsigned int) + 7) & ~(size_t)7;
      const size_t off_cnt = off_scal + nscal * sizeof(unsigned long long);
      zbytes = off_cnt + sizeof(int32_t) * (size_t)k;
      HIPCHK(pool.get(&zblock, zbytes));
      if (zblock) {
        counters = reinterpret_cast<unsigned int *>(zblock);
        flag = reinterpret_cast<unsigned int *>(zblock + off_flag);
        done = flag + 1;
        scal = reinterpret_cast<unsigned long long *>(zblock + off_scal);
        up.cnt = reinterpret_cast<int32_t *>(zblock + off_cnt);
      }
      if (!pool.count_only)   // (a size query touches no device and no page-locked memory)
        if (int rc = alloc_readback()) return rc;
    }
    HIPCHK(pool.get(&ratio_dev, (size_t)kMaxBlocks + 1));
    HIPCHK(pool.get(&obj_partial, (size_t)(n + 1023) / 1024));   // at least finalize_blocks(m) for every m <= n
    HIPCHK(pool.get(&change_start, (size_t)(n + 1023) / 1024));
    if (need_update) {
      HIPCHK(pool.get(&up.off, (size_t)k + 1));
      HIPCHK(pool.get(&up.cursor, (size_t)k));
      HIPCHK(pool.get(&up.segoff, (size_t)k + 1));
      HIPCHK(pool.get(&up.order, (size_t)n));
      // (a batch of a host-resident fit may be shorter than n: the rule is asked again there)
      if (stable_order_applies(n, k)) HIPCHK(pool.get(&up.base, (size_t)stable_order_words(n, k)));
      up.max_segments = update_max_segments(n, k);
      HIPCHK(pool.get(&up.partial, (size_t)up.max_segments * ds));
      HIPCHK(pool.get(&split_dev, (size_t)3 * k + 2));   // (empty, donor) pairs | first split of every chain
      HIPCHK(pool.get(&touched, (size_t)k));
      // the incremental update is used while at most one point in eight changes its label
      HIPCHK(pool.get(&S, (size_t)k * ds));
      inc.capacity = 2 * (n / 8) + 2;
      inc.max_segments = update_max_segments(inc.capacity, k);
      HIPCHK(pool.get(&inc.ent_id, (size_t)inc.capacity));
      HIPCHK(pool.get(&inc.ent_lab, (size_t)inc.capacity));
      HIPCHK(pool.get(&inc.order, (size_t)inc.capacity));
      HIPCHK(pool.get(&inc.cnt, (size_t)k));
      HIPCHK(pool.get(&inc.off, (size_t)k + 1));
      HIPCHK(pool.get(&inc.cursor, (size_t)k));
      HIPCHK(pool.get(&inc.segoff, (size_t)k + 1));
      if (stable_order_applies(inc.capacity, k)) HIPCHK(pool.get(&inc.base, (size_t)stable_order_words(inc.capacity, k)));
      HIPCHK(pool.get(&inc.partial, (size_t)inc.max_segments * ds));
    }
    return SKM_OK;
  }
};

// Bytes that a context of this shape takes from its pool (alloc_bounds + alloc_common), counted without allocating.
size_t plan_common_bytes(int64_t n, int32_t d, int32_t k, int64_t pair_budget, float dense_frac, bool need_update) {
  Ctx t;
  t.pool.count_only = true;
  t.n = n; t.d = d; t.k = k;
  t.ds = (d + 15) / 16 * 16;
  if (t.alloc_bounds() != SKM_OK || t.alloc_common(pair_budget, dense_frac, need_update) != SKM_OK) return 0;
  return t.pool.counted;
}

// One device allocation for the whole workspace of a top-level call instead of some forty (3.4 ms of allocation and
// release per fit of 1M x 1536 become 0.8 ms).  Declared before the context, so that the context's pool carves from it.
// A nested call (a worker of the hierarchical fit, the steps of the sampled fit) finds an arena in place and adds none;
// whatever does not fit, or the whole workspace if this allocation fails, comes from hipMalloc as before.
struct CallArena {
  Arena arena;
  bool on = false;
  bool too_small = false;   // a caller's workspace that cannot hold `bytes`
  explicit CallArena(size_t bytes, void *lent = nullptr, int64_t lent_bytes = 0) {
    if (tl_arena || bytes == 0) return;
    if (lent) {
      // the caller's memory: aligned up to the 256-byte granule of the pools
      const uintptr_t a = (reinterpret_cast<uintptr_t>(lent) + 255) & ~(uintptr_t)255;
      const size_t lost = (size_t)(a - reinterpret_cast<uintptr_t>(lent));
      if (lent_bytes < 0 || (size_t)lent_bytes < bytes + lost) {
        too_small = true;
        return;
      }
      arena.lend(reinterpret_cast<void *>(a), (size_t)lent_bytes - lost);
      tl_arena = &arena;
      on = true;
      return;
    }
    if (arena.init(bytes) != hipSuccess) {
      (void)hipGetLastError();
      arena.base = nullptr;
      arena.cap = 0;
      return;
    }
    tl_arena = &arena;
    on = true;
  }
  ~CallArena() {
    if (on) tl_arena = nullptr;
  }
  void finished() { arena.keep = true; }   // the call has waited for its stream
  CallArena(const CallArena &) = delete;
  CallArena &operator=(const CallArena &) = delete;
};

// Host-clock readings of one call: entry, workspace ready, body done; the destructor (declared before the arena, so it
// runs after the arena's release) writes them to the caller's trace.
struct HostTimes {
  using clk = std::chrono::steady_clock;
  clk::time_point t0 = clk::now(), t_ws = t0, t_done = t0;
  skm_trace *tr = nullptr;
  bool done = false;
  static float ms(clk::time_point a, clk::time_point b) { return std::chrono::duration<float, std::milli>(b - a).count(); }
  void workspace_ready() { t_ws = clk::now(); }
  void body_done(skm_trace *t) {
    tr = t;
    t_done = clk::now();
    done = true;
  }
  ~HostTimes() {
    if (!tr || !done) return;
    const auto t1 = clk::now();
    tr->ms_host_alloc = ms(t0, t_ws);
    tr->ms_host_free = ms(t_done, t1);
    tr->ms_host_total = ms(t0, t1);
  }
};

// Upper bound of the device bytes one plain fit (or one assignment call) of this shape carves from its arena: the
// context's buffers, the rotated points and their regrouped copy, the rotation matrices and their generator, the ETR
// buffers.  What skm_workspace_bytes reports.
inline bool assign_groups(int64_t n, int32_t ds, int32_t k, int32_t screen_mode);
inline bool assign_groups_always(int32_t k);
// ... of one assignment call (assign_impl)
size_t assign_workspace_need(int64_t n, int32_t d, int32_t k, const skm_params &p) {
  const size_t ds0 = (size_t)((d + 15) / 16 * 16);
  const size_t plan = plan_common_bytes(n, d, k, p.pair_budget, p.dense_frac, false);
  if (!plan) return 0;
  const size_t grouping = assign_groups(n, (int32_t)ds0, k, p.screen) ? (size_t)n * ds0 * 4 + (size_t)n * 9 + (size_t)k * 20 + (size_t)threshold_class_words(n) * 4 + 4096 : 0;
  return plan + grouping + (size_t)n * ds0 * 4 + 10 * (size_t)d * ds0 * 4 + (size_t)d * 16384 + ((size_t)32 << 20);
}
int64_t sample_size(int64_t n, int32_t k, float frac) {
  const int64_t s = (int64_t)std::llround((double)frac * (double)n);
  return std::min<int64_t>(std::max<int64_t>(s, k), n);
}
// Sizes of the form through the one-product multiply (etr.hip).
struct GtPlan {
  bool on = false;
  int32_t ds = 0, ngroups = 0;
  int64_t nsel = 0, chunk = 0;
  unsigned int cap = 0;
  size_t bytes = 0;   // of the call's buffers
};
GtPlan gt_plan(int64_t n, int32_t d, int32_t nq, int32_t K);
size_t gt_full_bytes(int64_t n, int32_t nq);
size_t fit_workspace_need(int64_t n, int32_t d, int32_t k, const skm_params &p) {
  const size_t ds0 = (size_t)((d + 15) / 16 * 16);
  if (p.sample_frac > 0.f && p.sample_frac < 1.f) {
    // the sampled fit: all rows rotated (and a dense copy of them when d is no multiple of 16), the sample, the
    // centroids, and below them first the fit on the sample, then the assignment of all rows
    skm_params q = p;
    q.sample_frac = 0.f;
    const int64_t s = sample_size(n, k, p.sample_frac);
    const size_t a = fit_workspace_need(s, d, k, q), b = assign_workspace_need(n, d, k, q);
    if (!a || !b) return 0;
    return std::max(a, b) + (size_t)n * ds0 * 4 + (ds0 != (size_t)d ? (size_t)n * d * 4 : 0) + (size_t)s * (8 + (size_t)d * 4) +
           (size_t)k * (d + ds0) * 4 + (size_t)n * 4 + 10 * (size_t)d * ds0 * 4 + (size_t)d * 16384 + ((size_t)32 << 20);
  }
  const size_t plan = plan_common_bytes(n, d, k, p.pair_budget, p.dense_frac, true);
  if (!plan) return 0;
  // (threshold_class_words(n), 6 MiB at most, is in the last term: a workspace that a caller lends has the size that it had without)
  size_t need = plan + 2 * (size_t)n * ds0 * 4 + (size_t)n * 5 + 10 * (size_t)d * ds0 * 4 + (size_t)d * 16384 +
                (size_t)k * 16 + ((size_t)32 << 20);
  if (p.etr && p.nq > 0 && p.topk > 0) {
    const size_t nq = (size_t)p.nq;
    const GtPlan plan = gt_plan(n, d, p.nq, p.topk);   // (and, should a candidate list run over, the full form behind it)
    need += (plan.on ? plan.bytes : 0) + gt_full_bytes(n, p.nq) + nq * (size_t)p.topk * 8 + nq * (ds0 + d) * 4 +
            nq * 8 + nq * (size_t)k * 4 + (size_t)k * 4 + ((size_t)1 << 16);
  }
  return need;
}

struct StepStats {
  double objective = 0;
  int64_t survivors = 0, completed = 0, changed = 0, dense_dims = 0, dense_pair_blocks = 0;
  int64_t gather_pair_blocks = 0, gather_pairs = 0, screen_dims = 0, listed_tiles = 0;
  int64_t enter[SKM_MAX_BLOCKS] = {0};
  int32_t dprime = 0, nblocks = 0;
  bool pruned = false;  // false for the exact step of iteration 1
};

// Iteration 1 with the low-precision filter in front (screen.hip, exact mode): one fp16 product over all dimensions
// lists, for every point, the centroids that can be its nearest; the gather kernel takes their exact distances and the
// packed minimum is the exact nearest centroid (lowest index on ties).  A third of the matrix work of the full
// three-product GEMM; pays once there are enough centroids.
// c.best[i] = packed (squared distance over dims [0, K), centroid) of the centroid nearest to point i on those dims,
// exact (direct form, lowest index on ties): the one-product multiply over K dims lists the candidates, the gather
// kernel takes their distances.  K = ds: the nearest centroid; K = d': the incumbent of a step that comes without one.
// Clears the step's counters; clobbers ynorm, Ypdx, Ys / Yh, ratio_dev, tau; sets bit 0 of the step's flag word if the
// candidate list overflowed.
int filtered_nearest(Ctx &c, int32_t K, StageTimer &tm) {
  const int32_t nbK = (K + kBlockDims - 1) / kBlockDims;
  if (nbK > kMaxBlocks) return fail(SKM_EINTERNAL, "too many blocks");
  stamp_t *start = tm.mark(ST_NONE);
  if (!c.xnp_valid || !c.xh_valid) {
    // the points' split copy, its hi plane and their norms do not exist before the first pruned step: the pass that
    // writes them runs now (its thresholds, against centroid 0, are discarded)
    HIPCHK(launch_fill_u32(reinterpret_cast<unsigned int *>(c.prev), c.n, 0u, c.st));
    HIPCHK(launch_tau_init(c.Xr, c.ldx, c.n, c.ds, c.Y, c.ds, c.prev, c.tau, nullptr, c.st, c.xnp, c.Xs,
                           c.xr_bound, nullptr, nullptr, nullptr, c.Xh, nullptr, start));
    start = nullptr;
    c.xnp_valid = c.xh_valid = true;
  }
  // ||y[0 : K)||^2 and the block-major copy of the first K dimensions, zero filled behind them (the gather kernel
  // starts every pair at dimension 0 and is told that rows end at K)
  if (int rc = c.measure_y()) return rc;
  float ratio[kMaxBlocks + 1];
  for (int m = 0; m <= nbK; ++m) ratio[m] = 1.f;   // nothing is dropped on the way
  CentroidPrep cp{c.Y, c.ds, c.k, c.ds};
  cp.ynorm = c.ynorm; cp.dn = K;
  cp.dprime = 0; cp.nb = nbK; cp.Ypdx = c.Ypdx; cp.pdx_cols = K;
  cp.Ys = c.Ys; cp.Yh = c.Yh; cp.hi_dims = K; cp.y_absmax = c.amax + Ctx::AM_Y;
  cp.ratio_out = c.ratio_dev;
  cp.stamp = start;
  c.clear_with(cp);
  HIPCHK(launch_prep_centroids(cp, c.st, ratio, nbK + 1));
  if (int rc = c.fill_best()) return rc;
  unsigned int *rowmin = reinterpret_cast<unsigned int *>(c.tau);   // (no thresholds while this runs)
  HIPCHK(launch_fill_u32(rowmin, c.n, 0xffffffffu, c.st));
  for (int32_t ch = 0; ch < c.nchunks; ++ch) {
    const int64_t r0 = (int64_t)ch * c.chunk_rows;
    const int64_t rows = std::min<int64_t>(c.chunk_rows, c.n - r0);
    unsigned int *fill = c.counters + (size_t)ch * kSubLists * kSubListStride;
    ScreenLaunch sl{};
    sl.A = c.Xh + r0 * (split_ld(c.ds) / 2); sl.lda = split_ld(c.ds) / 2; sl.M = (int32_t)rows;
    sl.B = c.Yh; sl.ldb = split_ld(c.ds) / 2; sl.N = c.k;
    sl.a_absmax = c.xr_bound; sl.b_absmax = c.amax + Ctx::AM_Y;
    sl.ds = c.ds; sl.dprime = K; sl.ratio0 = 1.f;
    sl.tau = c.tau; sl.row_base = r0;
    sl.xn = c.xnp + (int64_t)(K / 16 - 1) * c.n;   // ||x[0 : K)||^2: row K / 16 - 1 of the prefix table
    sl.yn = c.ynorm;
    sl.arow = c.scr_arow; sl.ycol = c.scr_ycol;
    sl.colmask = c.colmask; sl.cnt = c.scr_cnt; sl.first = c.scr_first; sl.ntiles = c.scr_ntiles;
    sl.col_list = c.scr_cols; sl.tile_rt = c.scr_tile_rt;
    sl.scal = c.scal;
    sl.exact = 1; sl.rowmin = rowmin; sl.pairs = c.pairs; sl.pair_count = fill; sl.sub_capacity = (unsigned int)c.sub_cap;
    sl.overflow = c.flag;
    if (ch == 0) sl.stamp = tm.mark(ST_TAU);
    HIPCHK(launch_screen(sl, c.st));
    PruneArgs pa{c.pairs, fill, (unsigned int)c.sub_cap, c.Xr, c.ldx, c.n, c.Ypdx, c.k, 0, K, nbK, c.Y, c.ratio_dev,
                 c.best, c.scal, 0};
    // Rows that outgrow the Infinity Cache (256 MB) are read once for all of their candidates instead of once for each.  The
    // whole stage, list -> rows: 1M x 1536, k = 1024 5.71 -> 4.94 ms, k = 4096 18.65 -> 14.8, 1M x 768, k = 4096 9.10 -> 7.92, 100 000 x
    // 1024, k = 3000 914 -> 855 us, 200 000 x 400, k = 4000 1067 -> 943; but 120 001 x 208, k = 777 159 -> 164, 20 000 x 1536, k = 600
    // 112 -> 134, and 1M x 96, k = 800 622 -> 640 (two blocks of 64 dimensions a row).
    // (the buffers of the filter's lists are free in this form: two slots a point and column tile, four or eight in all)
    const int32_t slots = std::min<int32_t>(8, (int32_t)progressive_tiles(1, c.k) * (kListCols / 128)) & ~3;
    if (slots > 0 && K >= 128 && rows * K >= (int64_t)1 << 26) {
      RowPairsArgs rp{};
      rp.pairs = c.pairs; rp.count = fill; rp.sub_capacity = (unsigned int)c.sub_cap; rp.overflow = c.flag;
      rp.left_count = c.counters + ((size_t)c.nchunks * kSubLists + (size_t)ch * 8) * kSubListStride;
      rp.row_count = reinterpret_cast<unsigned int *>(c.scr_pos); rp.cand = c.scr_cols;
      rp.slots = slots;
      rp.rows = (int32_t)rows; rp.row_base = r0;
      rp.Xr = c.Xr; rp.ldx = c.ldx; rp.Ypdx = c.Ypdx; rp.k = c.k; rp.K = K; rp.nb = nbK;
      rp.best = c.best; rp.scal = c.scal;
      HIPCHK(launch_row_pairs(rp, c.st));
      pa.pairs = c.pairs + c.sub_cap / 2;
      pa.count = rp.left_count;
    }
    HIPCHK(launch_prune(pa, c.st));
  }
  return SKM_OK;
}

int step_exact_filtered(Ctx &c, StageTimer &tm, StepStats &ss) {
  if (int rc = filtered_nearest(c, c.ds, tm)) return rc;
  // the packed minima already hold the direct distances
  c.prev_counts = false;
  stamp_t *fin = tm.mark(ST_GEMM);
  int rc = c.close_step(fin, tm.mark(ST_TAU));
  c.prev_counts = true;
  if (rc) return rc;
  if ((rc = c.wait_step())) return rc;
  ss = StepStats();
  ss.gather_pair_blocks = (int64_t)c.report->scal[SC_GATHER_PB];
  ss.gather_pairs = (int64_t)c.report->scal[SC_GATHER_PAIRS];
  ss.screen_dims = (int64_t)c.report->scal[SC_SCREEN_DIMS];
  ss.objective = c.report->objective;
  ss.dprime = c.d;
  ss.changed = c.n;
  return SKM_OK;
}

// Iteration 1 of Algorithm 1: exact assignment over all dims.  Leaves assign, dist, cluster sizes.
int step_exact(Ctx &c, StageTimer &tm, StepStats &ss) {
  // Many centroids: the low-precision filter first, exact distances for the few candidates it leaves.  It also writes the
  // tables that the next step would write.  Iterations 1 and 2 together, product -> filter, for 1M points: k = 512 16.9 -> 16.2
  // ms at d = 1536 and 2.67 -> 2.53 at d = 100, k = 1024 27.1 -> 24.7, k = 2047 47.0 -> 41.0; 300 000 x 1024, k = 800 7.81 -> 7.25,
  // 200 000 x 79, k = 700 900 -> 770 us; 5000 x 768, k = 600 438 -> 458.  It would pay from 512 clusters on, but the line lies at
  // 2048: the two sides round a distance differently, so that the winners of ties to 1e-7 differ (1M x 1536, k = 1024: 1 to 9
  // points a fit, either side the nearer one to 64 bits about as often), and such a point may send a fit to another end.
  if (c.colmask && !c.exact_filter_off && (c.screen_mode > 0 || c.k >= 2048)) {
    if (int rc = step_exact_filtered(c, tm, ss)) return rc;
    if ((c.report->flag & 1u) == 0) {
      if (c.report->flag != 0) return fail(SKM_EINTERNAL, "a point was left without a centroid");
      return SKM_OK;
    }
    c.exact_filter_off = true;   // the candidate list overflowed (with seven or more candidates a point, in eight lists): the full GEMM instead
  }
  if (int rc = c.measure_y()) return rc;
  CentroidPrep cp{c.Y, c.ds, c.k, c.ds};
  cp.stamp = tm.mark(ST_NONE);
  cp.ynorm = c.ynorm; cp.dn = c.ds;
  cp.Ys = c.Ys; cp.y_absmax = c.amax + Ctx::AM_Y;
  c.clear_with(cp);
  HIPCHK(launch_prep_centroids(cp, c.st));
  HIPCHK(launch_fill_u64(c.best, c.n, ~0ull, c.st));
  GemmOperands g{c.Xr, c.ldx, (int32_t)c.n, c.Y, c.ds, c.k, c.ds};
  g.a_absmax = c.xr_bound; g.b_absmax = c.amax + Ctx::AM_Y;
  g.b_presplit = c.Ys; g.ldbs = split_ld(c.ds);
  HIPCHK(gemm_argmin(g, c.ynorm, c.best, c.st));
  // winners -> direct squared distances (also the objective of this step)
  HIPCHK(launch_tau_init(c.Xr, c.ldx, c.n, c.ds, c.Y, c.ds, nullptr, nullptr, c.best, c.st, nullptr, nullptr, nullptr,
                         nullptr, nullptr, nullptr, nullptr, c.flag, tm.mark(ST_GEMM)));
  c.prev_counts = false;
  int rc = c.close_step(nullptr, tm.mark(ST_TAU));
  c.prev_counts = true;
  if (rc) return rc;
  if ((rc = c.wait_step())) return rc;
  if (c.report->flag != 0) return fail(SKM_EINTERNAL, "a point was left without a centroid");
  ss = StepStats();
  ss.objective = c.report->objective;
  ss.dprime = c.d;
  ss.changed = c.n;
  return SKM_OK;
}

// Whether the points of a fit are regrouped (Ctx) with `left` steps to go, this one included.  The rewrite costs about as much as
// three threshold passes and saves a part of every later step.  With fewer than four steps there have to be many centroids, a quarter
// of a row tile's worth of points to each, and work; and unless there are very many centroids the step before has to have cut a
// fifth to 85 % of the pairs (`cut`): with less the next one multiplies every column whatever the order, with more its tiles are
// few.  Fits of four iterations (left = 3) without -> with it: 1M x 768, k = 2048, cut 0.54 38.3 -> 32.8 ms, 200 000 x 384 5.5 -> 4.7, 1M x
// 1536, k = 4096, cut 0.995 77.0 -> 70.1, 1M x 128, k = 3000, cut 0.97 11.3 -> 10.4; beyond the lines 1M x 768, k = 2048, cut 0.95 29.6 -> 30.9 and
// k = 512 21.8 -> 23.0, 1M x 128, k = 1366, cut 0.04 10.7 -> 10.9, 50 000 x 768, k = 3000 (17 points to a centroid) 3.16 -> 3.35, 100 000 x 64,
// k = 2048 1.52 -> 1.60.
inline bool regroup_pays(int32_t left, int64_t n, int32_t ds, int32_t k) {
  return left >= 4 || (left >= 2 && (int64_t)left * k >= 4096 && n >= 32 * (int64_t)k && (double)n * ds * k >= 1e11);
}
inline bool regroup_pays_behind(int32_t left, int32_t k, double cut) {
  return left >= 4 || (int64_t)left * k >= 8192 || (cut >= 0.20 && cut < 0.85);
}
// ... and again, once a twentieth of the labels has changed since, where the last step left enough to save: `listed` is the share of
// the tiles that it worked on (1: all).  Without a second regrouping -> with, of 432 fits of 6, 10 and 20 iterations (1M x 128 to 1536,
// 400 000 x 1024, 200 000 x 384, 50 000 x 768, 100 000 x 64; 256 to 4096 clusters, mixtures of 1024 to 16 384): 1M x 1536, k = 4096, cut
// 0.83 184 -> 176 ms; 20 iterations of 400 000 x 1024, k = 4096, cut 0.78 12 % faster, 1M x 768, k = 3000, cut 0.52 8, 200 000 x 384, k = 2048, cut
// 0.25 11, cut 0.89 with 61 % listed 4.  Beyond the lines 20 iterations of 1M x 768, k = 3000, cut 0.999 are 5 % slower, of 1M x 128, k = 4096,
// cut 0.998 4, of 1M x 1536, k = 4096, a quarter of the tiles listed, nine steps to go, 3, of 1M x 128, k = 512, cut 0.03, three times regrouped, 7.
inline bool regroup_pays_again(int32_t left, int64_t n, int32_t k, int64_t moved, double cut, double listed) {
  return 20 * moved >= n && cut >= 0.20 && cut < 0.98 && (double)left * k * (double)moved * listed >= 1500.0 * (double)n;
}
// Iterations >= 2 of Algorithm 1: initial threshold, progressive-pruning GEMM, gather kernel for the
// pairs of sparse tiles, argmin.  On entry c.prev holds the incumbents (c.assign is overwritten);
// have_prev = false seeds the incumbent with the centroid of smallest partial distance.
int step_pruned(Ctx &c, StageTimer &tm, int32_t dprime, double eps0, bool have_prev, StepStats &ss) {
  const int32_t nb = (c.d - dprime + kBlockDims - 1) / kBlockDims;
  if (nb > kMaxBlocks) return fail(SKM_EINTERNAL, "too many trailing blocks");
  bool found = false;   // the incumbents of a step that came without them are in c.prev
  bool sought = false;  // ... and were looked for through the first filter
  if (!have_prev && c.colmask && !c.exact_filter_off && (c.screen_mode > 0 || c.k >= 2048)) {
    // many centroids: the nearest centroid on the first d' dimensions through the low-precision filter (a third of
    // the matrix work of the three-product GEMM below); if its candidate list overflows, that GEMM runs after all
    sought = true;
    if (int rc = filtered_nearest(c, dprime, tm)) return rc;
    c.pending = true;
    HIPCHK(launch_finalize_assign(FinalizeArgs{c.best, nullptr, c.n, c.prev, nullptr, nullptr, c.k, c.flag}, c.st));
    HIPCHK(hipMemcpyAsync(&c.report->flag, c.flag, sizeof(unsigned int), hipMemcpyDeviceToHost, c.st));
    if (int rc = c.wait_stream()) return rc;
    c.sizes_known = false;
    if (c.report->flag == 0) found = true;
    else if (c.report->flag & 1u) c.exact_filter_off = true;
    else return fail(SKM_EINTERNAL, "a point was left without a centroid");
  }

  if (int rc = c.measure_y()) return rc;
  // Low-precision first filter: worth its pass over the front dimensions when most columns of a tile die at the
  // first test.  The previous step's prune fraction predicts that from below (the centroids only get better): the
  // step after one that cut half of the pairs cuts 85 to 99 % on the mixture workloads, and a wasted filter pass
  // costs a tenth of the poorly pruned step it precedes.
  // Behind the first test of a listed tile one product and widened tests will do where the gather kernel finishes what is
  // left (not where every test's count is asked for, nor with a hand-over share beyond an eighth).
  const bool deep = nb >= 3 && !c.block_stats && c.emit_max > 0 && c.emit_max <= (unsigned int)progressive_tile_pairs() / 8;
  // A step after one that cut a third to a half of the pairs cuts 70 to 95 % of them, spread over nearly all columns: there is
  // nothing for the filter to drop, but the tiles are through with their first test after an eighth of the dimensions and
  // multiply the rest in one product, so all columns are listed as they are.  Tiles and gather of the third step of a fit, dense ->
  // listed (behind the filter): 1M x 1536, k = 1024 7.80 -> 6.51 (6.68) ms, k = 4096 36.1 -> 28.2 (28.8), 600 000 x 1280, k = 2000 10.0 ->
  // 9.4 (9.8).  Where the lines lie (that step of 196 mixtures of 45 000 to 920 000 rows, 448 to 2040 dimensions, 256 to 4000 clusters):
  // behind a step that cut less than a third, from 1.39 times as fast to 0.63; with fewer than some 1200 tiles 1.16 to 0.94 (with 350
  // to 700 down to 0.77); where the last test but the one of the whole row comes before 95 % of it (a quarter of the tiles then
  // has too many pairs left and is done twice) 1.22 to 0.74; the 112 others 1.60 to 0.89, 110 of them 0.96 and more.
  const bool list_all = deep && c.screen_mode == 0 && c.last_prune_frac >= 0.33 && c.last_prune_frac < 0.50 &&
                        (double)(dprime + kBlockDims * (nb - 1)) >= 0.95 * c.d &&
                        ((c.n + 127) / 128) * (int64_t)((c.k + kListCols - 1) / kListCols) >= 1200;
  bool screen = c.colmask && nb > 0 &&
                (c.screen_mode > 0 || (c.screen_mode == 0 && (c.last_prune_frac >= 0.50 || list_all)));
  // A grouping that scatters and then orders the members of a cluster does so only up to a size (larger clusters keep
  // the order in which the scatter placed them, which depends on scheduling): with such a cluster the new order, and with
  // it the rounding of the results, would differ from run to run, so the points keep the input order.  The updates of a
  // fit of n >= 8 k points into at most 8192 clusters order every cluster by counting, whatever its size; the same limit
  // holds for them, which leaves the results of such fits what they were.
  // (in a fit the sizes came back with the previous step's scalars: no copy, no wait here)
  auto order_is_reproducible = [&]() { return c.max_cluster >= 0 && c.max_cluster <= update_sort_cap(); };
  // (not before one pruned step has run: the labels of iteration 1, assigned against the initial rows, group the points
  // far less usefully than those of iteration 2)
  const bool again = c.permuted;
  bool regroup = c.regroup_left > 0 && c.xnp_valid && c.Xr2 && have_prev && c.pruned_steps >= 1 &&
                 (again ? regroup_pays_again(c.regroup_left, c.n, c.k, c.moved, c.last_prune_frac, c.last_listed)
                        : regroup_pays(c.regroup_left, c.n, c.ds, c.k) && regroup_pays_behind(c.regroup_left, c.k, c.last_prune_frac)) &&
                 order_is_reproducible();
  // In a fit the points lie by quarters of their distance first, and by label inside a quarter: a point far from its centroid
  // keeps most columns of its row tile alive, so that the three quarters near theirs are better off without it.  The distances are
  // those of the step before (to the centroids as they were): there is no pass for them.  Column tiles a row tile lists, by label
  // -> by quarters, steps 3, 4 and 7: 1M x 1536, k = 4096 32 -> 32, 18.8 -> 14.8, 13.4 -> 11.1, 1M x 768, k = 4096 (steps 3 and 4)
  // 20.0 -> 12.2, 8.3 -> 6.5; halves and eighths of the distances list 2 to 15 % more.  Whole fits 201.9 -> 183.9 and 62.2 -> 59.3
  // ms, 300 000 x 512, k = 1500 9.93 -> 9.51, 150 000 x 256, k = 900 3.66 -> 3.57.  The nine small launches (30 to 60 us) are not
  // earned back below 2^34 products a step: 120 001 x 208, k = 777 (2^34.2) 2.21 -> 2.21, 40 000 x 384, k = 250 1.60 -> 1.59, 60 000 x
  // 448, k = 256 1.64 -> 1.66, 20 000 x 512, k = 100 1.40 -> 1.42.
  const bool by_quarters = regroup && (double)c.n * c.ds * c.k >= 0x1p34;
  // The thresholds of short rows are taken beside the pass over the centroids, where nothing else comes in between.
  const bool thresholds_done = have_prev && !c.prev_in && !c.group_now && !regroup && c.tau_kept == Ctx::KEPT_NONE && c.xnp_valid &&
                               !(screen && !c.xh_valid) && c.ds <= 256;
  // theta ratio at checkpoint m: t_m = min(d, d' + 64 m) dimensions seen
  float ratio[kMaxBlocks + 1];
  for (int m = 0; m <= nb; ++m) ratio[m] = (float)theta_ratio(c.d, std::min(c.d, dprime + kBlockDims * m), eps0);
  {
    CentroidPrep cp{c.Y, c.ds, c.k, c.ds};
    cp.dprime = dprime; cp.nb = nb; cp.Ypdx = c.Ypdx; cp.ynp = c.ynp;
    if (!have_prev && !found) { cp.ynorm = c.ynorm; cp.dn = dprime; }   // (for the product below)
    cp.Ys = c.Ys; cp.Yh = screen ? c.Yh : nullptr; cp.hi_dims = dprime; cp.Yd = screen ? c.Yd : nullptr; cp.y_absmax = c.amax + Ctx::AM_Y;
    cp.ratio_out = c.ratio_dev;
    cp.stamp = tm.mark(sought ? ST_GEMM : ST_NONE);   // (the search for the incumbents ends here)
    c.clear_with(cp);
    const ShortThresholds t{c.Xr, c.ldx, c.n, c.prev, c.tau, c.best};
    HIPCHK(launch_prep_centroids(cp, c.st, ratio, nb + 1, thresholds_done ? &t : nullptr));
  }
  bool from_keys = false;   // the incumbents are the low halves of c.best
  stamp_t *tau_stamp = nullptr;
  if (!have_prev && !found) {
    if (int rc = c.fill_best()) return rc;
    GemmOperands g0{c.Xr, c.ldx, (int32_t)c.n, c.Y, c.ds, c.k, dprime};
    g0.a_absmax = c.xr_bound; g0.b_absmax = c.amax + Ctx::AM_Y;
    g0.b_presplit = c.Ys; g0.ldbs = split_ld(c.ds);
    HIPCHK(gemm_argmin(g0, c.ynorm, c.best, c.st));
    if (c.group_now) {
      HIPCHK(launch_finalize_assign(FinalizeArgs{c.best, nullptr, c.n, c.prev, nullptr, nullptr, c.k, c.flag}, c.st));
    } else {
      from_keys = true;   // the threshold pass unpacks them
    }
    tau_stamp = tm.mark(ST_GEMM);
  } else if (have_prev && c.prev_in) {
    HIPCHK(launch_copy_labels(c.prev_in, c.n, c.k, c.prev, c.flag, c.st));
  }
  bool by_threshold = false;   // the new order follows the thresholds before the labels
  if (c.group_now && !c.permuted && c.Xr2) {
    // A step on its own (no update before it left an order): the points are grouped by the incumbents they come with
    // (or were just given above), so that a row tile holds the points of one or two clusters and the first filter has
    // columns to drop.  One read-back of the group sizes decides whether the order is reproducible; with them comes
    // whether the thresholds of a sample have a tail.
    HIPCHK(launch_threshold_sample(c.Xr, c.ldx, c.n, c.ds, c.Y, c.ds, c.prev, c.tau, (int32_t *)c.dist, c.class_ws, c.grp_cnt + c.k, c.st));
    regroup = assign_groups_always(c.k);
    if (!regroup) {   // (asked first: the grouping is 3 to 6 % of a step that does not use it)
      int32_t above = 0;
      HIPCHK(hipMemcpyAsync(&above, c.grp_cnt + c.k, sizeof(int32_t), hipMemcpyDeviceToHost, c.st));
      HIPCHK(hipStreamSynchronize(c.st));
      regroup = thresholds_have_tail(c.n, above);
      if (!regroup && c.screen_mode == 0) screen = false;
    }
    if (regroup) {
      HIPCHK(launch_group_order(c.prev, c.n, c.k, c.grp_cnt, c.up.off, c.up.cursor, c.up.segoff, c.up.order, nullptr, c.st));
      std::vector<int32_t> sizes((size_t)c.k + 1);
      HIPCHK(hipMemcpyAsync(sizes.data(), c.grp_cnt, sizeof(int32_t) * ((size_t)c.k + 1), hipMemcpyDeviceToHost, c.st));
      HIPCHK(hipStreamSynchronize(c.st));
      c.max_cluster = *std::max_element(sizes.begin(), sizes.end() - 1);
      by_threshold = thresholds_have_tail(c.n, sizes.back());
      regroup = order_is_reproducible();
      if (!regroup && !assign_groups_always(c.k) && c.screen_mode == 0) screen = false;
    }
    c.group_now = false;
  }
  if (regroup) {
    if (c.regroup_left > 0 && !c.order_fresh)   // (the last update did not need the whole order)
      HIPCHK(launch_group_order(c.prev, c.n, c.k, c.inc.cnt, c.up.off, c.up.cursor, c.up.segoff, c.up.order, c.up.base, c.st));
    // this pass reads every point anyway: it writes them back grouped by cluster (see Ctx)
    // Inside a cluster that spans several row tiles the points follow the signs of their first four dimensions, then
    // their index: which points of a cluster share a tile matters (measured: -3 % on a fit with 1000 points per
    // cluster, nothing to gain where a cluster is smaller than a tile).
    // The order is made between up.order and `other`; pos_to_id is still in use where the points have been regrouped before (best
    // is free until the pass below writes this step's keys: it must not be where the order ends up).
    int32_t *other = again ? reinterpret_cast<int32_t *>(c.best) : c.pos_to_id;
    if (c.n / c.k >= 128)
      HIPCHK(launch_suborder(c.Xr, c.ldx, c.n, c.k, c.up.off, c.up.order, c.subkey, other, c.st));
    else
      HIPCHK(hipMemcpyAsync(other, c.up.order, sizeof(int32_t) * (size_t)c.n, hipMemcpyDeviceToDevice, c.st));
    int32_t *order = c.up.order;
    if (by_threshold) {
      // A step on its own takes its thresholds once more, in front of the order that they decide (1.2 of 41 ms at 2.5M x 384):
      // its incumbents are as old as the caller's, or come from the front dimensions alone.
      HIPCHK(launch_tau_init(c.Xr, c.ldx, c.n, c.ds, c.Y, c.ds, c.prev, c.tau, nullptr, c.st));
      HIPCHK(launch_threshold_classes(c.tau, c.n, 0, other, (int32_t *)c.dist, c.assign, c.class_ws, order, c.st));
    } else if (by_quarters) {
      HIPCHK(launch_threshold_classes(c.dist, c.n, 4, other, (int32_t *)c.tau, c.assign, c.class_ws, order, c.st));
    } else if (again) {
      HIPCHK(hipMemcpyAsync(order, other, sizeof(int32_t) * (size_t)c.n, hipMemcpyDeviceToDevice, c.st));
    } else {
      order = other;
    }
    HIPCHK(launch_tau_init(c.Xr, c.ldx, c.n, c.ds, c.Y, c.ds, c.prev, c.tau, c.best, c.st, c.xnp, c.Xs,
                           c.xr_bound, order, c.Xr2, c.assign, c.Xh, nullptr, tau_stamp));
    std::swap(c.prev, c.assign);   // the incumbents in the new order; the other buffer receives this step's labels
    if (c.point_keys) HIPCHK(launch_remap_key_ids(c.point_keys, c.n_point_keys, order, c.n, c.assign, c.st));
    if (again) {
      HIPCHK(launch_compose(c.pos_to_id, order, c.n, c.assign, c.st));
      HIPCHK(hipMemcpyAsync(c.pos_to_id, c.assign, sizeof(int32_t) * (size_t)c.n, hipMemcpyDeviceToDevice, c.st));
    } else if (order != c.pos_to_id) {
      std::swap(c.pos_to_id, c.up.order);   // (up.order is scratch until the next full update rebuilds it)
    }
    std::swap(c.Xr_own, c.Xr2);   // the rows as they lay are room for the next time (NULL where they were the caller's: there is none)
    c.Xr = c.Xr_own;
    c.ldx = c.ds;
    c.moved = 0;
    c.permuted = true;
    c.xh_valid = c.Xh != nullptr;
  } else if (thresholds_done) {
    // (already)
  } else if (have_prev && c.tau_kept != Ctx::KEPT_NONE && c.xnp_valid && !(screen && !c.xh_valid)) {
    HIPCHK(launch_tau_kept(c.Xr, c.ldx, c.n, c.ds, c.Y, c.ds, c.prev, c.tau_kept == Ctx::KEPT_ALL ? nullptr : c.touched, c.tau, c.best,
                           c.st, tau_stamp));
  } else {
    // The first pruned step of a context also writes the tables that depend on the points only.  The plane of hi halves
    // is left out where this step does not read it and a regrouping pass, which writes all of them again, is likely to
    // come before a step that does (3 of 16 GB of that pass at 1M x 1536); if it does not come, the first step that
    // needs the plane writes the tables once more.
    const bool tables = !c.xnp_valid || (screen && !c.xh_valid);
    uint32_t *xh = tables && (screen || !c.Xr2) ? c.Xh : nullptr;
    HIPCHK(launch_tau_init(c.Xr, c.ldx, c.n, c.ds, c.Y, c.ds, from_keys ? nullptr : c.prev, c.tau, c.best, c.st,
                           tables ? c.xnp : nullptr, tables ? c.Xs : nullptr, c.xr_bound, nullptr,
                           nullptr, from_keys ? c.prev : nullptr, xh, c.flag, tau_stamp));
    if (tables) c.xh_valid = xh != nullptr;
  }
  c.tau_kept = Ctx::KEPT_NONE;
  c.order_fresh = false;
  c.xnp_valid = true;
  stamp_t *border = tm.mark(ST_TAU);   // for the kernel that comes next
  for (int32_t ch = 0; ch < c.nchunks; ++ch) {
    const int64_t r0 = (int64_t)ch * c.chunk_rows;
    const int64_t rows = std::min<int64_t>(c.chunk_rows, c.n - r0);
    ProgArgs g{};
    g.A = c.Xs + r0 * split_ld(c.ds); g.lda = split_ld(c.ds); g.M = (int32_t)rows;
    g.B = c.Ys; g.ldb = split_ld(c.ds); g.N = c.k;
    g.a_absmax = c.xr_bound; g.b_absmax = c.amax + Ctx::AM_Y;
    g.ds = c.ds; g.d = c.d; g.dprime = dprime; g.nb = nb;
    g.ratio = c.ratio_dev; g.tau = c.tau; g.prev = c.prev; g.row_base = r0;
    g.xnp = c.xnp; g.xn_stride = c.n; g.ynp = c.ynp;
    unsigned int *fill = c.counters + (size_t)ch * kSubLists * kSubListStride;
    g.tile_counter = c.counters + ((size_t)c.nchunks * kSubLists + (size_t)ch * 8) * kSubListStride;
    g.pairs = c.pairs; g.pair_count = fill; g.sub_capacity = (unsigned int)c.sub_cap;
    g.overflow = c.flag; g.emit_max = c.emit_max;
    g.best = c.best; g.scal = c.scal; g.block_stats = c.block_stats ? 1 : 0;
    if (screen) {
      ScreenLaunch sl{};
      sl.A = c.Xh + r0 * (split_ld(c.ds) / 2); sl.lda = split_ld(c.ds) / 2; sl.M = g.M;
      sl.B = c.Yh; sl.ldb = split_ld(c.ds) / 2; sl.N = g.N;
      sl.a_absmax = g.a_absmax; sl.b_absmax = g.b_absmax;
      sl.ds = c.ds; sl.dprime = dprime; sl.ratio0 = ratio[0];
      sl.tau = c.tau; sl.row_base = r0;
      sl.xn = c.xnp + (int64_t)(dprime / 16 - 1) * c.n;
      sl.yn = c.ynp;
      if (deep) { sl.ynp = c.ynp; sl.nb = nb; sl.widen = c.scr_widen; }
      sl.arow = c.scr_arow; sl.ycol = c.scr_ycol;
      sl.colmask = c.colmask; sl.cnt = c.scr_cnt; sl.first = c.scr_first; sl.ntiles = c.scr_ntiles;
      sl.col_list = c.scr_cols; sl.tile_rt = c.scr_tile_rt; sl.prev = c.prev; sl.list_pos = c.scr_pos;
      sl.scal = c.scal;
      sl.all = list_all ? 1 : 0;
      sl.stamp = border;
      HIPCHK(launch_screen(sl, c.st));
      g.tile_rt = c.scr_tile_rt; g.col_list = c.scr_cols; g.ntiles = c.scr_ntiles; g.prev = c.scr_pos;
      if (deep) {
        // Whole calls in ms: a step of 2.5M x 384, k = 32 768 | of 600 000 x 1536, k = 10 000 | a fit of 1M x 1536, k = 4096,
        // ten iterations.  With deep_max at a quarter 110.3 | 45.7 | 241.7, three products throughout 187 | 59.1 | 247.3.
        //   emit_first (share of emit_max): flat from 2/16 to 8/16, all of it 118.0 | 47.9 | 241.6
        //   emit_deep: 6 110.5 | 45.6 | 246.5, 12 110.4 | 45.5 | 243.6, 48 110.4 | 46.1 | 242.4, 96 111.1 | 48.6 | 251.4
        //   deep_stride: 1 119.5 | 47.3 | 245.0, 2 113.7 | 46.0 | 242.0, 6 107.6 | 45.5 | 242.0 (1M x 768, k = 4096 93.4 -> 95.2)
        //   deep_max: 1/16 143.9 | 55.4 | 264.6, 1/8 123.7 | 49.5 | 253.4, 1/4 as it was, 1/2 105.8 | 44.3 | 239.8, no limit 104.4 | 44.2 |
        //   239.5; but half of it where poor incumbents are all there is, whose tiles are done twice (500 000 x 384 on the sphere
        //   against 6000 centroids, no incumbents 15.6, no limit 18.1 ms, random ones 14.6, 16.7).  The incumbents of a fit, and those
        //   of a caller whose thresholds have a tail, are right for the most part: the tiles of the tail, most of whose pairs are
        //   alive until the last tests, end there (the step against 32 768 centroids with its points in the order of
        //   their thresholds 36.1 -> 29.7, 1M x 384 against 8000, every seventh incumbent random 18.4 -> 16.2; the fit 179.5 -> 178.2)
        g.deep = 1;
        g.Ah = sl.A; g.Bh = c.Yd; g.widen = c.scr_widen;
        g.emit_first = c.emit_max * 5 / 16;
        g.emit_deep = 24;
        g.deep_stride = 3;
        g.deep_max = (unsigned int)progressive_tile_pairs() / (have_prev && (by_threshold || !c.single_step) ? 1 : 2);
      }
    }
    if (!screen) g.stamp = border;
    HIPCHK(launch_progressive(g, c.st));
    border = tm.mark(ST_GEMM);
    if (c.emit_max > 0) {
      PruneArgs pa{c.pairs, fill, (unsigned int)c.sub_cap, c.Xr, c.ldx, c.n, c.Ypdx, c.k, dprime, c.ds, nb, c.Y, c.ratio_dev,
                   c.best, c.scal, c.block_stats ? 1 : 0};
      pa.stamp = border;
      HIPCHK(launch_prune(pa, c.st));
      border = tm.mark(ST_PRUNE);
    }
  }
  if (int rc = c.close_step(border, tm.mark(ST_TAU))) return rc;
  // An update in which few points moved follows at once, and runs while the host takes the report: a fit of 20 000 x 128 into 100
  // clusters, eleven steps, 921 -> 880 us, of 120 001 x 200, seven steps, 2250 -> 2236.  Not where the step before says that it will
  // be another form: the workgroups that find nothing to do are not free with many clusters.
  c.ahead_most = 0;
  if (c.update_ahead && c.S_valid) {
    const int64_t most = update_ahead_most(c.ds, c.k, c.inc.capacity);
    if (most > 0 && c.last_changed > 0 && c.last_changed <= 4 * most) {
      const UpdateAhead a{c.scal + SC_CHANGED, c.flag, most};
      HIPCHK(launch_update_ahead(c.Xr, c.ldx, c.n, c.ds, c.assign, c.prev, c.change_start, c.k, c.up, c.inc, c.S, c.Y, c.ds, a, c.st,
                                 c.amax + Ctx::AM_Y));
      c.ahead_most = most;
    }
  }
  if (int rc = c.wait_step()) return rc;
  const unsigned int step_flag = c.report->flag;
  if (step_flag & 4u) return fail(SKM_EINVAL, "assignment label outside [0, k)");
  if (step_flag & 1u) return fail(SKM_EOVERFLOW, "the hand-over list of the dense tiles overflowed");
  if (step_flag != 0) return fail(SKM_EINTERNAL, "a point was left without a centroid");
  const unsigned long long *scal_h = c.report->scal;
  ss = StepStats();
  ss.survivors = (int64_t)scal_h[SC_SURVIVORS];
  ss.completed = (int64_t)scal_h[SC_COMPLETED];
  ss.changed = c.last_changed = (int64_t)scal_h[SC_CHANGED];
  ss.dense_dims = (int64_t)scal_h[SC_DENSE_DIMS];
  ss.dense_pair_blocks = (int64_t)scal_h[SC_DENSE_PB];
  ss.gather_pair_blocks = (int64_t)scal_h[SC_GATHER_PB];
  ss.gather_pairs = (int64_t)scal_h[SC_GATHER_PAIRS];
  ss.screen_dims = (int64_t)scal_h[SC_SCREEN_DIMS];
  ss.listed_tiles = (int64_t)scal_h[SC_LISTED_TILES];
  c.last_prune_frac = c.k > 1 ? 1.0 - (double)ss.survivors / ((double)c.n * (double)(c.k - 1)) : -1.0;
  c.last_listed = ss.listed_tiles > 0 ? (double)ss.listed_tiles / ((double)((c.n + 127) / 128) * (double)((c.k + 127) / 128)) : 1.0;
  ++c.pruned_steps;
  if (c.block_stats)
    for (int m = 0; m < std::min<int>(nb, SKM_MAX_BLOCKS); ++m) ss.enter[m] = (int64_t)scal_h[SC_ENTER + (size_t)m];
  ss.objective = c.report->objective;
  ss.dprime = dprime;
  ss.nblocks = nb;
  ss.pruned = true;
  return SKM_OK;
}

// Update + split of empty clusters (Section 3.2).  c.up.cnt must hold the cluster sizes of c.assign.
// `changed` = points whose label differs from c.prev (c.n after the exact step).  While few points move, the cluster
// sums of the previous update are corrected by the rows that joined and left instead of being recomputed from all
// points (full = true forces the recomputation).
int split_empty(Ctx &c, Rng &split_rng, float split_eps, int64_t *nempty_out);
int step_update(Ctx &c, Rng &split_rng, float split_eps, int64_t *nempty_out, int64_t changed, bool full) {
  bool fresh = false;   // up.order rebuilt from the labels of this step
  if (!full && c.S_valid && changed == 0) {
    // no point changed its cluster: sums, sizes and therefore the means are those of the previous update.  If that
    // update was followed by a split, the donor's row still holds its perturbed copy: Algorithm 1's update puts the
    // mean of its members back before the next split, so the means are rewritten from the sums.
    ++c.inc_updates;
    if (c.split_last) {
      HIPCHK(launch_means_from_sums(c.S, c.up.cnt, c.k, c.ds, c.Y, c.ds, c.amax + Ctx::AM_Y, c.st));
    }
  } else if (!full && c.S_valid && 2 * changed <= c.inc.capacity - 2) {
    ++c.inc_updates;
    if (changed > c.ahead_most)   // (else it has run, see step_pruned)
      HIPCHK(launch_update_incremental(c.Xr, c.ldx, c.n, c.ds, c.assign, c.prev, changed, c.change_start, c.k, c.up, c.inc,
                                       c.S, c.Y, c.ds, c.st, c.amax + Ctx::AM_Y));
  } else {
    HIPCHK(launch_update(c.Xr, c.ldx, c.n, c.ds, c.assign, c.k, c.up, c.Y, c.ds, c.st, c.S, c.amax + Ctx::AM_Y, 0,
                         c.sizes_known ? c.report->largest : -1));
    c.S_valid = true;
    fresh = true;
  }
  c.order_fresh = fresh;
  c.y_amax_valid = true;
  const bool split_before = c.split_last;
  if (int rc = split_empty(c, split_rng, split_eps, nempty_out)) return rc;
  // A cluster that no point joined or left has the centroid it had, bit by bit (unless one of the last two splits moved it).
  // Marking the others is a launch more: where the thresholds are a pass of some length, and at most a quarter to a half of the
  // clusters can be touched.
  c.tau_kept = Ctx::KEPT_NONE;
  if (!full && !fresh && !split_before && !c.split_last && c.ds <= kTauKeptMaxDims) {
    if (changed == 0) {
      c.tau_kept = Ctx::KEPT_ALL;
    } else if (4 * changed <= c.k && c.n * c.ds >= ((int64_t)1 << 24)) {
      HIPCHK(launch_mark_touched(c.inc.ent_lab, (int32_t)(2 * changed), c.k, c.touched, c.st));
      c.tau_kept = Ctx::KEPT_UNTOUCHED;
    }
  }
  return SKM_OK;
}

// Empty clusters after an update (Section 3.2): c.up.cnt holds the cluster sizes, and the step's report (if sizes_known)
// how many of them are zero and the largest.
int split_empty(Ctx &c, Rng &split_rng, float split_eps, int64_t *nempty_out) {
  // the report of the step has said whether there are any (neither update changes the sizes); the sizes themselves are
  // fetched only then
  *nempty_out = 0;
  c.split_last = false;
  std::vector<int32_t> cnt;
  if (!c.sizes_known || c.report->nempty > 0) {
    cnt.resize((size_t)c.k);
    HIPCHK(hipMemcpyAsync(cnt.data(), c.up.cnt, sizeof(int32_t) * (size_t)c.k, hipMemcpyDeviceToHost, c.st));
    HIPCHK(hipStreamSynchronize(c.st));
    for (int32_t v : cnt) *nempty_out += (v == 0);
    c.max_cluster = *std::max_element(cnt.begin(), cnt.end());
  } else {
    c.max_cluster = c.report->largest;   // of the labels the update just used (a split below moves a centroid, no label)
  }
  c.sizes_known = false;
  if (*nempty_out > 0) {
    // empty clusters in increasing index; donor drawn with probability proportional to its size
    // among clusters of at least two points; the donor's points are shared floor(n/2) / rest.
    // The draw "first cluster whose cumulative weight exceeds r" runs on a Fenwick tree over the weights
    // (size if >= 2, else 0): O(log k) per empty cluster instead of a pass over all sizes.
    const int32_t k = c.k;
    std::vector<uint64_t> fen((size_t)k + 1, 0);
    auto weight = [](int32_t v) { return v >= 2 ? (uint64_t)v : 0ull; };
    for (int32_t j = 0; j < k; ++j) fen[(size_t)j + 1] = weight(cnt[(size_t)j]);
    for (int32_t j = 1; j <= k; ++j) {
      const int32_t up = j + (j & -j);
      if (up <= k) fen[(size_t)up] += fen[(size_t)j];
    }
    uint64_t total = 0;
    for (int32_t v : cnt) total += weight(v);
    auto fen_add = [&](int32_t j, int64_t delta) {
      for (int32_t i = j + 1; i <= k; i += i & -i) fen[(size_t)i] = (uint64_t)((int64_t)fen[(size_t)i] + delta);
    };
    int32_t top = 1;
    while ((top << 1) <= k) top <<= 1;
    auto fen_find = [&](uint64_t r) {   // smallest j with weight(0) + ... + weight(j) > r   (r < total)
      int32_t pos = 0;
      for (int32_t step = top; step > 0; step >>= 1)
        if (pos + step <= k && fen[(size_t)(pos + step)] <= r) {
          pos += step;
          r -= fen[(size_t)pos];
        }
      return pos;
    };
    std::vector<int32_t> pairs;
    for (int32_t e = 0; e < k; ++e) {
      if (cnt[(size_t)e] != 0) continue;
      if (total == 0) continue;
      const uint64_t r = split_rng.next() % total;
      const int32_t donor = fen_find(r);
      const int32_t give = cnt[(size_t)donor] / 2, keep = cnt[(size_t)donor] - give;
      const int64_t dd = (int64_t)weight(keep) - (int64_t)weight(cnt[(size_t)donor]);
      const int64_t de = (int64_t)weight(give);
      fen_add(donor, dd);
      fen_add(e, de);
      total = (uint64_t)((int64_t)total + dd + de);
      cnt[(size_t)e] = give;
      cnt[(size_t)donor] = keep;
      pairs.push_back(e);
      pairs.push_back(donor);
    }
    if (!pairs.empty()) {
      // Splits that share no cluster commute: they are grouped into chains (connected components of the clusters they
      // touch, in order of first appearance, every chain keeping the order above) and the device applies the chains
      // side by side.
      const size_t ns = pairs.size() / 2;
      std::vector<int32_t> parent((size_t)k);
      for (int32_t j = 0; j < k; ++j) parent[(size_t)j] = j;
      auto root = [&](int32_t v) {
        while (parent[(size_t)v] != v) v = parent[(size_t)v] = parent[(size_t)parent[(size_t)v]];
        return v;
      };
      for (size_t q = 0; q < ns; ++q) {
        const int32_t a = root(pairs[2 * q]), b = root(pairs[2 * q + 1]);
        if (a != b) parent[(size_t)a] = b;
      }
      std::vector<int32_t> chain_of((size_t)k, -1), chain(ns), len;
      for (size_t q = 0; q < ns; ++q) {
        const int32_t r0 = root(pairs[2 * q]);
        if (chain_of[(size_t)r0] < 0) {
          chain_of[(size_t)r0] = (int32_t)len.size();
          len.push_back(0);
        }
        chain[q] = chain_of[(size_t)r0];
        ++len[(size_t)chain[q]];
      }
      const size_t nchain = len.size();
      // upload: [2 ns] pairs sorted by chain | at word 2 k: [nchain + 1] first split of every chain
      std::vector<int32_t> up((size_t)2 * k + nchain + 1, 0);
      std::vector<int32_t> cursor(nchain + 1, 0);
      for (size_t q = 0; q < nchain; ++q) cursor[q + 1] = cursor[q] + len[q];
      for (size_t q = 0; q <= nchain; ++q) up[(size_t)2 * k + q] = cursor[q];
      for (size_t q = 0; q < ns; ++q) {
        const int32_t at = cursor[(size_t)chain[q]]++;
        up[(size_t)2 * at] = pairs[2 * q];
        up[(size_t)2 * at + 1] = pairs[2 * q + 1];
      }
      HIPCHK(hipMemcpyAsync(c.split_dev, up.data(), sizeof(int32_t) * up.size(), hipMemcpyHostToDevice, c.st));
      HIPCHK(launch_split(c.Y, c.ds, c.d, c.split_dev, c.split_dev + (size_t)2 * k, (int32_t)nchain, split_eps, c.st));
      c.y_amax_valid = false;
      c.split_last = true;
      HIPCHK(hipStreamSynchronize(c.st));  // `up` must outlive the copy
    }
  }
  return SKM_OK;
}

void fill_row(skm_trace_row &r, const StepStats &ss, int64_t n, int32_t k, int64_t nempty, double recall) {
  std::memset(&r, 0, sizeof(r));
  r.objective = ss.objective;
  r.prune_frac = (ss.pruned && k > 1) ? 1.0 - (double)ss.survivors / ((double)n * (double)(k - 1)) : 0.0;
  r.recall = recall;
  r.survivors = ss.survivors;
  r.completed = ss.completed;
  r.changed = ss.changed;
  r.dense_dims = ss.dense_dims;
  r.dense_pair_blocks = ss.dense_pair_blocks;
  r.gather_pair_blocks = ss.gather_pair_blocks;
  r.gather_pairs = ss.gather_pairs;
  r.screen_dims = ss.screen_dims;
  r.listed_tiles = ss.listed_tiles;
  r.nempty = nempty;
  r.dprime = ss.dprime;
  r.nblocks = ss.nblocks;
  for (int m = 0; m < SKM_MAX_BLOCKS; ++m) r.enter[m] = ss.enter[m];
}
// stage times of step q into its row (after the stream has been waited for)
void fill_times(skm_trace_row &r, const StageTimer &tm, size_t q) {
  float ms[ST_COUNT], total;
  tm.collect(q, ms, &total);
  r.ms_tau = ms[ST_TAU];
  r.ms_gemm = ms[ST_GEMM];
  r.ms_prune = ms[ST_PRUNE];
  r.ms_update = ms[ST_UPDATE];
  r.ms_etr = ms[ST_ETR];
  r.ms_step = total;
}

// Rotation buffers: Rp = R padded to row stride ds, Rtp = R^T padded likewise (both d rows).
struct Rot {
  float *Rp = nullptr, *Rtp = nullptr;
  static constexpr int kSlots = 8;
  unsigned int *amax = nullptr;   // [0] max |R|, the others magnitude bounds of the inputs of the products, one after the other
  int used = 1;
  uint32_t *Rs = nullptr;         // workspace for the split-fp16 copy of R^T (tall rotations)
  int alloc_bounds(Pool &pool, hipStream_t st) {
    if (amax) return SKM_OK;
    HIPCHK(pool.get(&amax, (size_t)kSlots));
    HIPCHK(launch_fill_u32(amax, kSlots, 0u, st));
    return SKM_OK;
  }
  // a zero word for the bound of the next product's input (stream order: the words are cleared again when all are used)
  int next_slot(hipStream_t st, unsigned int **slot) {
    if (used == kSlots) {
      HIPCHK(launch_fill_u32(amax + 1, kSlots - 1, 0u, st));
      used = 1;
    }
    *slot = amax + used++;
    return SKM_OK;
  }
};
static_assert(Rot::kSlots == Ctx::AM_ROTATION, "Rot's words behind those of a context");
// (back = false: nothing will be rotated back, Rp is not made; jobs: what else opens the call)
int setup_rotation(Pool &pool, hipStream_t st, int32_t d, int32_t ds, const float *R_dev, uint64_t seed, Rot &rot,
                   bool back = true, OpeningJobs jobs = OpeningJobs()) {
  if (int rc = rot.alloc_bounds(pool, st)) return rc;
  float *Rown = nullptr;
  if (!R_dev) {
    HIPCHK(pool.get(&Rown, (size_t)d * d));
    int rc = make_rotation_dev(pool, d, seed, st, Rown);
    if (rc) return rc;
    R_dev = Rown;
  }
  if (back) HIPCHK(pool.get(&rot.Rp, (size_t)d * ds));
  HIPCHK(pool.get(&rot.Rtp, (size_t)d * ds));
  if (d % 32 == 0) HIPCHK(pool.get(&rot.Rs, split_words(d, d)));
  jobs.R = R_dev; jobs.d = d; jobs.ld = ds;
  jobs.Rp = rot.Rp; jobs.Rtp = rot.Rtp; jobs.r_bound = rot.amax;
  HIPCHK(launch_opening(jobs, st));
  return SKM_OK;
}
GemmOperands rotation_product(const float *in, int64_t ldin, int64_t rows, int32_t d, int32_t ds, const Rot &rot, const unsigned int *in_bound) {
  GemmOperands g{in, ldin, (int32_t)rows, rot.Rtp, ds, d, d};
  g.a_absmax = in_bound; g.b_absmax = rot.amax;
  g.b_split = rot.Rs;
  return g;
}
// out (rows x ds, zero padded) = in (rows x d, stride ldin) * R
// out_absmax (optional, zero before the call) receives the bit pattern of max |out|
// (in_bound: a word that already bounds |in|)
int rotate_into(const float *in, int64_t ldin, int64_t rows, int32_t d, int32_t ds, Rot &rot, float *out,
                hipStream_t st, unsigned int *out_absmax = nullptr, const unsigned int *in_bound = nullptr,
                stamp_t *stamp = nullptr) {
  if (!in_bound) {
    unsigned int *slot = nullptr;
    if (int rc = rot.next_slot(st, &slot)) return rc;
    HIPCHK(launch_absmax(in, ldin, rows, d, slot, st));
    in_bound = slot;
  }
  GemmOperands g = rotation_product(in, ldin, rows, d, ds, rot, in_bound);
  g.stamp = stamp;
  HIPCHK(gemm_store(g, out, ds, ds, 1.f, 0.f, st, out_absmax));
  return SKM_OK;
}
// out (rows x d) = Yr (rows x d, stride ldy) * R^T
int unrotate_into(const float *Yr, int64_t ldy, int32_t rows, int32_t d, int32_t ds, Rot &rot, float *out,
                  hipStream_t st, const unsigned int *in_bound = nullptr, stamp_t *stamp = nullptr) {
  if (!in_bound) {
    unsigned int *slot = nullptr;
    if (int rc = rot.next_slot(st, &slot)) return rc;
    HIPCHK(launch_absmax(Yr, ldy, rows, d, slot, st));
    in_bound = slot;
  }
  GemmOperands g{Yr, ldy, rows, rot.Rp, ds, d, d};
  g.a_absmax = in_bound; g.b_absmax = rot.amax;
  g.stamp = stamp;
  HIPCHK(gemm_store(g, out, d, d, 1.f, 0.f, st));
  return SKM_OK;
}

// Ground truth of ETR (Section 3.3): the K nearest points of every query by L2 over X (original space, lowest index
// on ties) as packed (distance, index) keys, ascending.
constexpr int64_t kGtChunk = 1 << 16;

GtPlan gt_plan(int64_t n, int32_t d, int32_t nq, int32_t K) {
  GtPlan p;
  p.ds = round_up(d, 32);
  // the sample: large enough that about 512 points of a query lie below its threshold, 65 536 at least (one pass of the
  // multiply over it costs little beside the one over all points)
  p.nsel = std::min<int64_t>(n, std::max<int64_t>(1 << 16, (int64_t)K * (n / 512)));
  const int64_t groups = (p.nsel + 63) / 64;
  // too few points for a useful threshold, or too many for its sort: the score matrix in full
  if (groups < 2 * (int64_t)K || groups > kGtMaxGroups || n >= ((int64_t)1 << 31)) return p;
  p.ngroups = (int32_t)groups;
  // chunks whose fp16 copy (128 MB) is still in the Infinity Cache when the multiply reads it, whole tiles
  p.chunk = std::max<int64_t>(16384, ((int64_t)64 << 20) / p.ds / 256 * 256);
  // ... that fill whole rounds of the 256 CUs (a tile is 256 points x 256 queries): 5.3 rounds of tiles take as long as
  // six (1M x 768, 1000 queries: 69 rounds in all, now 62)
  const int64_t qtiles = (nq + 255) / 256, rounds = p.chunk / 256 * qtiles / 256;
  if (rounds > 0) p.chunk = rounds * 256 / qtiles * 256;
  p.chunk = std::min<int64_t>(p.chunk, (n + 255) / 256 * 256);
  const double expect = (double)K * (double)n / (double)p.nsel;
  p.cap = 1024;
  while ((double)p.cap < 4.0 * expect + 512.0 && p.cap < kGtMaxCand) p.cap <<= 1;
  p.on = (double)p.cap >= 2.0 * expect;
  p.bytes = (size_t)(p.chunk + nq + 2) * p.ds * 2 + (size_t)p.chunk * 8 + (size_t)nq * (16 + 4 + (size_t)p.ngroups * 4 + (size_t)p.cap * 8) + 8192;
  return p;
}
size_t gt_full_bytes(int64_t n, int32_t nq) { return (size_t)n * 4 + (size_t)nq * (size_t)std::min<int64_t>(n, kGtChunk) * 4 + 4096; }

// *overflow_host (page-locked, valid once the stream has been waited for) != 0: a candidate list ran over, gt_keys is void
int ground_truth_screened(Pool &pool, const GtPlan &p, const float *X, int64_t n, int32_t d, const float *Q, int32_t nq,
                          int32_t K, unsigned long long *gt_keys, unsigned int *overflow_dev, hipStream_t st) {
  uint32_t *plane = nullptr, *qplane = nullptr;
  float *scale = nullptr, *term = nullptr, *qscale = nullptr, *qterm = nullptr, *tq = nullptr, *rterm = nullptr, *gmin = nullptr;
  unsigned long long *cand = nullptr;
  unsigned int *words = nullptr;   // max norm of the points so far | of the sample | of the queries | [nq] list lengths
  HIPCHK(pool.get(&plane, (size_t)((p.chunk + 1) / 2 * 2) * (p.ds / 2)));
  HIPCHK(pool.get(&qplane, (size_t)round_up(nq, 2) * (p.ds / 2)));
  HIPCHK(pool.get(&scale, (size_t)p.chunk));
  HIPCHK(pool.get(&term, (size_t)p.chunk));
  HIPCHK(pool.get(&qscale, (size_t)nq));
  HIPCHK(pool.get(&qterm, (size_t)nq));
  HIPCHK(pool.get(&tq, (size_t)nq));
  HIPCHK(pool.get(&rterm, (size_t)nq));
  HIPCHK(pool.get(&gmin, (size_t)nq * p.ngroups));
  HIPCHK(pool.get(&cand, (size_t)nq * p.cap));
  HIPCHK(pool.get(&words, (size_t)nq + 4));
  HIPCHK(launch_fill_u32(words, (int64_t)nq + 4, 0u, st));
  unsigned int *mx = words, *mx_sample = words + 1, *mx_q = words + 2, *count = words + 4;
  HIPCHK(launch_gt_convert(Q, d, nq, nq, 0, nq, d, p.ds, qplane, qscale, qterm, mx_q, st));
  NeighbourLaunch a{};
  a.A = qplane; a.B = plane; a.M = nq; a.ds = p.ds;
  a.row_term = rterm; a.row_scale = qscale; a.col_term = term; a.col_scale = scale;
  a.group_min = gmin; a.ngroups = p.ngroups;
  a.cand = cand; a.cand_count = count; a.cand_cap = p.cap;
  for (int64_t r0 = 0; r0 < p.nsel; r0 += p.chunk) {
    const int64_t m = std::min<int64_t>(p.chunk, p.nsel - r0);
    HIPCHK(launch_gt_convert(X, d, n, p.nsel, r0, m, d, p.ds, plane, scale, term, mx_sample, st));
    a.N = (int32_t)m;
    a.group0 = (int32_t)(r0 / 64);
    HIPCHK(launch_neighbour_screen(a, true, st));
  }
  HIPCHK(launch_gt_threshold(gmin, p.ngroups, nq, K, qscale, qterm, mx_sample, d, tq, st));
  for (int64_t r0 = 0; r0 < n; r0 += p.chunk) {
    const int64_t m = std::min<int64_t>(p.chunk, n - r0);
    HIPCHK(launch_gt_convert(X, d, n, n, r0, m, d, p.ds, plane, scale, term, mx, st));
    HIPCHK(launch_gt_terms(tq, qscale, qterm, nq, mx, d, rterm, st));
    a.N = (int32_t)m;
    a.point0 = r0;
    HIPCHK(launch_neighbour_screen(a, false, st));
  }
  HIPCHK(launch_gt_select(cand, count, p.cap, nq, K, X, d, Q, d, qscale, qterm, mx, gt_keys, overflow_dev, st));
  return SKM_OK;
}

// The scores q . x from the GEMM in chunks of 65 536 points; each chunk is merged into the running lists.  amax_x /
// amax_q: one word each for the operand bounds.
int ground_truth_full(Pool &pool, const float *X, int64_t n, int32_t d, const float *Q, int32_t nq, int32_t K,
                      unsigned int *amax_x, unsigned int *amax_q, unsigned long long *gt_keys, hipStream_t st) {
  float *xnorm = nullptr, *S = nullptr;
  const int64_t colchunk = std::min<int64_t>(n, kGtChunk);
  HIPCHK(pool.get(&xnorm, (size_t)n));
  HIPCHK(pool.get(&S, (size_t)nq * colchunk));
  HIPCHK(launch_row_norms(X, d, n, d, xnorm, st));
  HIPCHK(launch_fill_u64(gt_keys, (int64_t)nq * K, ~0ull, st));
  if (int rc = measure_absmax(X, d, n, d, amax_x, st)) return rc;
  if (int rc = measure_absmax(Q, d, nq, d, amax_q, st)) return rc;
  for (int64_t c0 = 0; c0 < n; c0 += colchunk) {
    const int64_t m = std::min<int64_t>(colchunk, n - c0);
    GemmOperands g{Q, d, nq, X + c0 * d, d, (int32_t)m, d};
    g.a_absmax = amax_q; g.b_absmax = amax_x;
    HIPCHK(gemm_store(g, S, colchunk, (int32_t)m, 1.f, 0.f, st));
    HIPCHK(launch_topk_merge(S, colchunk, nq, (int32_t)m, c0, xnorm, K, gt_keys, st));
  }
  return SKM_OK;
}

// Waits for the stream (in the screened form: for the word that says whether a list ran over).
int ground_truth_keys(Pool &pool, const float *X, int64_t n, int32_t d, const float *Q, int32_t nq, int32_t K,
                      unsigned int *amax_x, unsigned int *amax_q, unsigned long long *gt_keys, hipStream_t st) {
  const GtPlan plan = gt_plan(n, d, nq, K);
  if (plan.on) {
    PinnedWord over(st);
    if (!over.host) return fail(SKM_EHIP, "hipHostMalloc failed");
    *over.host = 0u;
    if (int rc = ground_truth_screened(pool, plan, X, n, d, Q, nq, K, gt_keys, over.dev, st)) return rc;
    if (int rc = over.wait()) return rc;
    if (!*over.host) return SKM_OK;
  }
  return ground_truth_full(pool, X, n, d, Q, nq, K, amax_x, amax_q, gt_keys, st);
}

// A single assignment step regroups the points itself (see assign_impl) when there are thousands of centroids, several
// points per centroid, rows that the regrouping pass covers, and the first filter is not switched off.  From 2048 centroids on
// only where there is work for some ten milliseconds (2^40 products) and the thresholds have a tail (see step_pruned): then
// 1M x 768, k = 3000 21.3 -> 12.1 ms, k = 2048 16.2 -> 11.4 (without incumbents 18.8 -> 14.4), 1.4M x 384, k = 2100 15.0 -> 8.0, 2.5M x 128,
// k = 3500 12.4 -> 8.4 (16.5 -> 15.5), 600 000 x 1200, k = 2048 18.4 -> 13.9; but 1M x 768, k = 1024 10.8 -> 10.5 (11.7 -> 12.0), 1M x 1536,
// k = 512 23.3 -> 25.5, 200 000 x 256, k = 2048 1.16 -> 1.05 (1.50 -> 2.01), 50 000 x 768, k = 2048 0.95 -> 1.03.  (Up to 2^33
// values, and where there is memory for the regrouped copy: the call is served without it otherwise.)
inline bool assign_groups_always(int32_t k) { return k >= 4096; }
inline bool assign_groups(int64_t n, int32_t ds, int32_t k, int32_t screen_mode) {
  if (screen_mode < 0 || n < 8 * (int64_t)k || ds > 2048 || n >= ((int64_t)1 << 31)) return false;
  return assign_groups_always(k) || (k >= 2048 && n * ds <= ((int64_t)1 << 33) && (double)n * ds * k >= 0x1p40);
}
int assign_impl(const float *X, int64_t n, int32_t d, const float *centroids, int32_t k, const int32_t *prev_assign,
                int32_t dprime_in, const skm_params *pp, int32_t *assign_out, float *dist_out);
int fit_sampled(const float *X, int64_t n, int32_t d, int32_t k, int32_t iters, uint64_t seed, const skm_params &p,
                float *centroids_out, int32_t *assign_out, float *dist_out);
int fit_impl(const float *X, int64_t n, int32_t d, int32_t k, int32_t iters, uint64_t seed, const skm_params *pp,
             float *centroids_out, int32_t *assign_out, float *dist_out, int32_t *dprime_out);

// Whether the program leaves it to the runtime to spin in its waits, as it does unless hipSetDeviceFlags says otherwise: only then is
// watching the report no more of the core than waiting for the stream.  With blocking waits 30 iterations of 1M x 768 into 200
// clusters take 10.6 ms of the core in 38 and would take 25.5 with the watch.
bool waits_spin() {
  unsigned int flags = 0;
  if (hipGetDeviceFlags(&flags) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  flags &= hipDeviceScheduleMask;
  return flags == hipDeviceScheduleAuto || flags == hipDeviceScheduleSpin;
}

// dprime_out (optional) receives the d' the next assignment step would use.
int fit_impl(const float *X, int64_t n, int32_t d, int32_t k, int32_t iters, uint64_t seed, const skm_params *pp,
             float *centroids_out, int32_t *assign_out, float *dist_out, int32_t *dprime_out) {
  int rc = check_shape(X, n, d, k);
  if (rc) return rc;
  if (!centroids_out) return fail(SKM_EINVAL, "centroids_out is null");
  if (iters < 1) return fail(SKM_EINVAL, "iters must be >= 1");
  HostTimes host;   // before the arena: its destructor runs after the workspace has been released
  skm_params p;
  if (pp) p = *pp; else skm_params_default(&p);
  if (!(p.dprime_frac > 0.f && p.dprime_frac <= 1.f)) return fail(SKM_EINVAL, "dprime_frac out of (0, 1]");
  if (!(p.eps0 >= 0.f)) return fail(SKM_EINVAL, "eps0 must be >= 0");
  if (p.tau_group != 0 && p.tau_group != k)
    return fail(SKM_EINVAL, "tau_group: only 0 (= k, the threshold frozen for the whole step) is implemented");
  if (!(p.conv_tol >= 0.f && p.conv_tol <= 1.f)) return fail(SKM_EINVAL, "conv_tol out of [0, 1]");
  skm_trace *tr = p.trace;
  if (tr && (!tr->row || tr->capacity < 1)) return fail(SKM_EINVAL, "trace without rows");
  if (p.angular && p.etr) return fail(SKM_EINVAL, "the angular metric is not combined with ETR");
  if (p.sample_frac > 0.f && p.sample_frac < 1.f) {
    if (p.angular) return fail(SKM_EINVAL, "the angular metric is not combined with sample_frac");
    return fit_sampled(X, n, d, k, iters, seed, p, centroids_out, assign_out, dist_out);
  }
  if ((rc = check_init_idx(p, n, k))) return rc;

  // the workspace in one piece (the caller's, if it lends one): the context's buffers, the rotated points, the rotation
  // matrices and their generator, the ETR buffers
  CallArena ws(fit_workspace_need(n, d, k, p), p.workspace, p.workspace_bytes);
  if (ws.too_small) return fail(SKM_ENOMEM, "params->workspace is smaller than skm_workspace_bytes() for this call");
  host.workspace_ready();
  Ctx c;
  c.st = (hipStream_t)p.stream;
  c.n = n; c.d = d; c.k = k;
  c.ds = round_up(d, 16);
  c.block_stats = p.block_stats != 0;
  c.screen_mode = p.screen;
  // stage times are taken only for a caller that asked for the trace (a small fit inside the hierarchical fit spends
  // a third of its host time creating and reading events otherwise)
  const bool timed = tr != nullptr;
  StageTimer tm(timed, c.st);
  if ((rc = tm.init(64 + (size_t)(std::min(iters, 4096) + 2) * 64))) return rc;
  Events evs;   // of the second stream below
  size_t t_begin = 0, t_rot0 = 0, t_rot = 0, t_unrot0 = 0, t_end = 0, t_gt0 = 0, t_gt1 = 0;
  rc = c.alloc_bounds(tm.point(&t_begin));
  if (rc) return rc;

  // ---- Algorithm 1: R, X~ = X R
  Rot rot;
  rot.amax = c.amax + Ctx::AM_COUNT;
  float *Xr_own = nullptr;
  if (p.rotate) {
    // The rotation matrix is made by a chain of small kernels that leaves most of the device idle: the pass over X
    // that bounds its magnitude (the scale of the split-fp16 product) runs beside it on a second stream.
    struct SideStream {
      hipStream_t s = nullptr;
      ~SideStream() {
        if (s) (void)hipStreamDestroy(s);
      }
    } side;
    hipEvent_t e_fork = nullptr, e_join = nullptr;
    const bool beside = !p.R && (int64_t)n * d >= ((int64_t)1 << 26);
    unsigned int *x_bound = nullptr;
    if (beside) {
      e_fork = evs.next();
      e_join = evs.next();
      if (!e_fork || !e_join) return fail(SKM_EHIP, "hipEventCreate failed");
      HIPCHK(hipStreamCreateWithFlags(&side.s, hipStreamNonBlocking));
      if ((rc = rot.alloc_bounds(c.pool, c.st))) return rc;
      if ((rc = rot.next_slot(c.st, &x_bound))) return rc;
      HIPCHK(hipEventRecord(e_fork, c.st));   // X is ready where the caller's stream stands now
      HIPCHK(hipStreamWaitEvent(side.s, e_fork, 0));
      HIPCHK(launch_absmax(X, d, n, d, x_bound, side.s, 1024));   // four workgroups per CU: the generator's kernels find room
      HIPCHK(hipEventRecord(e_join, side.s));
    }
    OpeningJobs jobs;
    if (!beside) {
      if ((rc = rot.next_slot(c.st, &x_bound))) return rc;
      jobs.bound[0] = {X, n * (int64_t)d, x_bound};
    }
    rc = setup_rotation(c.pool, c.st, d, c.ds, p.R, seed, rot, true, jobs);
    if (rc) return rc;
    HIPCHK(c.pool.get(&Xr_own, (size_t)n * c.ds));
    if (beside) HIPCHK(hipStreamWaitEvent(c.st, e_join, 0));
    rc = rotate_into(X, d, n, d, c.ds, rot, Xr_own, c.st, c.xr_bound, x_bound, tm.point(&t_rot0));
    if (rc) return rc;
    if (beside) HIPCHK(hipStreamSynchronize(side.s));   // nothing is left on the side stream when it is destroyed
    c.Xr = Xr_own; c.ldx = c.ds;
  } else if (d == c.ds && aligned16(X) && !p.angular) {
    c.Xr = X; c.ldx = d;
  } else {
    HIPCHK(c.pool.get(&Xr_own, (size_t)n * c.ds));
    HIPCHK(launch_pad_copy(X, d, n, d, Xr_own, c.ds, c.ds, 0, c.st));
    c.Xr = Xr_own; c.ldx = c.ds;
  }
  if (p.angular) {   // the library's own copy, in place; its bound is that of the scaled rows
    if (p.rotate) HIPCHK(launch_fill_u32(c.xr_bound, 1, 0u, c.st));
    HIPCHK(launch_normalize_rows(Xr_own, c.ds, n, c.ds, c.st, c.xr_bound));
  } else if (!p.rotate) {
    rc = c.measure_xr();
    if (rc) return rc;
  }
  rc = c.alloc_common(p.pair_budget, p.dense_frac, true);
  if (rc) return rc;

  // ---- InitCentroids: k distinct rows of X~.  The row numbers go through the page-locked block, so nothing waits here
  // (the numbers are drawn while the rotation runs); a few are read from there by the gather itself.
  {
    std::vector<int64_t> idx_big;
    if (!c.idx_host) idx_big.resize((size_t)k);
    int64_t *idx = c.idx_host ? c.idx_host : idx_big.data();
    if (p.init_idx) {
      std::copy(p.init_idx, p.init_idx + k, idx);
    } else {
      sample_rows(seed, STREAM_INIT, n, k, idx);
    }
    const int64_t *idx_view = c.idx_dev_view;
    c.pending = true;   // (the block is in use until the first step has been waited for)
    if (k > 1024) {
      int64_t *idx_dev = nullptr;
      HIPCHK(c.pool.get(&idx_dev, (size_t)k));
      HIPCHK(hipMemcpyAsync(idx_dev, idx, sizeof(int64_t) * (size_t)k, hipMemcpyHostToDevice, c.st));
      idx_view = idx_dev;
    }
    HIPCHK(launch_gather_rows(c.Xr, c.ldx, c.ds, idx_view, k, c.Y, c.ds, c.ds, c.st, c.amax + Ctx::AM_Y,
                              tm.point(&t_rot)));   // (the rotation has ended where this starts)
    c.y_amax_valid = true;
    if (!c.idx_host) HIPCHK(hipStreamSynchronize(c.st));
  }

  // ---- ETR set-up (Section 3.3): queries, ground truth, rotated queries
  float *Qr = nullptr, *Sq = nullptr, *ynorm_full = nullptr;
  unsigned long long *gt_keys = nullptr, *etr_scal = nullptr;
  int32_t nprobe = 0;
  if (p.etr) {
    if (p.nq < 1 || p.topk < 1 || p.topk > 256) return fail(SKM_EINVAL, "ETR: nq >= 1 and 1 <= topk <= 256 required");
    nprobe = nprobe_of(k, p.probe_frac);
    if (nprobe > kMaxProbe) return fail(SKM_EINVAL, "ETR: probe_frac * k exceeds 8192");
    const float *Q = p.queries;
    float *Qown = nullptr;
    if (!Q) {
      if (p.nq > n) return fail(SKM_EINVAL, "ETR: nq > n");
      std::vector<int64_t> qi((size_t)p.nq);
      sample_rows(seed, STREAM_QUERIES, n, p.nq, qi.data());
      int64_t *qi_dev = nullptr;
      HIPCHK(c.pool.get(&qi_dev, (size_t)p.nq));
      HIPCHK(c.pool.get(&Qown, (size_t)p.nq * d));
      HIPCHK(hipMemcpyAsync(qi_dev, qi.data(), sizeof(int64_t) * qi.size(), hipMemcpyHostToDevice, c.st));
      HIPCHK(launch_gather_rows(X, d, d, qi_dev, p.nq, Qown, d, d, c.st));
      HIPCHK(hipStreamSynchronize(c.st));
      Q = Qown;
    }
    HIPCHK(c.pool.get(&gt_keys, (size_t)p.nq * p.topk));
    if (p.gt) {
      HIPCHK(launch_index_to_keys(p.gt, (int64_t)p.nq * p.topk, gt_keys, c.st));
    } else {
      HIPCHK(launch_stamp(tm.point(&t_gt0), c.st));
      rc = ground_truth_keys(c.pool, X, n, d, Q, p.nq, p.topk, c.amax + Ctx::AM_X, c.amax + Ctx::AM_Q, gt_keys, c.st);
      if (rc) return rc;
      HIPCHK(launch_stamp(tm.point(&t_gt1), c.st));
    }
    HIPCHK(c.pool.get(&Qr, (size_t)p.nq * c.ds));
    if (p.rotate) {
      rc = rotate_into(Q, d, p.nq, d, c.ds, rot, Qr, c.st, c.amax + Ctx::AM_QR);
      if (rc) return rc;
    } else {
      HIPCHK(launch_pad_copy(Q, d, p.nq, d, Qr, c.ds, c.ds, 0, c.st));
      rc = measure_absmax(Qr, c.ds, p.nq, c.ds, c.amax + Ctx::AM_QR, c.st);
      if (rc) return rc;
    }
    HIPCHK(c.pool.get(&Sq, (size_t)p.nq * k));
    HIPCHK(c.pool.get(&ynorm_full, (size_t)k));
    HIPCHK(c.pool.get(&etr_scal, 2));
    c.point_keys = gt_keys;   // the ground truth names points: it follows them if they are regrouped
    c.n_point_keys = (int64_t)p.nq * p.topk;
  }

  // Regrouping of the points by cluster (Ctx): not for rows that the batched table writes of the threshold pass do not
  // cover; it happens in the third step at the earliest.  Its room is the last that the call takes, and given back where it cannot be
  // had in full: a fit may do without, and its points stay as they are.
  bool may_regroup = c.ds <= 2048 && n < ((int64_t)1 << 31) && regroup_pays(iters - 2 + (p.final_assign ? 1 : 0), n, c.ds, k);
  if (may_regroup) {
    const Pool::Mark before = c.pool.taken();
    auto room = [&]() -> int {
      HIPCHK(c.pool.get(&c.pos_to_id, (size_t)n));
      HIPCHK(c.pool.get(&c.subkey, (size_t)n));
      HIPCHK(c.pool.get(&c.class_ws, (size_t)threshold_class_words(n)));
      HIPCHK(c.pool.get(&c.Xr2, (size_t)n * c.ds));
      return SKM_OK;
    };
    rc = room();
    if (rc == SKM_ENOMEM) {
      (void)hipGetLastError();
      c.pool.give_back(before);
      c.pos_to_id = c.class_ws = nullptr;
      c.subkey = nullptr;
      c.Xr2 = nullptr;
      may_regroup = false;
    } else if (rc) {
      return rc;
    }
    c.Xr_own = Xr_own;
  }

  int32_t dprime = dprime_init(d, p.dprime_frac);
  Rng split_rng = rng_stream(seed, STREAM_SPLIT);
  int32_t run = 0, rows = 0, streak = 0;
  double best_recall = -1.0;
  // recall of (current centroids, current assignment): Section 3.3
  auto measure_recall = [&](double *out) -> int {
    CentroidPrep cp{c.Y, c.ds, k, c.ds};
    cp.ynorm = ynorm_full; cp.dn = c.ds;
    HIPCHK(launch_prep_centroids(cp, c.st));
    if (int mrc = c.measure_y()) return mrc;
    GemmOperands g{Qr, c.ds, p.nq, c.Y, c.ds, k, c.ds};
    g.a_absmax = c.amax + Ctx::AM_QR; g.b_absmax = c.amax + Ctx::AM_Y;
    HIPCHK(gemm_store(g, Sq, k, k, 1.f, 0.f, c.st));
    HIPCHK(launch_fill_u64(etr_scal, 2, 0ull, c.st));
    HIPCHK(launch_recall_scores(Sq, k, p.nq, k, ynorm_full, nprobe, gt_keys, p.topk, c.assign, etr_scal, etr_scal + 1,
                                c.st));
    unsigned long long h[2] = {0, 0};
    HIPCHK(hipMemcpyAsync(h, etr_scal, sizeof(h), hipMemcpyDeviceToHost, c.st));
    HIPCHK(hipStreamSynchronize(c.st));
    *out = h[1] ? (double)h[0] / (double)h[1] : 0.0;
    return SKM_OK;
  };

  // (not in the many small fits that share the host's cores, nor where the stream is waited for after every step anyway, for the recall)
  c.watch = ws.on && !p.etr && waits_spin();
  for (int32_t t = 1; t <= iters; ++t) {
    StepStats ss;
    tm.begin_step();
    if (t == 1) {
      rc = step_exact(c, tm, ss);
    } else {
      std::swap(c.assign, c.prev);
      c.regroup_left = may_regroup ? (iters - t + 1) + (p.final_assign ? 1 : 0) : 0;
      c.update_ahead = c.watch && p.full_update == 0;
      rc = step_pruned(c, tm, dprime, (double)p.eps0, true, ss);
    }
    if (rc) return rc;
    double recall = -1.0;
    if (p.etr) {
      rc = measure_recall(&recall);
      if (rc) return rc;
      HIPCHK(launch_stamp(tm.mark(ST_ETR), c.st));
    }
    int64_t nempty = 0;
    rc = step_update(c, split_rng, p.split_eps, &nempty, ss.changed, p.full_update != 0);
    if (rc) return rc;
    if (p.angular) {
      HIPCHK(launch_fill_u32(c.amax + Ctx::AM_Y, 1, 0u, c.st));
      HIPCHK(launch_normalize_rows(c.Y, c.ds, k, c.ds, c.st, c.amax + Ctx::AM_Y));
      c.y_amax_valid = true;
      c.tau_kept = Ctx::KEPT_NONE;   // (scaling a row that has been scaled before may change its last bits)
    }
    tm.mark_next(ST_UPDATE);   // (no wait: the next step's launches follow while the update runs)
    run = t;
    c.moved += ss.changed;
    if (tr && rows < tr->capacity) fill_row(tr->row[rows], ss, n, k, nempty, recall);
    ++rows;
    if (t > 1 && p.adjust_dprime && k > 1) {
      const double f = 1.0 - (double)ss.survivors / ((double)n * (double)(k - 1));
      dprime = dprime_adjust(d, dprime, f, p.adj_lo, p.adj_hi, p.adj_step);
    }
    bool stop = false;
    if (p.etr) {
      if (t == 1) {
        best_recall = recall;
      } else {
        if (recall - best_recall <= (double)p.etr_tol) ++streak; else streak = 0;
        if (recall > best_recall) best_recall = recall;
        if (streak >= p.etr_patience) stop = true;
      }
    }
    // Section 3.3, second condition (convergence): hardly any point changed its cluster
    if (p.conv_tol > 0.f && t > 1 && (double)ss.changed <= (double)p.conv_tol * (double)n) stop = true;
    if (stop) break;
  }

  // ---- final assignment with the two-phase approach (Section 3.3)
  bool written = false;   // the outputs per point are in the caller's arrays
  if (p.final_assign) {
    StepStats ss;
    std::swap(c.assign, c.prev);
    c.regroup_left = 0;
    c.update_ahead = false;
    written = !c.permuted;   // points in the caller's order: the last kernel writes the caller's arrays
    if (written && assign_out) c.assign = assign_out;
    if (written && dist_out) c.dist = dist_out;
    tm.begin_step();
    rc = step_pruned(c, tm, dprime, (double)p.eps0, true, ss);
    if (rc) return rc;
    if (tr && rows < tr->capacity) fill_row(tr->row[rows], ss, n, k, 0, -1.0);
    ++rows;
  }
  if (c.permuted) {   // per-point results back in the caller's order
    if (assign_out) HIPCHK(launch_scatter_by_index(c.assign, c.pos_to_id, n, assign_out, c.st));
    if (dist_out) HIPCHK(launch_scatter_by_index(c.dist, c.pos_to_id, n, dist_out, c.st));
  } else if (!written) {
    if (assign_out) HIPCHK(hipMemcpyAsync(assign_out, c.assign, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToDevice, c.st));
    if (dist_out) HIPCHK(hipMemcpyAsync(dist_out, c.dist, sizeof(float) * (size_t)n, hipMemcpyDeviceToDevice, c.st));
  }

  // ---- Algorithm 1, last line: Y = Y~ R^T (behind the final assignment, which does not change the centroids: a call that
  // fails there has written none of its outputs)
  if (p.rotate) {
    rc = unrotate_into(c.Y, c.ds, k, d, c.ds, rot, centroids_out, c.st, c.y_amax_valid ? c.amax + Ctx::AM_Y : nullptr,
                       tm.point(&t_unrot0));
    if (rc) return rc;
  } else {
    HIPCHK(hipMemcpy2DAsync(centroids_out, sizeof(float) * (size_t)d, c.Y, sizeof(float) * (size_t)c.ds,
                            sizeof(float) * (size_t)d, (size_t)k, hipMemcpyDeviceToDevice, c.st));
  }
  HIPCHK(launch_stamp(tm.point(&t_end), c.st));
  HIPCHK(hipStreamSynchronize(c.st));
  c.pending = false;
  tm.waited = true;
  if (dprime_out) *dprime_out = dprime;
  if (tr) {
    tr->rows = std::min(rows, tr->capacity);
    tr->iters_run = run;
    tr->inc_updates = c.inc_updates;
    tr->ms_rotate = p.rotate ? tm.between(t_rot0, t_rot) : 0.f;
    tr->ms_init = tm.marks.empty() ? 0.f : tm.between(t_begin, tm.marks.front().second);
    tr->ms_etr_gt = t_gt1 > t_gt0 ? tm.between(t_gt0, t_gt1) : 0.f;
    tr->ms_unrotate = p.rotate ? tm.between(t_unrot0, t_end) : 0.f;
    tr->ms_total = tm.between(t_begin, t_end);
    for (int32_t q = 0; q < tr->rows; ++q) fill_times(tr->row[q], tm, (size_t)q);
  }
  ws.finished();
  host.body_done(tr);
  return SKM_OK;
}


// Rotated rows of a host-resident fit that stay on the device between its passes (the first `batches` batches): a block of
// its own beside the workspace.  A pass over kept rows costs its kernels, one over streamed rows the transfer (17 ms per GB,
// ten times as much): 200 000 x 768 with k = 1024, four passes, 45.6 ms when all of them were sent every time, now 17.0.
// At most half of what is free is taken, and only where the caller left the batch size, and with it the memory in use, to
// the library; a block that cannot be had means that everything is streamed.  Tables stay with the rows only in a block that
// is kept between calls: freed memory is cleared by the engine that copies from the host, which then runs at 44 instead of 58
// GB/s, some 0.25 s behind rows of 6 GB, 0.7 s behind rows and tables of 16.  1M x 1536, k = 1024, ten iterations one call after
// the other 226 ms with tables, 238 without (195 and 213 after a pause); four fits of two streamed passes behind them 1152 and 949
// ms (880 otherwise).
struct KeptRows {
  int64_t batches = 0, rows = 0;
  bool tables = false;              // the split copies and prefix norms stay, too
  float *X = nullptr, *xnp = nullptr;
  uint32_t *Xs = nullptr, *Xh = nullptr;
  unsigned int *bound = nullptr;    // [batches] max |X~| of a batch
  std::vector<char> xnp_valid, xh_valid;   // of a batch's tables
  bool finished = false;            // the call has waited for its stream: the block goes to the cache
  ~KeptRows() {
    if (!block) return;
    if (finished) block_cache().give(block, cap);
    else (void)hipFree(block);
  }
  KeptRows() = default;
  KeptRows(const KeptRows &) = delete;
  KeptRows &operator=(const KeptRows &) = delete;
  // hi: the plane of hi halves is among the tables
  void plan(int64_t n, int64_t W, int32_t ds, bool hi) {
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    const size_t budget = (free_b + block_cache().idle_bytes()) / 2;
    const int64_t nbatch = (n + W - 1) / W;
    const size_t row = (size_t)ds * 4, more = (size_t)split_ld(ds) * 4 + (size_t)ds / 4 + (hi ? (size_t)split_ld(ds) * 2 : 0);
    const size_t fixed = (size_t)nbatch * 4 + 5 * 256 + (size_t)split_ld(ds) * 6;   // (an odd row more in the copies)
    if (budget <= fixed) return;
    // the tables of all rows, or the rows alone, as many whole batches as there is room for (for what cannot be had in one piece,
    // idle blocks of the library go back first; then less is asked for)
    bool with = (size_t)n * (row + more) + fixed <= std::min(budget, BlockCache::kMost);
    int64_t kept = with ? nbatch : std::min<int64_t>(nbatch, (int64_t)((budget - fixed) / ((size_t)W * row))), r = 0;
    while (kept >= 1) {
      r = std::min<int64_t>(n, kept * W);
      const size_t bytes = ((size_t)r * (row + (with ? more : 0)) + fixed + ((size_t)2 << 20) - 1) & ~(((size_t)2 << 20) - 1);
      block = static_cast<char *>(block_cache().take(bytes, &cap));
      if (block) break;
      void *p = nullptr;
      if (device_malloc(&p, bytes) == hipSuccess) {
        block = static_cast<char *>(p);
        cap = bytes;
        break;
      }
      (void)hipGetLastError();
      if (with) with = false;
      else kept /= 2;
    }
    if (!block) return;
    size_t at = 0;
    auto carve = [&](size_t want) {
      char *p = block + at;
      at = (at + want + 255) & ~(size_t)255;
      return p;
    };
    X = reinterpret_cast<float *>(carve((size_t)r * row));
    bound = reinterpret_cast<unsigned int *>(carve((size_t)nbatch * 4));
    if (with) {
      Xs = reinterpret_cast<uint32_t *>(carve(split_words(r, ds) * 4));
      xnp = reinterpret_cast<float *>(carve((size_t)r * ((size_t)ds / 4)));
      if (hi) Xh = reinterpret_cast<uint32_t *>(carve(split_words(r, ds) * 2));
    }
    batches = kept;
    rows = r;
    tables = with;
    xnp_valid.assign((size_t)kept, 0);
    xh_valid.assign((size_t)kept, 0);
  }

 private:
  char *block = nullptr;
  size_t cap = 0;
};

// Algorithm 1 on points that stay in host memory (Section 7.1: batches of X pass through the device, copies and kernels
// overlap).  In the first pass over the data all rows are sent, through two device buffers of `W` rows: while batch g is
// rotated and assigned, batch g + 1 is already there and batch g + 2 follows as soon as the rotation has released its
// buffer.  The rotated rows of as many batches as there is room for stay on the device (KeptRows); later passes (the other
// iterations, the final assignment) send and rotate only the others.
// An update adds the batch's cluster sums (fp64) to S; the means are taken once the pass is complete.
int fit_host_impl(const float *Xh, int64_t n, int32_t d, int32_t k, int32_t iters, uint64_t seed, const skm_params *pp,
                  int64_t batch_rows, float *centroids_out, int32_t *assign_out_host, float *dist_out_host) {
  int rc = check_shape(Xh, n, d, k);
  if (rc) return rc;
  if (!centroids_out) return fail(SKM_EINVAL, "centroids_out is null");
  if (iters < 1) return fail(SKM_EINVAL, "iters must be >= 1");
  if (batch_rows < 0) return fail(SKM_EINVAL, "batch_rows must be >= 0");
  skm_params p;
  if (pp) p = *pp; else skm_params_default(&p);
  if (!(p.dprime_frac > 0.f && p.dprime_frac <= 1.f)) return fail(SKM_EINVAL, "dprime_frac out of (0, 1]");
  if (!(p.eps0 >= 0.f)) return fail(SKM_EINVAL, "eps0 must be >= 0");
  if (p.etr || p.angular || (p.sample_frac > 0.f && p.sample_frac < 1.f))
    return fail(SKM_EINVAL, "the host-resident fit is not combined with ETR, the angular metric or sample_frac");
  skm_trace *tr = p.trace;
  if (tr && (!tr->row || tr->capacity < 1)) return fail(SKM_EINVAL, "trace without rows");
  if ((rc = check_init_idx(p, n, k))) return rc;

  // rows per batch: a multiple of 128 (whole tiles; the per-point arrays of a batch then start 512-byte aligned)
  int64_t W = batch_rows > 0 ? batch_rows : (int64_t)131072;
  W = std::min<int64_t>((W + 127) / 128 * 128, (n + 127) / 128 * 128);
  const int64_t nbatch = (n + W - 1) / W;
  const int npass = iters + (p.final_assign ? 1 : 0);

  // the workspace in one piece: the context of a batch, two raw batches and the rotated one, labels (and distances)
  // of all points, the rotation matrices and their generator, the initial rows
  const size_t ds0 = (size_t)round_up(d, 16);
  const size_t plan = plan_common_bytes(W, d, k, p.pair_budget, p.dense_frac, true);
  CallArena ws(plan ? plan + (size_t)W * (2 * (size_t)d + ds0) * 4 + 3 * (size_t)nbatch * W * 4 + 10 * (size_t)d * ds0 * 4 +
                          (size_t)d * 16384 + (size_t)k * d * 4 + ((size_t)32 << 20)
                    : 0);
  Ctx c;
  c.st = (hipStream_t)p.stream;
  c.n = W; c.d = d; c.k = k;
  c.ds = round_up(d, 16);
  c.block_stats = p.block_stats != 0;
  c.screen_mode = p.screen;
  StageTimer tm(tr != nullptr, c.st);
  Events evs;
  hipEvent_t e_begin = evs.next(), e_init = evs.next(), e_end0 = evs.next(), e_end = evs.next();
  hipEvent_t ev_copied[2] = {evs.next(), evs.next()}, ev_free[2] = {evs.next(), evs.next()};
  if (!e_begin || !e_init || !e_end0 || !e_end || !ev_copied[0] || !ev_copied[1] || !ev_free[0] || !ev_free[1])
    return fail(SKM_EHIP, "hipEventCreate failed");
  struct CopyStream {
    hipStream_t s = nullptr;
    ~CopyStream() {
      if (!s) return;
      (void)hipStreamSynchronize(s);   // (a call that fails: the caller's rows are not read any more once it returns)
      (void)hipStreamDestroy(s);
    }
  } cs;
  HIPCHK(hipStreamCreateWithFlags(&cs.s, hipStreamNonBlocking));
  HIPCHK(hipEventRecord(e_begin, c.st));
  rc = c.alloc_bounds();
  if (rc) return rc;
  rc = c.alloc_common(p.pair_budget, p.dense_frac, true);
  if (rc) return rc;
  const int64_t tile_rows = c.chunk_rows;   // rows per launch of the tile kernel inside a batch
  if ((rc = tm.init(16 + (size_t)nbatch * (8 + 2 * ((size_t)(W + tile_rows - 1) / tile_rows))))) return rc;

  Rot rot;
  if (p.rotate) {
    rc = setup_rotation(c.pool, c.st, d, c.ds, p.R, seed, rot);
    if (rc) return rc;
  }
  float *raw[2] = {nullptr, nullptr}, *Xr_buf = nullptr, *dist_all = nullptr;
  int32_t *lab[2] = {nullptr, nullptr};
  HIPCHK(c.pool.get(&raw[0], (size_t)W * d));
  HIPCHK(c.pool.get(&raw[1], (size_t)W * d));
  HIPCHK(c.pool.get(&Xr_buf, (size_t)W * c.ds));
  HIPCHK(c.pool.get(&lab[0], (size_t)nbatch * W));
  HIPCHK(c.pool.get(&lab[1], (size_t)nbatch * W));
  if (dist_out_host) HIPCHK(c.pool.get(&dist_all, (size_t)nbatch * W));
  KeptRows kept;
  if (batch_rows == 0 && npass > 1) kept.plan(n, W, c.ds, c.Xh != nullptr);

  // ---- the stream of batches: what is sent is every batch once, then in every later pass those that are not kept; send
  // number g goes through device buffer g & 1
  const int64_t per_pass = nbatch - kept.batches, gtotal = nbatch + (int64_t)(npass - 1) * per_pass;
  auto send = [&](int64_t g) -> int {   // enqueue the copy on the copy stream
    if (g >= gtotal) return SKM_OK;
    const int64_t b = g < nbatch ? g : kept.batches + (g - nbatch) % per_pass;
    const int64_t r0 = b * W, rows = std::min<int64_t>(W, n - r0);
    if (g >= 2) HIPCHK(hipStreamWaitEvent(cs.s, ev_free[g & 1], 0));
    HIPCHK(hipMemcpyAsync(raw[g & 1], Xh + (size_t)r0 * d, sizeof(float) * (size_t)rows * d, hipMemcpyHostToDevice, cs.s));
    HIPCHK(hipEventRecord(ev_copied[g & 1], cs.s));
    return SKM_OK;
  };
  // (the generator's kernels are enqueued: the first copies run beside them and the initial centroids)
  HIPCHK(hipStreamWaitEvent(cs.s, e_begin, 0));   // (the block may still be in use by what the caller's stream did before)
  if ((rc = send(0))) return rc;
  if ((rc = send(1))) return rc;
  float *dist_batch = c.dist;
  int32_t *cnt_total = nullptr;   // [k] cluster sizes of the pass
  HIPCHK(c.pool.get(&cnt_total, (size_t)k));

  // ---- InitCentroids: k distinct rows of X, rotated like the points
  {
    std::vector<int64_t> idx((size_t)k);
    if (p.init_idx) {
      std::copy(p.init_idx, p.init_idx + k, idx.begin());
    } else {
      sample_rows(seed, STREAM_INIT, n, k, idx.data());
    }
    std::vector<float> rows_h((size_t)k * d);
    for (int32_t i = 0; i < k; ++i)
      std::memcpy(rows_h.data() + (size_t)i * d, Xh + (size_t)idx[(size_t)i] * d, sizeof(float) * (size_t)d);
    float *rows_dev = nullptr;
    HIPCHK(c.pool.get(&rows_dev, (size_t)k * d));
    HIPCHK(hipMemcpyAsync(rows_dev, rows_h.data(), sizeof(float) * rows_h.size(), hipMemcpyHostToDevice, c.st));
    if (p.rotate) {
      rc = rotate_into(rows_dev, d, k, d, c.ds, rot, c.Y, c.st);
      if (rc) return rc;
    } else {
      HIPCHK(launch_pad_copy(rows_dev, d, k, d, c.Y, c.ds, c.ds, 0, c.st));
    }
    HIPCHK(hipStreamSynchronize(c.st));   // rows_h must outlive the copy
  }
  HIPCHK(hipEventRecord(e_init, c.st));

  int32_t dprime = dprime_init(d, p.dprime_frac);
  Rng split_rng = rng_stream(seed, STREAM_SPLIT);
  int32_t rows_out = 0;
  int cur = 0;   // lab[cur] receives the labels of the pass in work, lab[cur ^ 1] holds those of the pass before
  int64_t sent = 0;   // batches taken from the device buffers so far
  uint32_t *const own_Xs = c.Xs, *const own_Xh = c.Xh;
  float *const own_xnp = c.xnp;
  for (int pass = 0; pass < npass; ++pass) {
    const bool final_pass = pass >= iters;
    StepStats tot;
    tot.pruned = pass > 0;
    tm.begin_step();
    if (!final_pass) {
      HIPCHK(launch_fill_u64(reinterpret_cast<unsigned long long *>(c.S), (int64_t)k * c.ds, 0ull, c.st));
      HIPCHK(launch_fill_u32(reinterpret_cast<unsigned int *>(cnt_total), k, 0u, c.st));
    }
    for (int64_t b = 0; b < nbatch; ++b) {
      const int64_t r0 = b * W, rows = std::min<int64_t>(W, n - r0);
      const bool keep = b < kept.batches;
      float *Xb = keep ? kept.X + (size_t)r0 * c.ds : Xr_buf;
      c.n = rows;
      c.nchunks = (int32_t)((rows + tile_rows - 1) / tile_rows);
      c.Xr = Xb; c.ldx = c.ds;
      c.xr_bound = keep ? kept.bound + b : c.amax + Ctx::AM_XR;
      c.Xs = keep && kept.tables ? kept.Xs + (size_t)r0 * split_ld(c.ds) : own_Xs;
      c.xnp = keep && kept.tables ? kept.xnp + (size_t)r0 * (c.ds / 16) : own_xnp;
      c.Xh = keep && kept.tables ? (kept.Xh ? kept.Xh + (size_t)r0 * (split_ld(c.ds) / 2) : nullptr) : own_Xh;
      c.xnp_valid = keep && kept.tables && kept.xnp_valid[(size_t)b];
      c.xh_valid = keep && kept.tables && kept.xh_valid[(size_t)b];
      if (pass == 0 || !keep) {   // the rows arrive
        const int64_t g = sent++;
        HIPCHK(hipStreamWaitEvent(c.st, ev_copied[g & 1], 0));
        HIPCHK(launch_fill_u32(c.xr_bound, 1, 0u, c.st));
        if (p.rotate) {
          rc = rotate_into(raw[g & 1], d, rows, d, c.ds, rot, Xb, c.st, c.xr_bound);
          if (rc) return rc;
        } else {
          HIPCHK(launch_pad_copy(raw[g & 1], d, rows, d, Xb, c.ds, c.ds, 0, c.st));
        }
        HIPCHK(hipEventRecord(ev_free[g & 1], c.st));
        if ((rc = send(g + 2))) return rc;
        if (!p.rotate) {
          rc = c.measure_xr();
          if (rc) return rc;
        }
      }
      c.assign = lab[cur] + r0;
      c.prev = lab[cur ^ 1] + r0;
      c.dist = dist_all ? dist_all + r0 : dist_batch;
      StepStats ss;
      rc = pass == 0 ? step_exact(c, tm, ss) : step_pruned(c, tm, dprime, (double)p.eps0, true, ss);
      if (rc) return rc;
      if (keep && kept.tables) {
        kept.xnp_valid[(size_t)b] = c.xnp_valid;
        kept.xh_valid[(size_t)b] = c.xh_valid;
      }
      tot.objective += ss.objective;
      tot.survivors += ss.survivors;
      tot.completed += ss.completed;
      tot.changed += ss.changed;
      tot.dense_dims += ss.dense_dims;
      tot.dense_pair_blocks += ss.dense_pair_blocks;
      tot.gather_pair_blocks += ss.gather_pair_blocks;
      tot.gather_pairs += ss.gather_pairs;
      tot.screen_dims += ss.screen_dims;
      tot.listed_tiles += ss.listed_tiles;
      for (int m = 0; m < SKM_MAX_BLOCKS; ++m) tot.enter[m] += ss.enter[m];
      tot.dprime = ss.dprime;
      tot.nblocks = ss.nblocks;
      if (!final_pass) {
        HIPCHK(launch_add_counts(c.up.cnt, k, cnt_total, c.st));
        UpdateWs uw = c.up;
        if (!stable_order_applies(rows, k)) uw.base = nullptr;
        HIPCHK(launch_update(c.Xr, c.ldx, rows, c.ds, c.assign, k, uw, nullptr, c.ds, c.st, c.S, nullptr, 1, c.report->largest));
        HIPCHK(launch_stamp(tm.mark(ST_UPDATE), c.st));
      }
    }
    int64_t nempty = 0;
    if (!final_pass) {
      // means of the whole pass, then the split of empty clusters on the total sizes
      HIPCHK(launch_means_from_sums(c.S, cnt_total, k, c.ds, c.Y, c.ds, c.amax + Ctx::AM_Y, c.st));
      c.y_amax_valid = true;
      c.sizes_known = false;   // (the report holds those of the last batch)
      int32_t *batch_cnt = c.up.cnt;
      c.up.cnt = cnt_total;
      rc = split_empty(c, split_rng, p.split_eps, &nempty);
      c.up.cnt = batch_cnt;
      if (rc) return rc;
      HIPCHK(launch_stamp(tm.mark(ST_UPDATE), c.st));
    }
    HIPCHK(hipStreamSynchronize(c.st));
    if (tr && rows_out < tr->capacity) {
      fill_row(tr->row[rows_out], tot, n, k, nempty, -1.0);
      fill_times(tr->row[rows_out], tm, 0);
    }
    tm.reset();
    ++rows_out;
    if (pass > 0 && !final_pass && p.adjust_dprime && k > 1) {
      const double f = 1.0 - (double)tot.survivors / ((double)n * (double)(k - 1));
      dprime = dprime_adjust(d, dprime, f, p.adj_lo, p.adj_hi, p.adj_step);
    }
    cur ^= 1;
  }
  const int last = cur ^ 1;   // labels of the last pass
  if (assign_out_host)
    HIPCHK(hipMemcpyAsync(assign_out_host, lab[last], sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost, c.st));
  if (dist_out_host)
    HIPCHK(hipMemcpyAsync(dist_out_host, dist_all, sizeof(float) * (size_t)n, hipMemcpyDeviceToHost, c.st));
  HIPCHK(hipEventRecord(e_end0, c.st));
  if (p.rotate) {
    rc = unrotate_into(c.Y, c.ds, k, d, c.ds, rot, centroids_out, c.st);
    if (rc) return rc;
  } else {
    HIPCHK(hipMemcpy2DAsync(centroids_out, sizeof(float) * (size_t)d, c.Y, sizeof(float) * (size_t)c.ds,
                            sizeof(float) * (size_t)d, (size_t)k, hipMemcpyDeviceToDevice, c.st));
  }
  HIPCHK(hipEventRecord(e_end, c.st));
  HIPCHK(hipStreamSynchronize(c.st));
  tm.waited = true;
  HIPCHK(hipStreamSynchronize(cs.s));
  if (tr) {
    tr->rows = std::min(rows_out, tr->capacity);
    tr->iters_run = iters;
    tr->inc_updates = 0;
    tr->ms_rotate = 0.f;
    tr->ms_etr_gt = 0.f;
    (void)hipEventElapsedTime(&tr->ms_init, e_begin, e_init);
    (void)hipEventElapsedTime(&tr->ms_unrotate, e_end0, e_end);
    (void)hipEventElapsedTime(&tr->ms_total, e_begin, e_end);
  }
  ws.finished();
  kept.finished = true;
  return SKM_OK;
}

int assign_impl(const float *X, int64_t n, int32_t d, const float *centroids, int32_t k, const int32_t *prev_assign,
                int32_t dprime_in, const skm_params *pp, int32_t *assign_out, float *dist_out) {
  int rc = check_shape(X, n, d, k, false);
  if (rc) return rc;
  if (!centroids || !assign_out) return fail(SKM_EINVAL, "null pointer");
  skm_params p;
  if (pp) p = *pp; else skm_params_default(&p);
  if (p.angular) return fail(SKM_EINVAL, "the angular metric is a fit option: normalise the inputs for a single step");
  if (p.tau_group != 0 && p.tau_group != k)
    return fail(SKM_EINVAL, "tau_group: only 0 (= k, the threshold frozen for the whole step) is implemented");
  skm_trace *tr = p.trace;
  HostTimes host;
  CallArena ws(assign_workspace_need(n, d, k, p), p.workspace, p.workspace_bytes);
  if (ws.too_small) return fail(SKM_ENOMEM, "params->workspace is smaller than skm_workspace_bytes() for this call");
  host.workspace_ready();
  Ctx c;
  c.st = (hipStream_t)p.stream;
  c.n = n; c.d = d; c.k = k;
  c.ds = round_up(d, 16);
  c.block_stats = p.block_stats != 0;
  c.screen_mode = p.screen;
  StageTimer tm(tr != nullptr && tr->row && tr->capacity >= 1, c.st);
  if ((rc = tm.init(256))) return rc;
  Rot rot;
  float *Xr_own = nullptr;
  rc = c.alloc_bounds();
  if (rc) return rc;
  rc = c.alloc_common(p.pair_budget, p.dense_frac, false);
  if (rc) return rc;
  if (p.rotate) {
    OpeningJobs jobs;
    unsigned int *x_bound = nullptr, *y_bound = nullptr;
    rot.amax = c.amax + Ctx::AM_COUNT;
    if ((rc = rot.next_slot(c.st, &x_bound)) || (rc = rot.next_slot(c.st, &y_bound))) return rc;
    jobs.bound[0] = {X, n * (int64_t)d, x_bound};
    jobs.bound[1] = {centroids, k * (int64_t)d, y_bound};
    if (!prev_assign) {   // (the search for the incumbents starts from keys of ~0)
      jobs.fill = c.best;
      jobs.nfill = n;
      c.best_filled = true;
    }
    rc = setup_rotation(c.pool, c.st, d, c.ds, p.R, 0, rot, false, jobs);
    if (rc) return rc;
    HIPCHK(c.pool.get(&Xr_own, (size_t)n * c.ds));
    const GemmOperands gx = rotation_product(X, d, n, d, c.ds, rot, x_bound), gy = rotation_product(centroids, d, k, d, c.ds, rot, y_bound);
    HIPCHK(gemm_store_two(gx, Xr_own, c.xr_bound, gy, c.Y, c.amax + Ctx::AM_Y, c.ds, c.ds, c.st));
    c.y_amax_valid = true;
    c.Xr = Xr_own; c.ldx = c.ds;
  } else {
    if (d == c.ds && aligned16(X)) {
      c.Xr = X; c.ldx = d;
    } else {
      HIPCHK(c.pool.get(&Xr_own, (size_t)n * c.ds));
      HIPCHK(launch_pad_copy(X, d, n, d, Xr_own, c.ds, c.ds, 0, c.st));
      c.Xr = Xr_own; c.ldx = c.ds;
    }
    HIPCHK(launch_pad_copy(centroids, d, k, d, c.Y, c.ds, c.ds, 0, c.st));
    rc = c.measure_xr();
    if (rc) return rc;
  }
  c.single_step = true;
  c.prev_in = prev_assign;   // checked and copied at the start of the step; a bad label leaves the outputs untouched (close_step)
  // Many centroids: a step on its own pays for what a fit does once in its third step.  The points are rewritten
  // grouped by their incumbents and the first filter runs in front of the exact kernel (a million tiles of two slabs
  // each otherwise: the fixed costs of a tile, not the arithmetic, are then the whole run time).
  if (assign_groups(n, c.ds, k, p.screen) && c.colmask) {
    auto room = [&]() -> int {
      HIPCHK(c.pool.get(&c.pos_to_id, (size_t)n));
      HIPCHK(c.pool.get(&c.subkey, (size_t)n));
      HIPCHK(c.pool.get(&c.up.off, (size_t)k + 1));
      HIPCHK(c.pool.get(&c.up.cursor, (size_t)k));
      HIPCHK(c.pool.get(&c.up.segoff, (size_t)k + 1));
      HIPCHK(c.pool.get(&c.up.order, (size_t)n));
      HIPCHK(c.pool.get(&c.grp_cnt, (size_t)k + 1));
      HIPCHK(c.pool.get(&c.class_ws, (size_t)threshold_class_words(n)));
      HIPCHK(c.pool.get(&c.Xr2, (size_t)n * c.ds));
      return SKM_OK;
    };
    rc = room();
    if (rc == SKM_OK) {
      c.group_now = true;
      c.last_prune_frac = 1.0;   // the filter runs: with points grouped and thousands of centroids it has columns to drop
    } else if (rc != SKM_ENOMEM || assign_groups_always(k)) {
      return rc;
    } else {   // no memory for what such a step may do without: the points stay as they are
      (void)hipGetLastError();
      c.Xr2 = nullptr;
    }
  }
  const int32_t dprime = dprime_in > 0 ? snap16((double)dprime_in, d) : dprime_init(d, p.dprime_frac);
  StepStats ss;
  const bool direct = !c.group_now;   // the last kernel writes the caller's arrays (not in a step that may regroup the points)
  if (direct) {
    c.assign = assign_out;
    if (dist_out) c.dist = dist_out;
  }
  tm.begin_step();
  rc = step_pruned(c, tm, dprime, (double)p.eps0, prev_assign != nullptr, ss);
  if (rc) return rc;
  if (!direct) {
    if (c.permuted) {   // per-point results back in the caller's order
      HIPCHK(launch_scatter_by_index(c.assign, c.pos_to_id, n, assign_out, c.st));
      if (dist_out) HIPCHK(launch_scatter_by_index(c.dist, c.pos_to_id, n, dist_out, c.st));
    } else {
      HIPCHK(hipMemcpyAsync(assign_out, c.assign, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToDevice, c.st));
      if (dist_out) HIPCHK(hipMemcpyAsync(dist_out, c.dist, sizeof(float) * (size_t)n, hipMemcpyDeviceToDevice, c.st));
    }
    HIPCHK(hipStreamSynchronize(c.st));
  }
  tm.waited = true;   // (the step itself ends with a wait)
  if (tr && tr->row && tr->capacity >= 1) {
    fill_row(tr->row[0], ss, n, k, 0, -1.0);
    fill_times(tr->row[0], tm, 0);
    tr->rows = 1;
    tr->iters_run = 0;
    tr->ms_total = tr->row[0].ms_step;
    host.body_done(tr);
  }
  ws.finished();
  return SKM_OK;
}

// The exact assignment through the one-product search of iteration 1 (a third of the matrix work of the three-product argmin;
// the candidates' distances are the direct ones), a batch of rows at a time.  A batch with a candidate list that ran over or a
// row that no centroid was offered to (one that is no number) takes the product of all pairs, in the same buffers: nothing is
// allocated behind the first label that is written.  done = false: no room for the buffers, and the caller takes the other form.
// Up to 2^18 rows to a batch, fewer where the call's block (6.25 d + 2.3 K bytes a row, 10.25 d with a padded copy, 18 d a centroid)
// would pass half of what the library keeps between calls: a block that it does not keep costs 25 ms a GB once it is freed
// (262 144 x 3072, k = 2048 in one batch 166 ms, in four 8.9, three products 10.4).  Where the centroids alone are too much for that
// the search has to save twice as much as the block costs (3 ns for 10^6 multiply-adds: 20 000 x 1024, k = 400 000 220 ms, three
// products 48).
constexpr int64_t kExactRows = (int64_t)1 << 18, kExactLeast = (int64_t)1 << 14;
struct ExactPlan {
  int64_t rows = 0;   // 0: not this way
  size_t bytes = 0;
};
ExactPlan exact_plan(int64_t n, int32_t d, int32_t k, bool pad) {
  auto bytes = [&](int64_t rows) -> size_t {
    const size_t plan = plan_common_bytes(rows, d, k, 0, 0.f, false);
    return plan ? plan + (pad ? (size_t)rows * round_up(d, 16) * 4 : 0) + ((size_t)1 << 20) : 0;
  };
  ExactPlan p;
  const size_t fixed = bytes(1);
  if (!fixed) return p;
  for (p.rows = std::min<int64_t>(n, kExactRows);; p.rows = (p.rows / 2 + 127) / 128 * 128) {
    p.bytes = bytes(p.rows);
    if (!p.bytes) return ExactPlan();
    if (p.rows <= kExactLeast || p.bytes <= BlockCache::kMost / 2 || p.bytes - fixed <= BlockCache::kMost / 4) break;
  }
  if (p.bytes > BlockCache::kMost && (double)n * d * k < 2e4 * (double)p.bytes) return ExactPlan();
  return p;
}
// From 2048 centroids on, for rows that the argmin with the rows in registers does not take, and from 2^34 multiply-adds on (the
// search is a dozen launches more).  Three products -> search: 16 384 x 256, k = 4096 178 -> 173 us, 8000 x 384, k = 8000 228 -> 204,
// 100 000 x 384, k = 2048 565 -> 493, 700 001 x 300, k = 5000 8.7 -> 4.9 ms, 400 000 x 768, k = 8000 14.8 -> 7.1; but 60 000 x 192, k = 1536
// 200 -> 214 us, 300 000 x 160, k = 1300 685 -> 702, 200 000 x 96, k = 2000 310 -> 435.  A row's tables are written for every call, and
// take as long as a few thousand centroids (more beyond 2048 dimensions, where they are written point by point): 20 000 x 8192, k = 2048
// 2.41 -> 2.27 ms, 20 000 x 10 001 4.35 -> 3.88, 40 000 x 16 384, k = 4096 15.9 -> 15.0; but 40 000 x 12 288, k = 2048 6.41 -> 6.60, 40 000 x
// 16 384 8.6 -> 11.2.  Labels unlike those of fp64: 2 of 100 000 -> 0, 3 of 60 000 (k = 4000) -> 1.
bool exact_filter_pays(int64_t n, int32_t d, int32_t k) {
  return k >= 2048 && d > 128 && d <= 5 * k && (double)n * d * k >= 17179869184.0;
}
int exact_through_filter(const float *X, int64_t n, int32_t d, const float *centroids, int32_t k, hipStream_t st,
                         int32_t *assign_out, float *dist_out, bool &done) {
  done = false;
  const int32_t ds = round_up(d, 16);
  const bool pad = d != ds || !aligned16(X);
  const ExactPlan plan = exact_plan(n, d, k, pad);
  const int64_t W = plan.rows;
  if (!W) return SKM_OK;
  CallArena ws(plan.bytes);
  Ctx c;
  c.st = st;
  c.n = W; c.d = d; c.k = k; c.ds = ds;
  StageTimer tm(false, st);
  float *Xo = nullptr;
  if (c.alloc_bounds() != SKM_OK || c.alloc_common(0, 0.f, false) != SKM_OK || !c.colmask || (pad && c.pool.get(&Xo, (size_t)W * ds) != hipSuccess)) {
    (void)hipGetLastError();
    return SKM_OK;
  }
  HIPCHK(launch_pad_copy(centroids, d, k, d, c.Y, ds, ds, 0, st));
  const int64_t tile_rows = c.chunk_rows;
  for (int64_t r0 = 0; r0 < n; r0 += W) {
    const int64_t rows = std::min<int64_t>(W, n - r0);
    c.n = rows;
    c.nchunks = (int32_t)((rows + tile_rows - 1) / tile_rows);
    c.Xr = X + r0 * d;
    c.ldx = d;
    if (pad) {
      HIPCHK(launch_pad_copy(c.Xr, d, rows, d, Xo, ds, ds, 0, st));
      c.Xr = Xo;
      c.ldx = ds;
    }
    if (int rc = c.measure_xr()) return rc;
    c.xnp_valid = c.xh_valid = false;
    if (int rc = filtered_nearest(c, ds, tm)) return rc;
    c.pending = true;
    // labels (and distances) from c.best
    auto deliver = [&](unsigned int *unset) -> int {
      if (dist_out)   // (not the search's own distances, which add the blocks of a row one after the other: 2 to 3.7e-7 off, these 1.7e-7)
        HIPCHK(launch_tau_init(c.Xr, c.ldx, rows, ds, c.Y, ds, nullptr, dist_out + r0, c.best, st, nullptr, nullptr, nullptr, nullptr, nullptr,
                               assign_out + r0, nullptr, unset));
      else
        HIPCHK(launch_finalize_assign(FinalizeArgs{c.best, nullptr, rows, assign_out + r0, nullptr, nullptr, k, unset}, st));
      return SKM_OK;
    };
    if (int rc = deliver(c.flag)) return rc;
    HIPCHK(hipMemcpyAsync(&c.report->flag, c.flag, sizeof(unsigned int), hipMemcpyDeviceToHost, st));
    if (int rc = c.wait_stream()) return rc;
    if (c.report->flag != 0) {   // (the search has left the centroids' norms and their split copy)
      HIPCHK(launch_fill_u64(c.best, rows, ~0ull, st));
      GemmOperands g{c.Xr, c.ldx, (int32_t)rows, c.Y, ds, k, ds};
      g.a_absmax = c.xr_bound; g.b_absmax = c.amax + Ctx::AM_Y;
      g.b_presplit = c.Ys; g.ldbs = split_ld(ds);
      HIPCHK(gemm_argmin(g, c.ynorm, c.best, st));
      if (int rc = deliver(nullptr)) return rc;
      HIPCHK(hipStreamSynchronize(st));
    }
  }
  ws.finished();
  done = true;
  return SKM_OK;
}

// Sampled fit (Section 4.4): Algorithm 1 runs on a uniform sample of the rows, then every point is assigned
// to the resulting centroids by the two-phase step without a previous assignment.
int fit_sampled(const float *X, int64_t n, int32_t d, int32_t k, int32_t iters, uint64_t seed, const skm_params &p,
                float *centroids_out, int32_t *assign_out, float *dist_out) {
  if (p.etr) return fail(SKM_EINVAL, "sample_frac and ETR cannot be combined");
  if (!p.final_assign) return fail(SKM_EINVAL, "sample_frac needs the final assignment pass");
  const int64_t s = sample_size(n, k, p.sample_frac);
  hipStream_t st = (hipStream_t)p.stream;
  const int32_t ds = round_up(d, 16);
  HostTimes host;
  // one workspace for the whole call (the caller's, if it lends one); the nested fit and the nested assignment carve
  // theirs from it, one after the other
  CallArena ws(fit_workspace_need(n, d, k, p), p.workspace, p.workspace_bytes);
  if (ws.too_small) return fail(SKM_ENOMEM, "params->workspace is smaller than skm_workspace_bytes() for this call");
  host.workspace_ready();
  Pool pool;
  Events evs;
  hipEvent_t e0 = evs.next(), e1 = evs.next();
  if (!e0 || !e1) return fail(SKM_EHIP, "hipEventCreate failed");
  HIPCHK(hipEventRecord(e0, st));
  // rotate everything once: the final pass needs all rows in the rotated space
  Rot rot;
  const float *Xr = X;
  int64_t ldx = d;
  float *Xr_own = nullptr;
  if (p.rotate) {
    int rc = setup_rotation(pool, st, d, ds, p.R, seed, rot);
    if (rc) return rc;
    HIPCHK(pool.get(&Xr_own, (size_t)n * ds));
    rc = rotate_into(X, d, n, d, ds, rot, Xr_own, st);
    if (rc) return rc;
    Xr = Xr_own; ldx = ds;
  }
  // the sample: s distinct rows, ascending
  std::vector<int64_t> idx((size_t)s);
  sample_rows(seed, STREAM_SAMPLE, n, (int32_t)std::min<int64_t>(s, 0x7fffffff), idx.data());
  std::sort(idx.begin(), idx.end());
  int64_t *idx_dev = nullptr;
  float *Xs = nullptr, *Yr = nullptr;
  HIPCHK(pool.get(&idx_dev, (size_t)s));
  HIPCHK(pool.get(&Xs, (size_t)s * d));
  HIPCHK(pool.get(&Yr, (size_t)k * d));
  HIPCHK(hipMemcpyAsync(idx_dev, idx.data(), sizeof(int64_t) * idx.size(), hipMemcpyHostToDevice, st));
  HIPCHK(launch_gather_rows(Xr, ldx, d, idx_dev, (int32_t)s, Xs, d, d, st));
  HIPCHK(hipStreamSynchronize(st));
  // Algorithm 1 on the sample, in the rotated space
  skm_params pin = p;
  pin.sample_frac = 0.f;
  pin.rotate = 0;
  pin.R = nullptr;
  pin.final_assign = 0;
  pin.workspace = nullptr;   // the nested calls carve from the arena of this call
  pin.workspace_bytes = 0;
  skm_trace inner{};
  skm_trace *tr = p.trace;
  if (tr) {
    inner = *tr;
    pin.trace = &inner;
  }
  int32_t dprime = 0;
  int rc = fit_impl(Xs, s, d, k, iters, seed, &pin, Yr, nullptr, nullptr, &dprime);
  if (rc) return rc;
  // every point against the final centroids, no previous assignment
  skm_params pfin = p;
  pfin.rotate = 0;
  pfin.R = nullptr;
  pfin.workspace = nullptr;
  pfin.workspace_bytes = 0;
  skm_trace last{};
  if (tr) {
    last.capacity = tr->capacity - inner.rows;
    last.row = tr->row + inner.rows;
    pfin.trace = last.capacity >= 1 ? &last : nullptr;
  }
  if (Xr_own && ds != d) {
    // the assignment call takes dense n x d rows; the rotated buffer has stride ds when d is no multiple of 16
    float *Xd = nullptr;
    HIPCHK(pool.get(&Xd, (size_t)n * d));
    HIPCHK(hipMemcpy2DAsync(Xd, sizeof(float) * (size_t)d, Xr_own, sizeof(float) * (size_t)ds, sizeof(float) * (size_t)d,
                            (size_t)n, hipMemcpyDeviceToDevice, st));
    Xr = Xd;
  }
  float *dist_tmp = dist_out;
  int32_t *assign_tmp = assign_out;
  if (!assign_tmp) HIPCHK(pool.get(&assign_tmp, (size_t)n));
  rc = assign_impl(Xr, n, d, Yr, k, nullptr, dprime, &pfin, assign_tmp, dist_tmp);
  if (rc) return rc;
  // centroids back in the original space
  if (p.rotate) {
    float *Yp = nullptr;
    HIPCHK(pool.get(&Yp, (size_t)k * ds));
    HIPCHK(launch_pad_copy(Yr, d, k, d, Yp, ds, ds, 0, st));
    rc = unrotate_into(Yp, ds, k, d, ds, rot, centroids_out, st);
    if (rc) return rc;
  } else {
    HIPCHK(hipMemcpyAsync(centroids_out, Yr, sizeof(float) * (size_t)k * d, hipMemcpyDeviceToDevice, st));
  }
  HIPCHK(hipEventRecord(e1, st));
  HIPCHK(hipStreamSynchronize(st));
  if (tr) {
    tr->rows = inner.rows + ((pfin.trace && last.rows > 0) ? 1 : 0);
    tr->iters_run = inner.iters_run;
    tr->ms_rotate = 0.f;
    tr->ms_init = inner.ms_init;
    tr->ms_etr_gt = 0.f;
    tr->ms_unrotate = 0.f;
    (void)hipEventElapsedTime(&tr->ms_total, e0, e1);
    host.body_done(tr);
  }
  ws.finished();
  return SKM_OK;
}

// Upper bound of what a hierarchical fit carves from its workspace: the rotated rows (and a dense copy when d is no
// multiple of 16), the meso and fine centroids, the membership arrays, and below them, one after the other, the meso
// fit, the fine phase and the final assignment.  The fine phase is bounded by its worst case, a single meso-cluster
// that holds nearly all rows and clusters; with balanced meso-clusters eight workers fit in that room many times over.
size_t hier_workspace_need(int64_t n, int32_t d, int32_t k, const skm_params &p) {
  const size_t ds0 = (size_t)((d + 15) / 16 * 16);
  skm_params q = p;
  q.sample_frac = 0.f;
  q.etr = 0;
  const size_t a = fit_workspace_need(n, d, k, q), b = assign_workspace_need(n, d, k, q);
  if (!a || !b) return 0;
  return std::max(a + (size_t)n * d * 4 + (size_t)n * 4 + 4096, b) + (size_t)n * ds0 * 4 + (ds0 != (size_t)d ? (size_t)n * d * 4 : 0) +
         (size_t)k * (2 * (size_t)d + ds0) * 4 + (size_t)n * 16 + 10 * (size_t)d * ds0 * 4 + (size_t)d * 16384 + ((size_t)32 << 20);
}

// Hierarchical SuperKMeans (Section 6): Algorithm 1 with sqrt(k) clusters on all points (MESO), then Algorithm 1 inside
// every meso-cluster with its share of the k clusters (FINE), then the two-phase assignment of every point to the k
// fine centroids.  Everything runs in the rotated space; X is rotated once.
int fit_hierarchical(const float *X, int64_t n, int32_t d, int32_t k, int32_t meso_iters, int32_t fine_iters, uint64_t seed,
                     const skm_params *pp, float *centroids_out, int32_t *assign_out, float *dist_out,
                     int64_t *meso_sizes_out, int32_t *fine_counts_out) {
  int rc = check_shape(X, n, d, k);
  if (rc) return rc;
  if (!centroids_out) return fail(SKM_EINVAL, "centroids_out is null");
  if (meso_iters < 1 || fine_iters < 1) return fail(SKM_EINVAL, "meso_iters and fine_iters must be >= 1");
  skm_params p;
  if (pp) p = *pp; else skm_params_default(&p);
  if (p.etr) return fail(SKM_EINVAL, "the hierarchical fit does not take ETR");
  if (p.angular) return fail(SKM_EINVAL, "the hierarchical fit does not take the angular metric");
  if (p.sample_frac > 0.f && p.sample_frac < 1.f) return fail(SKM_EINVAL, "the hierarchical fit does not take sample_frac");
  if (p.init_idx) return fail(SKM_EINVAL, "the hierarchical fit draws its initial rows from the seed");
  if (!p.final_assign) return fail(SKM_EINVAL, "the hierarchical fit needs the final assignment pass");
  skm_trace *tr = p.trace;
  if (tr && (!tr->row || tr->capacity < 1)) return fail(SKM_EINVAL, "trace without rows");
  hipStream_t st = (hipStream_t)p.stream;
  const int32_t ds = round_up(d, 16);
  HostTimes host;
  CallArena ws(hier_workspace_need(n, d, k, p), p.workspace, p.workspace_bytes);
  if (ws.too_small) return fail(SKM_ENOMEM, "params->workspace is smaller than skm_hier_workspace_bytes() for this call");
  host.workspace_ready();
  Pool pool;
  Events evs;
  hipEvent_t e0 = evs.next(), e1 = evs.next(), e_meso = evs.next(), e_fine = evs.next();
  if (!e0 || !e1 || !e_meso || !e_fine) return fail(SKM_EHIP, "hipEventCreate failed");
  HIPCHK(hipEventRecord(e0, st));
  Rot rot;
  const float *Xr = X;   // dense n x d rows in the rotated space
  if (p.rotate) {
    rc = setup_rotation(pool, st, d, ds, p.R, seed, rot);
    if (rc) return rc;
    float *Xp = nullptr;
    HIPCHK(pool.get(&Xp, (size_t)n * ds));
    rc = rotate_into(X, d, n, d, ds, rot, Xp, st);
    if (rc) return rc;
    Xr = Xp;
    if (ds != d) {
      float *Xd = nullptr;
      HIPCHK(pool.get(&Xd, (size_t)n * d));
      HIPCHK(hipMemcpy2DAsync(Xd, sizeof(float) * (size_t)d, Xp, sizeof(float) * (size_t)ds, sizeof(float) * (size_t)d,
                              (size_t)n, hipMemcpyDeviceToDevice, st));
      Xr = Xd;
    }
  }
  skm_params pin = p;
  pin.rotate = 0;
  pin.R = nullptr;
  pin.trace = nullptr;
  pin.workspace = nullptr;   // the nested calls carve from the arena of this call
  pin.workspace_bytes = 0;

  // ---- MESO
  const int32_t km = hier_meso_count(k);
  float *Ymeso = nullptr, *Yr = nullptr;
  int32_t *meso_assign = nullptr;
  HIPCHK(pool.get(&Ymeso, (size_t)km * d));
  HIPCHK(pool.get(&Yr, (size_t)k * d));
  HIPCHK(pool.get(&meso_assign, (size_t)n));
  skm_params pm = pin;
  skm_trace inner{};
  if (tr) {
    inner = *tr;
    pm.trace = &inner;
  }
  rc = fit_impl(Xr, n, d, km, meso_iters, seed, &pm, Ymeso, meso_assign, nullptr, nullptr);
  if (rc) return rc;
  HIPCHK(hipEventRecord(e_meso, st));
  // members of every meso-cluster in ascending row order (counting sort on the host)
  std::vector<int32_t> ma((size_t)n);
  HIPCHK(hipMemcpyAsync(ma.data(), meso_assign, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  std::vector<int64_t> sizes((size_t)km, 0), start((size_t)km + 1, 0);
  for (int64_t i = 0; i < n; ++i) {
    if (ma[(size_t)i] < 0 || ma[(size_t)i] >= km) return fail(SKM_EINTERNAL, "meso assignment out of range");
    ++sizes[(size_t)ma[(size_t)i]];
  }
  for (int32_t c = 0; c < km; ++c) start[(size_t)c + 1] = start[(size_t)c] + sizes[(size_t)c];
  std::vector<int64_t> order((size_t)n), cursor(start.begin(), start.end() - 1);
  for (int64_t i = 0; i < n; ++i) order[(size_t)cursor[(size_t)ma[(size_t)i]]++] = i;
  std::vector<int32_t> counts((size_t)km, 0);
  hier_alloc(sizes.data(), km, k, counts.data());
  if (meso_sizes_out) std::copy(sizes.begin(), sizes.end(), meso_sizes_out);
  if (fine_counts_out) std::copy(counts.begin(), counts.end(), fine_counts_out);

  // ---- FINE: the meso-clusters are independent small problems; a few host threads, each with its own stream and
  // workspace arena, take them from a shared counter so that their short kernels overlap on the device.  The result
  // does not depend on who runs what: every fit writes its own block of Yr and draws from its own seed.
  const int64_t nmax = *std::max_element(sizes.begin(), sizes.end());
  const int32_t kmax = *std::max_element(counts.begin(), counts.end());
  std::vector<int32_t> koffs((size_t)km + 1, 0);
  for (int32_t c = 0; c < km; ++c) koffs[(size_t)c + 1] = koffs[(size_t)c] + counts[(size_t)c];
  if (koffs[(size_t)km] != k) return fail(SKM_EINTERNAL, "fine cluster counts do not add up to k");
  int64_t *order_dev = nullptr;
  HIPCHK(pool.get(&order_dev, (size_t)n));
  HIPCHK(hipMemcpyAsync(order_dev, order.data(), sizeof(int64_t) * (size_t)n, hipMemcpyHostToDevice, st));
  HIPCHK(hipStreamSynchronize(st));
  {
    struct Worker {
      hipStream_t st = nullptr;
      Arena arena;
      float *Xs = nullptr;
      int rc = SKM_OK;
      std::string err;
    };
    // The device exposes four hardware queues to a process; twice as many threads still gain a little (2 workers: 152 ms
    // for the fine phase of 1M x 1536 into 16 384 clusters, 4: 124, 8: 120, 12: 116), because the host side of one small
    // fit (some seventy launches and a dozen waits) then overlaps the device side of another.
    int nworkers = (int)std::min<int32_t>(8, km);
    // workspace of the largest fine fit (a bound for every other: the need grows with the rows and with the clusters)
    skm_params pneed = pin;
    pneed.final_assign = 0;
    const size_t want = fit_workspace_need(std::max<int64_t>(nmax, 1), d, std::max<int32_t>(kmax, 1), pneed);
    if (!want) return fail(SKM_EINVAL, "pair_budget too large (must stay below 2^32 pairs)");
    const size_t per_worker = want + (size_t)std::max<int64_t>(nmax, 1) * d * 4 + 1024;
    Arena *top = tl_arena;
    if (top && top->strict) {
      // a caller's workspace: every worker's share comes out of it, so there are as many workers as shares fit
      const size_t shares = (top->cap - std::min(top->cap, top->off + 512)) / per_worker;
      if (shares < 1) return fail(SKM_ENOMEM, "params->workspace cannot hold the largest fine fit");
      nworkers = (int)std::min<size_t>((size_t)nworkers, shares);
    }
    std::vector<Worker> workers((size_t)nworkers);
    Pool fine_pool;   // the workers' buffers and shares: given back to the arena when the fine phase ends
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    struct StreamGuard {
      std::vector<Worker> &w;
      ~StreamGuard() {
        for (Worker &x : w)
          if (x.st) (void)hipStreamDestroy(x.st);
      }
    } guard{workers};
    for (Worker &w : workers) {
      HIPCHK(hipStreamCreateWithFlags(&w.st, hipStreamNonBlocking));
      HIPCHK(fine_pool.get(&w.Xs, (size_t)std::max<int64_t>(nmax, 1) * d));
      if (top && top->cap - std::min(top->cap, top->off + 512) >= want) {
        char *share = nullptr;
        HIPCHK(fine_pool.get(&share, want));
        w.arena.lend(share, want);
        w.arena.strict = top->strict;   // the library's own arena: what does not fit may still come from hipMalloc
      } else if (w.arena.init(want) != hipSuccess) {
        (void)hipGetLastError();
        w.arena.base = nullptr;
        w.arena.cap = 0;   // every buffer of this worker then comes from hipMalloc
      }
    }
    std::atomic<int32_t> next_cluster{0};
    auto body = [&](Worker &w) {
      if (hipSetDevice(dev) != hipSuccess) {
        w.rc = fail(SKM_EHIP, "hipSetDevice failed in a worker thread");
        w.err = g_last_error;
        return;
      }
      ArenaScope scope(w.arena.base ? &w.arena : nullptr);
      skm_params pfine = pin;
      pfine.final_assign = 0;   // only the centroids of a fine fit are used
      pfine.stream = (void *)w.st;
      for (;;) {
        const int32_t c = next_cluster.fetch_add(1);
        if (c >= km) break;
        const int32_t kc = counts[(size_t)c];
        if (kc == 0) continue;
        const int64_t nc = sizes[(size_t)c];
        hipError_t e = launch_gather_rows(Xr, d, d, order_dev + start[(size_t)c], (int32_t)nc, w.Xs, d, d, w.st);
        int rcw = e == hipSuccess ? SKM_OK : fail_hip(e, "launch_gather_rows");
        if (!rcw)
          rcw = fit_impl(w.Xs, nc, d, kc, fine_iters, seed + 1 + (uint64_t)c, &pfine, Yr + (size_t)koffs[(size_t)c] * d,
                         nullptr, nullptr, nullptr);
        if (rcw) {
          w.rc = rcw;
          w.err = g_last_error;
          next_cluster.store(km);   // stop handing out work
          break;
        }
      }
    };
    std::vector<std::thread> threads;
    for (int t = 1; t < nworkers; ++t) {
      try {
        threads.emplace_back(
            [&body](Worker &w) {
              body(w);
              tl_pinned.release();   // this thread's page-locked blocks go with it
            },
            std::ref(workers[(size_t)t]));
      } catch (const std::system_error &) {
        break;   // fewer threads: the others take the work
      }
    }
    body(workers[0]);
    for (std::thread &t : threads) t.join();
    for (Worker &w : workers) {
      if (w.st) (void)hipStreamSynchronize(w.st);
    }
    for (Worker &w : workers) {
      if (w.rc) {
        g_last_error = w.err;
        return w.rc;
      }
    }
  }
  HIPCHK(hipEventRecord(e_fine, st));

  // ---- every point against the k fine centroids, no previous assignment
  skm_params pfin = pin;
  skm_trace last{};
  if (tr) {
    last.capacity = tr->capacity - inner.rows;
    last.row = tr->row + inner.rows;
    pfin.trace = last.capacity >= 1 ? &last : nullptr;
  }
  int32_t *assign_tmp = assign_out;
  if (!assign_tmp) HIPCHK(pool.get(&assign_tmp, (size_t)n));
  rc = assign_impl(Xr, n, d, Yr, k, nullptr, 0, &pfin, assign_tmp, dist_out);
  if (rc) return rc;
  if (p.rotate) {
    float *Yp = nullptr;
    HIPCHK(pool.get(&Yp, (size_t)k * ds));
    HIPCHK(launch_pad_copy(Yr, d, k, d, Yp, ds, ds, 0, st));
    rc = unrotate_into(Yp, ds, k, d, ds, rot, centroids_out, st);
    if (rc) return rc;
  } else {
    HIPCHK(hipMemcpyAsync(centroids_out, Yr, sizeof(float) * (size_t)k * d, hipMemcpyDeviceToDevice, st));
  }
  HIPCHK(hipEventRecord(e1, st));
  HIPCHK(hipStreamSynchronize(st));
  if (tr) {
    tr->rows = inner.rows + ((pfin.trace && last.rows > 0) ? 1 : 0);
    tr->iters_run = inner.iters_run;
    tr->ms_rotate = 0.f;
    (void)hipEventElapsedTime(&tr->ms_init, e0, e_meso);      // rotation + the whole meso phase
    (void)hipEventElapsedTime(&tr->ms_etr_gt, e_meso, e_fine);  // the whole fine phase
    tr->ms_unrotate = 0.f;
    (void)hipEventElapsedTime(&tr->ms_total, e0, e1);
    host.body_done(tr);
  }
  ws.finished();
  return SKM_OK;
}

}  // namespace

namespace skm {
int report_error(int rc, const char *what) { return fail(rc, what); }
int report_hip_error(hipError_t e, const char *where) { return fail_hip(e, where); }
}  // namespace skm

// ==================================================================== C ABI
extern "C" {
#pragma GCC visibility push(default)

void skm_params_default(skm_params *p) {
  if (!p) return;
  std::memset(p, 0, sizeof(*p));
  p->dprime_frac = 0.125f;
  p->eps0 = 2.1f;
  p->adjust_dprime = 1;
  p->adj_lo = 0.95f;
  p->adj_hi = 0.97f;
  p->adj_step = 0.20f;
  p->split_eps = 1.0f / 1024.0f;
  p->final_assign = 1;
  p->block_stats = 0;
  p->rotate = 1;
  p->etr = 0;
  p->nq = 1000;
  p->topk = 10;
  p->probe_frac = 0.01f;
  p->etr_tol = 0.005f;
  p->etr_patience = 2;
  p->pair_budget = 0;
  p->dense_frac = 0.0125f;
  p->sample_frac = 0.f;
  p->workspace = nullptr;
  p->workspace_bytes = 0;
  p->conv_tol = 0.f;
  p->screen = 0;
  p->tau_group = 0;
}

int64_t skm_workspace_bytes(int64_t n, int32_t d, int32_t k, const skm_params *params) {
  if (n < 1 || n >= (int64_t)1 << 31 || d < 16 || d > 16384 || k < 1 || k > (1 << 24))
    return fail(SKM_EINVAL, "shape out of range");
  skm_params p;
  if (params) p = *params; else skm_params_default(&p);
  const size_t need = fit_workspace_need(n, d, k, p);
  if (!need) return fail(SKM_EINVAL, "pair_budget too large (must stay below 2^32 pairs)");
  return (int64_t)need + 256;   // room to align the caller's pointer
}

int64_t skm_hier_workspace_bytes(int64_t n, int32_t d, int32_t k, const skm_params *params) {
  if (n < 1 || n >= (int64_t)1 << 31 || d < 16 || d > 16384 || k < 1 || k > (1 << 24) || k > n)
    return fail(SKM_EINVAL, "shape out of range");
  skm_params p;
  if (params) p = *params; else skm_params_default(&p);
  const size_t need = hier_workspace_need(n, d, k, p);
  if (!need) return fail(SKM_EINVAL, "pair_budget too large (must stay below 2^32 pairs)");
  return (int64_t)need + 256;   // room to align the caller's pointer
}

int skm_fit(const float *X, int64_t n, int32_t d, int32_t k, int32_t iters, uint64_t seed, float *centroids_out,
            int32_t *assign_out) {
  return fit_impl(X, n, d, k, iters, seed, nullptr, centroids_out, assign_out, nullptr, nullptr);
}

int skm_fit_ex(const float *X, int64_t n, int32_t d, int32_t k, int32_t iters, uint64_t seed, const skm_params *params,
               float *centroids_out, int32_t *assign_out, float *dist_out) {
  return fit_impl(X, n, d, k, iters, seed, params, centroids_out, assign_out, dist_out, nullptr);
}

int skm_fit_host(const float *X_host, int64_t n, int32_t d, int32_t k, int32_t iters, uint64_t seed,
                 const skm_params *params, int64_t batch_rows, float *centroids_out, int32_t *assign_out_host,
                 float *dist_out_host) {
  return fit_host_impl(X_host, n, d, k, iters, seed, params, batch_rows, centroids_out, assign_out_host, dist_out_host);
}

int skm_fit_hierarchical(const float *X, int64_t n, int32_t d, int32_t k, int32_t meso_iters, int32_t fine_iters,
                         uint64_t seed, const skm_params *params, float *centroids_out, int32_t *assign_out,
                         float *dist_out, int64_t *meso_sizes_out_host, int32_t *fine_counts_out_host) {
  return fit_hierarchical(X, n, d, k, meso_iters, fine_iters, seed, params, centroids_out, assign_out, dist_out,
                          meso_sizes_out_host, fine_counts_out_host);
}

int32_t skm_hier_meso_count(int32_t k) { return k >= 1 ? hier_meso_count(k) : 0; }

int skm_hier_alloc(const int64_t *sizes_host, int32_t km, int32_t k, int32_t *counts_out_host) {
  if (!sizes_host || !counts_out_host || km < 1 || k < km) return fail(SKM_EINVAL, "bad arguments");
  int64_t total = 0;
  for (int32_t i = 0; i < km; ++i) {
    if (sizes_host[i] < 0) return fail(SKM_EINVAL, "negative size");
    total += sizes_host[i];
  }
  if (total < k) return fail(SKM_EINVAL, "fewer points than clusters");
  hier_alloc(sizes_host, km, k, counts_out_host);
  return SKM_OK;
}

int skm_assign(const float *X, int64_t n, int32_t d, const float *centroids, int32_t k, const int32_t *prev_assign,
               int32_t *assign_out, float *dist_out) {
  return assign_impl(X, n, d, centroids, k, prev_assign, 0, nullptr, assign_out, dist_out);
}

int skm_assign_ex(const float *X, int64_t n, int32_t d, const float *centroids, int32_t k, const int32_t *prev_assign,
                  int32_t dprime, const skm_params *params, int32_t *assign_out, float *dist_out) {
  return assign_impl(X, n, d, centroids, k, prev_assign, dprime, params, assign_out, dist_out);
}

int skm_assign_exact(const float *X, int64_t n, int32_t d, const float *centroids, int32_t k, void *stream,
                     int32_t *assign_out, float *dist_out) {
  int rc = check_shape(X, n, d, k, false);
  if (rc) return rc;
  if (!centroids || !assign_out) return fail(SKM_EINVAL, "null pointer");
  hipStream_t st = (hipStream_t)stream;
  if (exact_filter_pays(n, d, k)) {
    bool done = false;
    if ((rc = exact_through_filter(X, n, d, centroids, k, st, assign_out, dist_out, done))) return rc;
    if (done) return SKM_OK;
  }
  const int32_t ds = round_up(d, 16);
  // Rows whose length is no multiple of 16, or without alignment, go through a padded copy, 256 MB at a time, unless the
  // multiply can read them as they are: it takes whole float4s and masks the end of the last slab (from 32 dimensions
  // on; where the padded length is a multiple of 32 its 256 x 256 form wants whole slabs).  100 003 x 100 against 1000
  // centroids: 27 of 229 us went into the copy.
  const bool whole = d == ds || (d % 4 == 0 && d >= 32 && ds % 32 != 0);
  const bool pad_x = !whole || !aligned16(X), pad_y = d != ds || !aligned16(centroids);
  const int32_t dx = pad_x ? ds : d;   // dimensions of a row as the kernels below read it
  const int64_t chunk = pad_x ? std::min<int64_t>(n, std::max<int64_t>(((int64_t)64 << 20) / ds, 1024)) : n;
  CallArena ws(((pad_x ? (size_t)chunk * ds : 0) + (pad_y ? (size_t)k * ds : 0) + (size_t)k + split_words(k, ds)) * 4 + (size_t)n * 8 + 8192);
  Pool pool;
  float *Xo = nullptr, *Yo = nullptr, *ynorm = nullptr;
  unsigned long long *best = nullptr;
  unsigned int *amax = nullptr;
  uint32_t *ysplit = nullptr;
  if (pad_x) HIPCHK(pool.get(&Xo, (size_t)chunk * ds));
  if (pad_y) HIPCHK(pool.get(&Yo, (size_t)k * ds));
  HIPCHK(pool.get(&ynorm, (size_t)k));
  HIPCHK(pool.get(&best, (size_t)n));
  HIPCHK(pool.get(&amax, 2));
  HIPCHK(pool.get(&ysplit, split_words(k, ds)));
  HIPCHK(launch_fill_u32(amax, 2, 0u, st));
  OpeningJobs jobs;
  jobs.bound[0] = {X, n * (int64_t)d, amax};
  jobs.bound[1] = {centroids, k * (int64_t)d, amax + 1};
  if (pad_y) {
    jobs.src = centroids; jobs.lds = d; jobs.rows = k; jobs.cols = d;
    jobs.dst = Yo; jobs.ldd = ds; jobs.dpad = ds;
  }
  jobs.fill = best; jobs.nfill = n;
  HIPCHK(launch_opening(jobs, st));
  const float *Yp = pad_y ? Yo : centroids;
  CentroidPrep cp{Yp, ds, k, ds};
  cp.ynorm = ynorm; cp.dn = ds;
  cp.Ys = ysplit; cp.y_absmax = amax + 1;
  HIPCHK(launch_prep_centroids(cp, st));
  for (int64_t r0 = 0; r0 < n; r0 += chunk) {
    const int64_t rows = std::min<int64_t>(chunk, n - r0);
    const float *Xp = X + r0 * d;
    if (pad_x) {
      HIPCHK(launch_pad_copy(Xp, d, rows, d, Xo, ds, ds, 0, st));
      Xp = Xo;
    }
    GemmOperands g{Xp, dx, (int32_t)rows, Yp, ds, k, dx};
    g.a_absmax = amax; g.b_absmax = amax + 1;
    g.b_presplit = ysplit; g.ldbs = split_ld(ds);
    HIPCHK(gemm_argmin(g, ynorm, best + r0, st));
    if (dist_out)   // labels and direct distances in one pass over the rows
      HIPCHK(launch_tau_init(Xp, dx, rows, dx, Yp, ds, nullptr, dist_out + r0, best + r0, st, nullptr, nullptr, nullptr,
                             nullptr, nullptr, assign_out + r0));
  }
  if (!dist_out)
    HIPCHK(launch_finalize_assign(FinalizeArgs{best, nullptr, n, assign_out, nullptr, nullptr, k, nullptr}, st));
  HIPCHK(hipStreamSynchronize(st));
  ws.finished();
  return SKM_OK;
}

int skm_update(const float *X, int64_t n, int32_t d, const int32_t *assign, int32_t k, void *stream, float *centroids,
               int32_t *counts_out) {
  int rc = check_shape(X, n, d, k);
  if (rc) return rc;
  if (!assign || !centroids) return fail(SKM_EINVAL, "null pointer");
  hipStream_t st = (hipStream_t)stream;
  // rows and centroids are read and written where they are, whatever their length and alignment; only the partial sums
  // are padded
  const int32_t ds = round_up(d, 16);
  UpdateWs w{};
  w.max_segments = update_max_segments(n, k);
  const bool stable = stable_order_applies(n, k);
  CallArena ws((size_t)w.max_segments * ds * sizeof(double) + (size_t)n * 4 + (size_t)k * 20 +
               (stable ? (size_t)stable_order_words(n, k) * 4 : 0) + 4096);
  Pool pool;
  unsigned int *flag = nullptr;
  HIPCHK(pool.get(&flag, 1));
  HIPCHK(pool.get(&w.cnt, (size_t)k));
  HIPCHK(pool.get(&w.off, (size_t)k + 1));
  HIPCHK(pool.get(&w.cursor, (size_t)k));
  HIPCHK(pool.get(&w.segoff, (size_t)k + 1));
  HIPCHK(pool.get(&w.order, (size_t)n));
  if (stable) HIPCHK(pool.get(&w.base, (size_t)stable_order_words(n, k)));
  HIPCHK(pool.get(&w.partial, (size_t)w.max_segments * ds));
  PinnedWord bad(st);
  if (!bad.host) return fail(SKM_EHIP, "hipHostMalloc failed");
  const UnsafeLabels unsafe{flag, bad.dev, counts_out};
  HIPCHK(launch_fill_u32(flag, 1, 0u, st));
  HIPCHK(launch_update(X, d, n, d, assign, k, w, centroids, d, st, nullptr, nullptr, 0, -1, &unsafe));
  if (int wrc = bad.wait()) return wrc;
  ws.finished();
  if (*bad.host) return fail(SKM_EINVAL, "assignment label outside [0, k)");
  return SKM_OK;
}

int skm_etr_ground_truth(const float *X, int64_t n, int32_t d, const float *queries, int32_t nq, int32_t topk,
                         void *stream, int64_t *gt_out) {
  if (!X || !queries || !gt_out) return fail(SKM_EINVAL, "null pointer");
  if (n < 1 || n >= (int64_t)1 << 31 || d < 1 || d > 16384) return fail(SKM_EINVAL, "shape out of range");
  if (nq < 1 || topk < 1 || topk > 256) return fail(SKM_EINVAL, "nq >= 1 and 1 <= topk <= 256 required");
  hipStream_t st = (hipStream_t)stream;
  const GtPlan plan = gt_plan(n, d, nq, topk);
  CallArena ws((plan.on ? plan.bytes : gt_full_bytes(n, nq)) + (size_t)nq * topk * 8 + 4096);
  Pool pool;
  unsigned int *amax = nullptr;
  unsigned long long *keys = nullptr;
  HIPCHK(pool.get(&amax, 2));
  HIPCHK(pool.get(&keys, (size_t)nq * topk));
  if (int rc = ground_truth_keys(pool, X, n, d, queries, nq, topk, amax, amax + 1, keys, st)) return rc;
  HIPCHK(launch_keys_to_index(keys, (int64_t)nq * topk, gt_out, st));
  HIPCHK(hipStreamSynchronize(st));
  ws.finished();
  return SKM_OK;
}

int skm_make_rotation(int32_t d, uint64_t seed, void *stream, float *R_out) {
  if (!R_out) return fail(SKM_EINVAL, "null pointer");
  if (d < 1 || d > 16384) return fail(SKM_EINVAL, "d out of range");
  hipStream_t st = (hipStream_t)stream;
  CallArena ws(((size_t)d * d + 20 * 64 * (size_t)d + (size_t)((d + 63) / 64) * 64 * (d + 64) + 8192) * sizeof(double));
  Pool pool;
  int rc = make_rotation_dev(pool, d, seed, st, R_out);
  if (rc) return rc;
  HIPCHK(hipStreamSynchronize(st));
  ws.finished();
  return SKM_OK;
}

int skm_rotate(const float *X, int64_t n, int32_t d, const float *R, int32_t transpose, void *stream, float *out) {
  if (!X || !R || !out) return fail(SKM_EINVAL, "null pointer");
  if (n < 1 || n >= (int64_t)1 << 31 || d < 1 || d > 16384) return fail(SKM_EINVAL, "shape out of range");
  hipStream_t st = (hipStream_t)stream;
  const int32_t ds = round_up(d, 16);
  CallArena ws(((size_t)d * ds + split_words(d, d)) * 4 + 4096);
  Pool pool;
  float *B = nullptr;  // B[c][kk] = R[kk][c] for X R, R[c][kk] for X R^T
  unsigned int *amax = nullptr;
  HIPCHK(pool.get(&B, (size_t)d * ds));
  HIPCHK(pool.get(&amax, 2));
  HIPCHK(launch_fill_u32(amax, 2, 0u, st));
  OpeningJobs jobs;
  jobs.R = R; jobs.d = d; jobs.ld = ds; jobs.r_bound = amax + 1;
  (transpose ? jobs.Rp : jobs.Rtp) = B;
  if (n * (int64_t)d >= 4) jobs.bound[0] = {X, n * (int64_t)d, amax};
  else HIPCHK(launch_absmax(X, d, n, d, amax, st));
  HIPCHK(launch_opening(jobs, st));
  GemmOperands g{X, d, (int32_t)n, B, ds, d, d};
  g.a_absmax = amax; g.b_absmax = amax + 1;
  if (d % 32 == 0) HIPCHK(pool.get(&g.b_split, split_words(d, d)));
  HIPCHK(gemm_store(g, out, d, d, 1.f, 0.f, st));
  HIPCHK(hipStreamSynchronize(st));
  ws.finished();
  return SKM_OK;
}

int skm_sample_rows(uint64_t seed, int64_t n, int32_t k, int64_t *idx_out_host) {
  if (!idx_out_host || n < 1 || k < 0 || k > n) return fail(SKM_EINVAL, "bad arguments");
  sample_rows(seed, STREAM_INIT, n, k, idx_out_host);
  return SKM_OK;
}

float skm_theta_ratio(int32_t d, int32_t t, float eps0) { return (float)theta_ratio(d, t, (double)eps0); }
int32_t skm_dprime_init(int32_t d, float frac) { return dprime_init(d, (double)frac); }
int32_t skm_dprime_adjust(int32_t d, int32_t dprime, double prune_frac, float lo, float hi, float step) {
  return dprime_adjust(d, dprime, prune_frac, (double)lo, (double)hi, (double)step);
}

void skm_debug_gemm_config(int32_t tile256, int32_t panel_cols, int64_t max_tiles) {
  gemm_debug_config(tile256, panel_cols, max_tiles);
}

void skm_release_memory(void) { block_cache().release(); }

const char *skm_strerror(int rc) {
  switch (rc) {
    case SKM_OK: return "ok";
    case SKM_EINVAL: return "invalid argument";
    case SKM_ENOMEM: return "out of memory";
    case SKM_EHIP: return "HIP runtime error";
    case SKM_EINTERNAL: return "internal error";
    case SKM_EOVERFLOW: return "hand-over list overflow";
    default: return "unknown error";
  }
}
const char *skm_last_error(void) { return g_last_error.c_str(); }
const char *skm_version(void) { return "skm 0.2 (gfx950)"; }

#pragma GCC visibility pop
}  // extern "C"
