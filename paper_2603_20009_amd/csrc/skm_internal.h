// Internal declarations shared by the HIP translation units of libskm.
// Nothing here is part of the public ABI (see include/skm.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace skm {

// four floats at any 4-byte boundary: one 16-byte load from global memory (the vector memory path takes unaligned addresses)
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));


constexpr int kBlockDims = 64;  // Section 3.2: trailing dimensions are explored 64 at a time
constexpr int kMaxBlocks = 256; // (16384 - 16) / 64 rounded up
constexpr int kSegPoints = 512; // points per partial-sum segment of the centroid update

// One surviving (point, centroid) pair produced by the first pruning test
// (Algorithm 1, the `likely(distances[i,j] > theta(d', tau))` line inverted).
struct __attribute__((aligned(16))) Pair {
  int32_t i;   // point index (global row)
  int32_t j;   // centroid index in bits 0..23, first trailing block still to be added in bits 24..31
  float p;     // partial squared distance on the dimensions seen so far
  float tau;   // the point's pruning threshold for this step
};

#if defined(__HIPCC__)
typedef __attribute__((address_space(3))) uint32_t *lds_words_t;
// a raw buffer at p, which is uniform (the compiler cannot always tell)
__device__ inline __amdgpu_buffer_rsrc_t uniform_buffer(const void *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>((hi << 32) | lo), 0, (int)0xffffffffu, 0x00027000);
}

// One step of a reduce-scatter of keys over the lanes of a wavefront half: of the two keys, lanes with BIT clear go on
// with the first and lanes with it set with the second, each merged (minimum) with the partner's.
template <int DPP, int BIT>
__device__ inline unsigned long long halve_min(unsigned long long p, unsigned long long q, int lane) {
  const bool up = lane & BIT;
  const unsigned long long keep = up ? q : p, give = up ? p : q;
  const unsigned int lo = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)(unsigned int)give, DPP, 0xF, 0xF, false);
  const unsigned int hi = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)(unsigned int)(give >> 32), DPP, 0xF, 0xF, false);
  const unsigned long long got = ((unsigned long long)hi << 32) | lo;
  return got < keep ? got : keep;
}
// A lane holds a key for each of 32 rows (a, v), a < 2, v < 16, and the 32 lanes of its half share the rows.  Reducing row
// by row takes five exchanges of a 64-bit key per row, 160 in all, each through LDS.  Here the rows are shared out on
// the way (reduce-scatter): a step halves the rows a lane is responsible for, so 16 + 8 + 4 + 2 + 1 exchanges do, on
// the row swap and the lane moves of the vector unit; lane (r32, kh) ends with the smallest key of the row
// (a, v) = (r32 >> 4, r32 & 15) of its half.
template <class F>
__device__ inline unsigned long long reduce_rows32(F key_of, int lane) {
  unsigned long long k8[8];
#pragma unroll
  for (int h = 0; h < 8; ++h) {   // rows v = h and h + 8: lane bit 4 takes a, lane bit 3 takes bit 3 of v
    unsigned long long k16[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const unsigned long long p = key_of(0, h + 8 * u), q = key_of(1, h + 8 * u);
      // rows of 16 lanes: (p0 p1), (q0 q1) -> (p0 q0), (p1 q1)
      const auto lo = __builtin_amdgcn_permlane16_swap((unsigned int)p, (unsigned int)q, false, false);
      const auto hi = __builtin_amdgcn_permlane16_swap((unsigned int)(p >> 32), (unsigned int)(q >> 32), false, false);
      const unsigned long long x = ((unsigned long long)hi[0] << 32) | lo[0], y = ((unsigned long long)hi[1] << 32) | lo[1];
      k16[u] = x < y ? x : y;
    }
    k8[h] = halve_min<0x128, 8>(k16[0], k16[1], lane);   // row_ror:8
  }
  unsigned long long k4[4];
#pragma unroll
  for (int h = 0; h < 4; ++h) k4[h] = halve_min<0x141, 4>(k8[h], k8[h + 4], lane);   // row_half_mirror
  const unsigned long long k2a = halve_min<0x4E, 2>(k4[0], k4[2], lane);             // quad_perm [2,3,0,1]
  const unsigned long long k2b = halve_min<0x4E, 2>(k4[1], k4[3], lane);
  return halve_min<0xB1, 1>(k2a, k2b, lane);                                         // quad_perm [1,0,3,2]
}
// The same of a float per row (fminf: a NaN counts only where there is nothing else).
template <int DPP, int BIT>
__device__ inline float halve_min_f32(float p, float q, int lane) {
  const bool up = lane & BIT;
  const float keep = up ? q : p, give = up ? p : q;
  return fminf(keep, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, give), DPP, 0xF, 0xF, false)));
}
template <class F>
__device__ inline float reduce_rows32_f32(F value_of, int lane) {
  float k8[8];
#pragma unroll
  for (int h = 0; h < 8; ++h) {
    float k16[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned int, value_of(0, h + 8 * u)),
                                                      __builtin_bit_cast(unsigned int, value_of(1, h + 8 * u)), false, false);
      k16[u] = fminf(__builtin_bit_cast(float, (unsigned int)r[0]), __builtin_bit_cast(float, (unsigned int)r[1]));
    }
    k8[h] = halve_min_f32<0x128, 8>(k16[0], k16[1], lane);
  }
  float k4[4];
#pragma unroll
  for (int h = 0; h < 4; ++h) k4[h] = halve_min_f32<0x141, 4>(k8[h], k8[h + 4], lane);
  const float k2a = halve_min_f32<0x4E, 2>(k4[0], k4[2], lane), k2b = halve_min_f32<0x4E, 2>(k4[1], k4[3], lane);
  return halve_min_f32<0xB1, 1>(k2a, k2b, lane);
}
// The first `valid` of four values at any 4-byte boundary, zeros behind them: one load unless the row ends among them (X R of 46 467 x
// 495 with a load a value: 441 us, now 245; the fp16 copy of 131 072 x 357 points 67 -> 51).
__device__ inline float4 load4_any(const float *p, int valid) {
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (valid >= 4) {
    const f32x4_u u = *reinterpret_cast<const f32x4_u *>(p);
    v = make_float4(u.x, u.y, u.z, u.w);
  } else {
    if (valid > 0) v.x = p[0];
    if (valid > 1) v.y = p[1];
    if (valid > 2) v.z = p[2];
  }
  return v;
}
#endif

int num_cus();   // compute units of the current device

// Error reporting shared by the translation units that hold entry points: records the text skm_last_error() returns
// on this thread and gives back the code (SKM_ENOMEM for an out-of-memory HIP error, SKM_EHIP for any other).
int report_error(int rc, const char *what);
int report_hip_error(hipError_t e, const char *where);

// ---- order-preserving float <-> uint32 map (for packed 64-bit atomic min) ----
__host__ __device__ inline uint32_t f2ord(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__host__ __device__ inline float ord2f(uint32_t u) {
  u = (u & 0x80000000u) ? (u & 0x7fffffffu) : ~u;
  return __builtin_bit_cast(float, u);
}
__host__ __device__ inline uint64_t pack_key(float v, int32_t idx) {
  return ((uint64_t)f2ord(v) << 32) | (uint32_t)idx;
}

// Times of a call's stages without commands of their own: a kernel at a stage's border stores the device's constant
// clock (100 MHz) as its first workgroup starts.  (An event record cost 5 us of host and stream time each, a quarter of
// a small fit.)  NULL: no stamp.
typedef unsigned long long stamp_t;
__device__ inline void put_stamp(stamp_t *stamp) {
  if (stamp && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *stamp = wall_clock64();
}

// ---------------------------------------------------------------- GEMM family
// C-shaped work: scores s(i, j) = sum_k A[i][k] * B[j][k] for an M x K row-major A and an
// N x K row-major B (both K-contiguous), on fp32 MFMA, with one of three fused epilogues.
struct GemmOperands {
  const float *A;
  int64_t lda;
  int32_t M;
  const float *B;
  int64_t ldb;
  int32_t N;
  int32_t K;
  int32_t panel_cols = 16;  // column tiles per panel of the tile walk (set by the launcher)
  // Device words holding the bit pattern of an upper bound of |A| and of |B| (see launch_absmax).  With both
  // set (and 16-byte aligned operands, K >= 32) the product runs in the split-fp16 form described below.
  const unsigned int *a_absmax = nullptr;
  const unsigned int *b_absmax = nullptr;
  // Optional workspace of N * (K + 32) words, 16-byte aligned: with it (and the bounds above, K a multiple of 32) a
  // tall product splits B into fp16 pairs there first and runs on 256 x 256 tiles.  b_presplit: such a copy (row stride
  // ldbs words, rows of K columns or more, scaled by *b_absmax) that the caller has already, used instead.
  uint32_t *b_split = nullptr;
  const uint32_t *b_presplit = nullptr;
  int64_t ldbs = 0;
  stamp_t *stamp = nullptr;
};

// Split-fp16 arithmetic.  A matrix whose largest magnitude is m is scaled by the power of two that brings m
// into [2^14, 2^15); a scaled value v is staged as hi = fp16(v) and lo = fp16(v - hi), which keeps 22
// significant bits of v (and an absolute error below 2^-40 m for values too small for that), and a product
// is taken as hi*hi' + hi*lo' + lo*hi' on v_mfma_f32_32x32x16_f16 with fp32 accumulation.  The dropped
// lo*lo' term is 2^-22 of the product.  Scaling by powers of two is exact, so the result is that of an fp32
// GEMM whose inputs were rounded to 22 bits.
__device__ inline float split_scale(unsigned int absmax_bits) {   // 2^(14 - floor(log2 m)), clamped to normal floats
  int e = 268 - (int)(absmax_bits >> 23);
  e = e < 1 ? 1 : (e > 253 ? 253 : e);
  return __builtin_bit_cast(float, (unsigned int)e << 23);
}
__device__ inline float split_unscale(unsigned int absmax_bits) {  // exactly 1 / split_scale
  int e = 268 - (int)(absmax_bits >> 23);
  e = e < 1 ? 1 : (e > 253 ? 253 : e);
  return __builtin_bit_cast(float, (unsigned int)(254 - e) << 23);
}
// *out = max(*out, bit pattern of max |A[i][j]|) over rows x cols; *out must hold 0 (or an earlier bound) before.
// max_blocks > 0 limits the grid (a pass that shares the device with other work should not take every wavefront slot).
hipError_t launch_absmax(const float *A, int64_t lda, int64_t rows, int32_t cols, unsigned int *out, hipStream_t st,
                         int max_blocks = 0);

// C[i][j] = alpha * s(i,j) + beta * C[i][j] for j < N; columns N <= j < Nstore are written as 0.
// If c_absmax is given, max |C| is folded into *c_absmax (as launch_absmax does).
hipError_t gemm_store(const GemmOperands &g, float *C, int64_t ldc, int32_t Nstore, float alpha, float beta,
                      hipStream_t st, unsigned int *c_absmax = nullptr);
// C and D (rows of ldc) = the products g and h, which share B; in one launch where neither is tall or large tiles fill the device
hipError_t gemm_store_two(const GemmOperands &g, float *C, unsigned int *c_absmax, const GemmOperands &h, float *D, unsigned int *d_absmax,
                          int64_t ldc, int32_t Nstore, hipStream_t st);

// best[i] = min(best[i], pack_key(ynorm[j] - 2 s(i,j), j)) over all j: the row argmin of the squared
// distance up to the per-row constant ||x_i||^2 (Algorithm 1, iteration 1).
hipError_t gemm_argmin(const GemmOperands &g, const float *ynorm, unsigned long long *best, hipStream_t st);

// Launch choices of the GEMM family that tests force (process-wide; nothing here changes what is computed):
// tile256 -1 = by shape, 0 = never the 256 x 256 form, 1 = whenever the operands allow it; panel_cols > 0 = width of
// the tile walk's panels; max_tiles > 0 = tiles per launch (tall problems are cut into bands of row tiles).
void gemm_debug_config(int tile256, int panel_cols, int64_t max_tiles);

// Device scalars of one assignment step.  Every workgroup adds to the replica (blockIdx & (kStatReplicas-1))
// so that same-address atomics do not serialise; the host sums the replicas.
enum { SC_COMPLETED = 0, SC_CHANGED = 1, SC_SURVIVORS = 2, SC_DENSE_DIMS = 3, SC_DENSE_PB = 4, SC_GATHER_PB = 5,
       SC_GATHER_PAIRS = 6, SC_SCREEN_DIMS = 7, SC_LISTED_TILES = 8, SC_ENTER = 9, SC_COUNT = 9 + kMaxBlocks };
constexpr int kStatReplicas = 32;
// The hand-over list is split in kSubLists equal parts, one per XCD (workgroup id mod 8), each with its own
// fill counter (counters are kSubListStride words apart).
constexpr int kSubLists = 8;
constexpr int kSubListStride = 16;
constexpr int kListCols = 256;   // columns of a tile of listed centroids
constexpr int kListGroup = 8;    // row tiles whose listed tiles are placed in turn

// Progressive-pruning GEMM (Algorithm 1, iterations >= 2): a 128 x 256 tile is multiplied densely over
// d', d'+64, d'+128, ... dimensions; after each step the pairs whose partial distance exceeds
// theta(t, tau_i) die; the tile stops when nothing is alive, hands its pairs to the gather kernel when
// at most emit_max are alive, and offers finished distances below tau_i to best[] at t = d.
// Rows are local to the chunk: global row = row_base + i; tau/prev/best are indexed by global row.
// Split-fp16 copy of a matrix in the byte order of the progressive kernel's LDS tiles (launch_split_rows): row stride
// split_ld(ds) words.  Granule g + 1 of a row, dims 16 g .. 16 g + 15, is 16 words: 8 of hi halves, 8 of lo halves of the
// values scaled by split_scale(*absmax); granule 0 and the one behind the row's data are zero.  Rows lie in pairs: word
// split_row(r, ld) + 32 g is where granule g of row r starts, the two rows' granules g side by side in 128 bytes.
// What a tile kernel loads of a row at a time is 64 bytes (four lanes of a global -> LDS load), and the load unit takes a
// line of 128 bytes every two clocks whether all of it is wanted or half: 17 TB/s of 64-byte pieces from the L2s where two
// neighbours share a line 32 (gathered pieces across two lines 18).  In pairs of rows, dense tiles of 1M x 1536, k = 1024,
// took 10.0 instead of 10.75 ms, the one-product multiply of all their pairs 2.9 instead of 4.1 (there the rows used to
// start in the middle of a 64-byte block as well).
// The hi halves once more as a plane of their own (what the low-precision filter reads): split_ld(ds) / 2 words a row, unit
// u (dims 32 u .. 32 u + 31) of row r at word split_row(r, split_ld(ds) / 2) + 32 u; a last unit of 16 dims ends in zeros.
// Buffers hold an even number of rows; the odd one out is never read.
__host__ __device__ inline int32_t split_ld(int32_t ds) { return (ds + 31) / 32 * 32 + 32; }
__host__ __device__ inline int64_t split_row(int64_t r, int64_t ld) { return (r >> 1) * (2 * ld) + 16 * (r & 1); }
inline size_t split_words(int64_t rows, int32_t ds) { return (size_t)((rows + 1) / 2 * 2) * (size_t)split_ld(ds); }
hipError_t launch_split_rows(const float *A, int64_t lda, int64_t rows, int32_t ds, const unsigned int *absmax,
                             uint32_t *out, hipStream_t st);

struct ProgArgs {
  const uint32_t *A;       // split-fp16 copy of the rotated points of the chunk (launch_split_rows)
  int64_t lda;             // split_ld(ds)
  int32_t M;
  const uint32_t *B;       // split-fp16 copy of the rotated centroids
  int64_t ldb;
  int32_t N;
  const unsigned int *a_absmax, *b_absmax;   // the bounds the copies were scaled by
  int32_t ds, d, dprime, nb;
  const float *ratio;      // [nb + 1] theta ratio at checkpoint m (t_m = min(d, d' + 64 m)); device array
  const float *tau;        // [n]
  const int32_t *prev;     // [n] incumbent (never a challenger)
  int64_t row_base;
  const float *xnp;        // [ds / 16][xn_stride] ||x_i[0 : 16 (p + 1))||^2, indexed like tau (row_base + tile row)
  int64_t xn_stride;
  const float *ynp;        // [nb + 1][N] ||y_c[0 : t_m)||^2
  Pair *pairs;             // kSubLists parts of sub_capacity slots each
  unsigned int *pair_count;   // [kSubLists * kSubListStride] fill counters of the parts
  unsigned int *tile_counter; // [8 * kSubListStride] next tile of every XCD's range; zero before the launch
  unsigned int sub_capacity;
  unsigned int *overflow;
  unsigned int emit_max;   // a tile with at most this many alive pairs is handed over
  unsigned long long *best;       // [n] packed (distance, centroid)
  unsigned long long *scal;       // [kStatReplicas][SC_COUNT] step scalars (SC_SURVIVORS, SC_COMPLETED, SC_DENSE_*, SC_ENTER..)
  int32_t block_stats;            // also count pairs entering every trailing block (SC_ENTER + m)
  // Listed columns (after launch_screen; all NULL otherwise): tile t is row tile tile_rt[t].x against the 256 centroids
  // col_list[256 t ..] (ascending ids, -1 = none); *ntiles tiles in all.
  // prev then holds the position of the incumbent in the row tile's list (-1 = not listed), and tile_rt[t] also how many of
  // the list's columns come before the tile.
  const int2 *tile_rt = nullptr;
  const int32_t *col_list = nullptr, *ntiles = nullptr;
  // Listed columns only: one product and widened tests behind the first test (deep = 1).  Ah: the plane of hi
  // halves; Bh: those of the centroids, dims d' + 32 u .. of row r at word split_row(r, ldb) + 32 (d' / 32 + u) (rows as far
  // apart as B's: one offset serves both; a listed row's units lie in whole blocks of 64 bytes for every d'); widen[m] = (widening per unit of the row's norm behind d', guard) of checkpoint m.  A tile hands over at
  // the first test with at most emit_first pairs alive, later with at most emit_deep columns (of half a tile's rows) that
  // hold any; one with more than deep_max pairs alive at the first test takes three products throughout.  A test every
  // deep_stride blocks.
  int32_t deep = 0;
  const uint32_t *Ah = nullptr, *Bh = nullptr;
  const float2 *widen = nullptr;
  unsigned int emit_first = 0, emit_deep = 0, deep_max = 0;
  int32_t deep_stride = 1;
  stamp_t *stamp = nullptr;
};
hipError_t launch_progressive(const ProgArgs &g, hipStream_t st);

// Low-precision first filter (screen.hip): one fp16 product on the first d' dimensions and the first test
// theta(d', tau) widened by the error bound of the dropped halves; then, per row tile of 128 points, the centroids
// that some point of the tile may still pass, as an ascending id list padded with -1 to a multiple of 256.
// Outputs: cnt[row tiles], first[row tiles] (tiles of 256 listed columns before every row tile), *ntiles,
// col_list[256 * ntiles], tile_rt[ntiles] (see ProgArgs); capacity needed: one tile per (row tile, column tile) of the full problem.
struct ScreenLaunch {
  int32_t all = 0;               // no filter: every column of every row tile is listed
  const uint32_t *A; int64_t lda; int32_t M;
  const uint32_t *B; int64_t ldb; int32_t N;
  const unsigned int *a_absmax, *b_absmax;
  int32_t ds, dprime;
  float ratio0;              // theta(d', tau) / tau
  const float *tau;          // [n], indexed by row_base + row
  int64_t row_base;
  const float *xn;           // [n] ||x_i[0 : d')||^2, indexed like tau
  const float *yn;           // [N] ||y_j[0 : d')||^2
  float *arow, *ycol;        // scratch: [M] and [N] (the test's per-point and per-centroid terms)
  const float *ynp = nullptr;   // (first test) [nb + 1][N] prefix norms of the centroids, row 0 = yn; with it widen[0 .. nb]
  int32_t nb = 0;               // receives the terms of the later, widened tests (ProgArgs)
  float2 *widen = nullptr;
  uint32_t *colmask;         // scratch: [row tiles][4 * column tiles]
  int32_t *cnt, *first, *ntiles, *col_list;   // (ntiles: two words, the second is scratch)
  int2 *tile_rt;
  const int32_t *prev;       // (first test) [n] incumbents, indexed like tau; list_pos[row_base + row] receives the position
  int32_t *list_pos;         // of a row's incumbent in its row tile's list, -1 if it is not listed
  unsigned long long *scal;     // step scalars (SC_SCREEN_DIMS)
  // Exact mode (iteration 1: dprime = ds, xn / yn the full norms, tau and ratio0 unused, no column lists): for every
  // point the centroids that can be its nearest are appended to `pairs` (partial distance 0, first block 0, no
  // threshold) for the gather kernel, which finishes their exact distances.  rowmin: [n] words of 0xffffffff before
  // the first launch of the step, indexed by row_base + row.
  int exact = 0;
  unsigned int *rowmin = nullptr;
  Pair *pairs = nullptr;
  unsigned int *pair_count = nullptr;
  unsigned int sub_capacity = 0;
  unsigned int *overflow = nullptr;
  stamp_t *stamp = nullptr;
};
hipError_t launch_screen(const ScreenLaunch &a, hipStream_t st);

// The same one-product multiply for the ground truth (etr.hip): rows are queries, columns points.  A, B: planes of fp16
// values, ds a multiple of 32, row stride ds / 2 words, every row scaled by row_scale[i] / col_scale[j];
// col_term[j] = ||x_j||^2 col_scale[j] / 2.  groups: group_min[i][group0 + j / 64] = smallest score ||x||^2 - 2 q.x of the
// 64 columns.  Otherwise every column with a score <= t_i, row_term[i] = -t_i row_scale[i] / 2, is appended to cand[i].
struct NeighbourLaunch {
  const uint32_t *A, *B;
  int32_t M, N, ds;
  const float *row_term, *row_scale, *col_term, *col_scale;
  float *group_min;
  int32_t ngroups, group0;
  unsigned long long *cand;    // [M][cand_cap]: (order-preserving bits of the score << 32) | point
  unsigned int *cand_count;    // [M]; may exceed cand_cap
  unsigned int cand_cap;
  int64_t point0;
};
hipError_t launch_neighbour_screen(const NeighbourLaunch &a, bool groups, hipStream_t st);
int64_t progressive_tiles(int64_t rows, int32_t k);
int32_t progressive_tile_pairs();

// ---------------------------------------------------------------- pruning
struct PruneArgs {
  const Pair *pairs;           // kSubLists parts of sub_capacity slots each
  const unsigned int *count;   // [kSubLists * kSubListStride] fill counters
  unsigned int sub_capacity;
  const float *Xr;       // rotated points, row stride ldx, zero padded to ds columns
  int64_t ldx;
  int64_t n;             // number of points (entries naming a point beyond it are skipped)
  const float *Ypdx;     // [nb][k][64] trailing centroid dimensions, block-major (PDX-style)
  int32_t k;
  int32_t dprime;
  int32_t ds;            // padded row length (multiple of 16)
  int32_t nb;            // trailing blocks
  const float *Y;        // rotated centroids, row stride ds: the first d' dimensions of a pair that starts over (p < 0)
  const float *ratio;    // [nb + 1] theta ratio at checkpoint m, t_m = min(d, d' + 64 m) (device array)
  unsigned long long *best;        // [n] packed (distance, centroid)
  unsigned long long *scal;        // [kStatReplicas][SC_COUNT]: SC_COMPLETED, SC_GATHER_*, and SC_ENTER + m when block_stats
  int32_t block_stats;
  stamp_t *stamp = nullptr;
};
hipError_t launch_prune(const PruneArgs &a, hipStream_t st);

// The candidates of a search over the first K dimensions in which no pair is dropped, a point with all of its own at a time;
// what does not fit a point's slots is left to launch_prune on pairs + sub_capacity / 2 and left_count.  A part of the list that is
// more than half full sets bit 0 of *overflow.
constexpr float kFarAway = 3.0e38f;   // the threshold of such pairs
struct RowPairsArgs {
  Pair *pairs;                 // kSubLists parts of sub_capacity slots each
  const unsigned int *count;   // [kSubLists * kSubListStride] fill counters
  unsigned int sub_capacity;
  unsigned int *overflow;
  unsigned int *left_count;    // [kSubLists * kSubListStride], zero
  unsigned int *row_count;     // [rows], cleared here
  int32_t *cand;               // [rows][slots]
  int32_t slots, rows;
  int64_t row_base;            // point of row 0
  const float *Xr;             // all points
  int64_t ldx;
  const float *Ypdx;           // [nb][k][64]: the first K dimensions, zero filled
  int32_t k, K, nb;
  unsigned long long *best;    // by point
  unsigned long long *scal;
};
hipError_t launch_row_pairs(const RowPairsArgs &a, hipStream_t st);

// ---------------------------------------------------------------- streaming kernels
// tau_i = ||x_i - y_{a_i}||^2 over all dims, best_i = pack(tau_i, a_i)
// (Algorithm 1, "Initial pruning threshold").  Either output may be NULL.
// With xnp ([ds / 16][n], ds a multiple of 16) the same pass writes the table of prefix norms
// xnp[p][i] = ||x_i[0 : 16 (p + 1))||^2 that the progressive kernel reads at its checkpoints; with xs also the
// split-fp16 copy of the points (the layout of launch_split_rows, scaled by the bound *x_absmax).
// Regrouping (order, xr_out, label_out: all or none): output slot p of every array above takes point order[p] (a
// permutation of 0 .. n - 1); the row of that point is copied to xr_out[p] (row stride ds) and its label to
// label_out[p].  `assign` is still indexed by point.
// xh (optional, with xs): also the plane of hi halves of launch_split_rows' out_hi.
// assign = NULL: the labels are the low halves of best[] (packed keys of an argmin); a point whose key is ~0 takes label 0
// and sets bit 1 of *unset (optional).  label_out without order receives the label of every point.
// The thresholds of the last step, kept where a point's cluster was not touched since (touched[c], NULL: none was): tau[] in
// and out, best[] out.
constexpr int32_t kTauKeptMaxDims = 2048;
hipError_t launch_tau_kept(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const float *Y, int64_t ldy, const int32_t *assign,
                           const uint32_t *touched, float *tau, unsigned long long *best, hipStream_t st, stamp_t *stamp);
hipError_t launch_mark_touched(const int32_t *labels, int32_t m, int32_t k, uint32_t *touched, hipStream_t st);
hipError_t launch_tau_init(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const float *Y, int64_t ldy,
                           const int32_t *assign, float *tau, unsigned long long *best, hipStream_t st,
                           float *xnp = nullptr, uint32_t *xs = nullptr, const unsigned int *x_absmax = nullptr,
                           const int32_t *order = nullptr, float *xr_out = nullptr, int32_t *label_out = nullptr,
                           uint32_t *xh = nullptr, unsigned int *unset = nullptr, stamp_t *stamp = nullptr);
// dst[idx[p]] = src[p] for 4-byte items
hipError_t launch_scatter_by_index(const void *src, const int32_t *idx, int64_t n, void *dst, hipStream_t st);
// order_out = order_in (points grouped by cluster, segment c = [off[c], off[c+1])) with every segment stably sorted by
// the signs of the first four dimensions of its points.  key_scratch: n bytes.
hipError_t launch_suborder(const float *Xr, int64_t ldx, int64_t n, int32_t k, const int32_t *off, const int32_t *order_in,
                           unsigned char *key_scratch, int32_t *order_out, hipStream_t st);
hipError_t launch_compose(const int32_t *a, const int32_t *b, int64_t n, int32_t *out, hipStream_t st);   // out[p] = a[b[p]]
// keys hold a point id in their low 32 bits (packed (distance, point) keys; ~0 = none): every id becomes the position
// p with perm[p] = id.  inv_scratch: n ints.
hipError_t launch_remap_key_ids(unsigned long long *keys, int64_t m, const int32_t *perm, int64_t n, int32_t *inv_scratch,
                                hipStream_t st);

// What a step needs from the centroids (all outputs optional), and two jobs of the step's start that ride along: words to
// clear and theta ratios (a host array, copied into the launch) to store on the device.  Y 16-byte aligned, ldy a
// multiple of 4, ds, dn and dprime multiples of 16.
struct CentroidPrep {
  const float *Y;
  int64_t ldy;
  int32_t k, ds;
  float *ynorm = nullptr;      // [k] ||Y[c][0 : dn)||^2
  int32_t dn = 0;
  int32_t dprime = 0, nb = 0;
  float *Ypdx = nullptr;       // [nb][k][64] block-major copy of the dims from dprime on, zero filled past column pdx_cols
  int32_t pdx_cols = 1 << 30;
  float *ynp = nullptr;        // [nb + 1][k] prefix norms at the checkpoints min(ds, dprime + 64 m)
  uint32_t *Ys = nullptr;      // split-fp16 copy (launch_split_rows), scaled by the bound *y_absmax
  uint32_t *Yh = nullptr;      // its plane of hi halves, zero from dimension hi_dims on
  int32_t hi_dims = 0;
  uint32_t *Yd = nullptr;      // the hi halves from dprime on (with Ys; see ProgArgs::Bh)
  const unsigned int *y_absmax = nullptr;
  unsigned int *clear = nullptr;
  int64_t clear_words = 0;
  float *ratio_out = nullptr;
  stamp_t *stamp = nullptr;
};
struct ThetaRatios {
  int n;
  float v[kMaxBlocks + 1];
};
// thresholds (optional, ds <= 256): those of launch_tau_init for labelled rows, against the same centroids
struct ShortThresholds {
  const float *Xr;
  int64_t ldx, n;
  const int32_t *labels;
  float *tau;
  unsigned long long *best;
};
hipError_t launch_prep_centroids(const CentroidPrep &a, hipStream_t st, const float *ratio = nullptr, int nratio = 0,
                                 const ShortThresholds *thresholds = nullptr);

// every non-zero row of A scaled to unit Euclidean length, in place (cols, lda multiples of 4; A 16-byte aligned)
// (absmax, optional: max |A| of the scaled rows is folded into it)
hipError_t launch_normalize_rows(float *A, int64_t lda, int64_t rows, int32_t cols, hipStream_t st,
                                 unsigned int *absmax = nullptr);

hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t st);
hipError_t launch_fill_u32(unsigned int *p, int64_t n, unsigned int v, hipStream_t st, stamp_t *stamp = nullptr);
hipError_t launch_stamp(stamp_t *stamp, hipStream_t st);   // a stamp with no kernel to carry it

// What the last kernel of a step writes into page-locked host memory.
struct StepReport {
  double objective;          // sum over the points of the squared distance found
  unsigned int flag;         // bit 0: list overflow, bit 1: a point without a centroid, bit 2: a label of the caller's outside [0, k)
  int32_t nempty, largest;   // of the cluster sizes
  unsigned int seq;          // FinalizeArgs::seq, written when all else is there
  unsigned long long scal[SC_COUNT];   // the step scalars, replicas added up; SC_CHANGED = points with another label than prev
};
// Unpack best -> assign, dist (not if *flag is set already); cluster sizes into cnt[k] (zero before).  With `done` (a zero word) the launch also closes
// the step: see finalize_assign_kernel.
struct FinalizeArgs {
  const unsigned long long *best;
  const int32_t *prev;        // [n] or NULL
  int64_t n;
  int32_t *assign;
  float *dist;                // or NULL
  int32_t *cnt;               // or NULL
  int32_t k;
  unsigned int *flag;         // or NULL
  unsigned int *done = nullptr;
  double *obj_partial = nullptr;      // [finalize_blocks(n)]
  int32_t *change_start = nullptr;    // [finalize_blocks(n)] changed points before the points of each workgroup
  unsigned long long *scal = nullptr;   // [kStatReplicas][SC_COUNT]; its first SC_CHANGED receives the changed points
  int nscal = SC_COUNT;               // scalars to report
  StepReport *report = nullptr;       // device-visible address of the page-locked block
  unsigned int seq = 0;               // number of the report
  stamp_t *stamp = nullptr, *stamp_end = nullptr;   // start and (of the closing workgroup) end
};
hipError_t launch_finalize_assign(const FinalizeArgs &a, hipStream_t st);
int64_t finalize_blocks(int64_t n);
// cnt[l] += number of i with assign[i] = l; labels outside [0, k) are left out and set bit 2 of *flag (optional)
hipError_t launch_histogram(const int32_t *assign, int64_t n, int32_t k, int32_t *cnt, unsigned int *flag, hipStream_t st);
hipError_t launch_copy_labels(const int32_t *a, int64_t n, int32_t k, int32_t *out, unsigned int *flag, hipStream_t st);

// Centroid update (Section 3.2) as a segmented reduction.
struct UpdateWs {
  int32_t *cnt;        // [k]   cluster sizes (input)
  int32_t *off;        // [k+1] exclusive scan of cnt
  int32_t *cursor;     // [k]
  int32_t *segoff;     // [k+1] exclusive scan of ceil(cnt / kSegPoints)
  int32_t *order;      // [n]   point ids grouped by cluster
  int32_t *base = nullptr;   // [stable_order_words(n, k)] where stable_order_applies(n, k); NULL otherwise
  double *partial;     // [max_segments][ds]
  int64_t max_segments;
};
int64_t update_max_segments(int64_t n, int32_t k);
bool stable_order_applies(int64_t n, int32_t k);
int64_t stable_order_words(int64_t n, int32_t k);   // of `base` below, for n points or fewer
// The grouping half of launch_update alone: cnt[k] sizes, off[k+1] starts, order[n] point ids grouped by label (cursor[k]
// and segoff[k+1] are scratch; base as in UpdateWs, or NULL).
hipError_t launch_group_order(const int32_t *labels, int64_t n, int32_t k, int32_t *cnt, int32_t *off, int32_t *cursor,
                              int32_t *segoff, int32_t *order, int32_t *base, hipStream_t st);
// order_out[] = order[] with the points of low thresholds first (stably, in a few classes; see there).  quarters = 0: the
// classes of a tail; else that many (at most six) of equal size.  bin[n], cls[n] and words[threshold_class_words(n)] are scratch.
int64_t threshold_class_words(int64_t n);
// *above = how many of every 16th point have a threshold that puts them into a class of its own (tau, bin and words as above)
hipError_t launch_threshold_sample(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const float *Y, int64_t ldy,
                                   const int32_t *labels, float *tau, int32_t *bin, int32_t *words, int32_t *above, hipStream_t st);
bool thresholds_have_tail(int64_t n, int32_t above);
hipError_t launch_threshold_classes(const float *tau, int64_t n, int quarters, const int32_t *order, int32_t *bin, int32_t *cls,
                                    int32_t *words, int32_t *order_out, hipStream_t st);
// largest cluster whose members launch_update leaves sorted by index in w.order (larger ones: any order)
int32_t update_sort_cap();
// S (optional, [k][ds] fp64) receives the sum of every cluster; y_absmax (optional) the bit pattern of max |Y| of
// the new centroids (the launcher clears it first).  With `accumulate` the sums of these n points are added to S
// instead (one batch of a larger update); Y may then be NULL, and launch_means_from_sums finishes the update.
// largest: the largest cluster size if known, else -1.  unsafe: the labels are a caller's, unchecked, and w.cnt is not
// known yet: they are counted first, and if one lies outside [0, k) nothing but *flag_host is written.
struct UnsafeLabels {
  unsigned int *flag;        // a zero word
  unsigned int *flag_host;   // receives it (device-visible)
  int32_t *counts_out;       // [k] or NULL: the sizes
};
hipError_t launch_update(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const int32_t *assign, int32_t k,
                         const UpdateWs &w, float *Y, int64_t ldy, hipStream_t st, double *S = nullptr,
                         unsigned int *y_absmax = nullptr, int accumulate = 0, int32_t largest = -1,
                         const UnsafeLabels *unsafe = nullptr);
hipError_t launch_add_counts(const int32_t *cnt, int32_t k, int32_t *total, hipStream_t st);
hipError_t launch_means_from_sums(const double *S, const int32_t *cnt, int32_t k, int32_t ds, float *Y, int64_t ldy,
                                  unsigned int *y_absmax, hipStream_t st);

// Workspace of the incremental update: room for 2 * (points that changed label) entries.
struct IncUpdateWs {
  int32_t *ent_id;     // [capacity] point id, or ~id for a point that left the cluster
  int32_t *ent_lab;    // [capacity] cluster of the entry
  int32_t *order;      // [capacity]
  int32_t *cnt, *off, *cursor, *segoff;   // [k], [k+1], [k], [k+1]
  int32_t *base = nullptr;                // [stable_order_words(capacity, k)], or NULL
  double *partial;     // [max_segments][ds]
  int64_t capacity, max_segments;
};
// Centroids from the cluster sums S of the previous update and the points whose label changed since
// (Section 3.2, the same means computed from the difference).
hipError_t launch_update_incremental(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const int32_t *assign,
                                     const int32_t *prev, int64_t changed, const int32_t *change_start, int32_t k,
                                     const UpdateWs &w, const IncUpdateWs &inc, double *S, float *Y, int64_t ldy,
                                     hipStream_t st, unsigned int *y_absmax = nullptr);
// The same, launched before the host knows how many labels changed: it does nothing where none did, more than `most`, or *flag is
// set.  The sums, the means and *y_absmax are then as they were.
struct UpdateAhead {
  const unsigned long long *changed = nullptr;   // of the finalize kernel (scal[SC_CHANGED])
  const unsigned int *flag = nullptr;
  int64_t most = 0;                              // at most update_ahead_most
  __device__ int entries() const {
    const unsigned long long c = *changed;
    return c > (unsigned long long)most || *flag != 0u ? 0 : 2 * (int)c;
  }
};
int64_t update_ahead_most(int32_t ds, int32_t k, int64_t capacity);   // what the direct form takes (launch_update_incremental)
hipError_t launch_update_ahead(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const int32_t *assign, const int32_t *prev,
                               const int32_t *change_start, int32_t k, const UpdateWs &w, const IncUpdateWs &inc, double *S,
                               float *Y, int64_t ldy, const UpdateAhead &ahead, hipStream_t st, unsigned int *y_absmax);

// Empty-cluster splits: pairs_dev = (empty, donor) pairs grouped into chains (splits that share a cluster, in the
// host's order); chain_first_dev[c] .. chain_first_dev[c + 1] are the splits of chain c.  One workgroup per chain.
hipError_t launch_split(float *Y, int64_t ldy, int32_t d, const int32_t *pairs_dev, const int32_t *chain_first_dev,
                        int32_t nchains, float eps, hipStream_t st);
// dst[c] = src[idx[c]] (idx: device or page-locked host memory), zero padded to dpad; max |.| folded into *absmax (optional)
hipError_t launch_gather_rows(const float *src, int64_t lds, int32_t d, const int64_t *idx, int32_t k, float *dst,
                              int64_t ldd, int32_t dpad, hipStream_t st, unsigned int *absmax = nullptr,
                              stamp_t *stamp = nullptr);
// Jobs that open a call, independent of each other, in one launch: the bounds of the operands, the copies of the rotation matrix, a
// padded copy, keys set to ~0.
struct OpeningJobs {
  struct Bound {
    const float *A = nullptr;      // count >= 4 values without gaps
    int64_t count = 0;
    unsigned int *out = nullptr;   // max |A| is folded into it
  } bound[2];
  const float *R = nullptr;        // d x d: Rp = R, Rtp = R^T (either may be NULL), rows of ld, zero padded; max |R| folded into r_bound
  int32_t d = 0, ld = 0;
  float *Rp = nullptr, *Rtp = nullptr;
  unsigned int *r_bound = nullptr;
  const float *src = nullptr;      // dst = src as in launch_pad_copy
  float *dst = nullptr;
  int64_t lds = 0, ldd = 0, rows = 0;
  int32_t cols = 0, dpad = 0;
  unsigned long long *fill = nullptr;
  int64_t nfill = 0;
};
hipError_t launch_opening(const OpeningJobs &j, hipStream_t st);
hipError_t launch_pad_copy(const float *src, int64_t lds, int64_t n, int32_t d, float *dst, int64_t ldd, int32_t dpad,
                           int32_t transpose, hipStream_t st);

// ---------------------------------------------------------------- rotation matrix
// Haar-distributed orthogonal d x d matrix (fp32) from (d, seed); workspaces in doubles:
// Qwork d*d + 2, Cwork rotation_cwork(d), Wwork ceil(d/64)*64*d.
// (coefficients in six parts; the parts of a panel's Gram matrix and their sum take their place)
inline size_t rotation_cwork(int32_t d) {
  return std::max((size_t)6 * 64 * d, ((size_t)(d + 63) / 64 + 1) * 64 * 64);
}
hipError_t launch_make_rotation(int32_t d, uint64_t seed, double *Qwork, double *Cwork, double *Wwork, float *R_out,
                                hipStream_t st);

// ---------------------------------------------------------------- ETR helpers
// Key lists hold (order-preserving distance bits << 32 | index), ascending; ~0 marks an empty slot.
// For each row q of S (nq x m scores q . x_c, row stride lds): merge the K smallest of
// colnorm[col_base + c] - 2 S[q][c] into the running list top[q][0..K).
hipError_t launch_topk_merge(const float *S, int64_t lds, int32_t nq, int32_t m, int64_t col_base,
                             const float *colnorm, int32_t K, unsigned long long *top, hipStream_t st);
// Recall numerator/denominator: per query, the nprobe centroids of smallest ynorm[c] - 2 S[q][c] are
// probed; a ground-truth neighbour counts as found iff its cluster (assign[id]) is probed.
hipError_t launch_recall_scores(const float *S, int64_t lds, int32_t nq, int32_t k, const float *ynorm, int32_t nprobe,
                                const unsigned long long *gt_keys, int32_t K, const int32_t *assign,
                                unsigned long long *hits, unsigned long long *total, hipStream_t st);
// Ground truth through the one-product multiply.  launch_gt_convert: rows [row0, row0 + rows) of the nsel rows spread
// evenly over the n rows of X (nsel = n: the rows themselves) as fp16 rows of ds values in units of a power of two of
// their own: plane, scale, term = ||x||^2 scale / 2, and max ||x||^2 folded into *maxnorm (bit pattern).
hipError_t launch_gt_convert(const float *X, int64_t ldx, int64_t n, int64_t nsel, int64_t row0, int64_t rows, int32_t d,
                             int32_t ds, uint32_t *plane, float *scale, float *term, unsigned int *maxnorm, hipStream_t st);
// tq[i] = K-th smallest of group_min[i][0 .. ngroups) + the error bound of a score of query i
hipError_t launch_gt_threshold(const float *group_min, int32_t ngroups, int32_t nq, int32_t K, const float *q_scale,
                               const float *q_term, const unsigned int *maxnorm, int32_t d, float *tq, hipStream_t st);
// row_term[i] = -(tq[i] + the error bound) q_scale[i] / 2
hipError_t launch_gt_terms(const float *tq, const float *q_scale, const float *q_term, int32_t nq, const unsigned int *maxnorm,
                           int32_t d, float *row_term, hipStream_t st);
// keys[i][0 .. K) = the K nearest of the candidates of query i by their exact distance (direct form); *overflow is set (a
// plain store: page-locked memory will do) if a list is longer than its capacity (a power of two) or shorter than K
hipError_t launch_gt_select(const unsigned long long *cand, const unsigned int *count, unsigned int cap, int32_t nq, int32_t K,
                            const float *X, int64_t ldx, const float *Q, int32_t d, const float *q_scale, const float *q_term,
                            const unsigned int *maxnorm, unsigned long long *keys, unsigned int *overflow, hipStream_t st);
constexpr unsigned int kGtMaxCand = 8192;
constexpr int32_t kGtMaxGroups = 16384;
hipError_t launch_row_norms(const float *X, int64_t ldx, int64_t n, int32_t d, float *out, hipStream_t st);
hipError_t launch_keys_to_index(const unsigned long long *keys, int64_t n, int64_t *idx, hipStream_t st);
hipError_t launch_index_to_keys(const int64_t *idx, int64_t n, unsigned long long *keys, hipStream_t st);
constexpr int kMaxProbe = 8192;

}  // namespace skm
