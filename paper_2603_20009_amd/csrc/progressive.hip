// Progressive-pruning GEMM (Algorithm 1, iterations >= 2; Section 3.4 "Progressive Pruning").
//
// The paper multiplies only the first d' dimensions densely and finishes survivors one by one.
// On MI355X a 64-dimension step of a dense tile (128 x 256, or 128 x 128 where the wider ones would be too few) on the
// matrix cores costs about as much as gathering the same step for 2 % of the tile's pairs, so this kernel keeps multiplying
// a tile densely, 64 dimensions at a time, while more than a small share of its pairs is alive, and
// hands the pairs over to the gather kernel (prune.hip) only once the tile is sparse.  The tests are
// the paper's: after t = d', d'+64, d'+128, ... dimensions a pair is dropped when its partial squared
// distance exceeds theta(t, tau_i); a pair that reaches t = d is offered to the point's packed
// (distance, centroid) minimum if it beats tau_i.
//
// Partial distances come from the norm expansion ||x_t||^2 + ||y_t||^2 - 2 x_t.y_t (Section 3.1).
// The prefix norms at the checkpoints are inputs (xnp, ynp): passes that read every point and every
// centroid anyway write them, and this kernel fetches one number per row and column and checkpoint.
//
// Operands arrive already split into fp16 pairs (the points once per fit, by the first threshold pass; the
// centroids once per step, by the pass over them that starts it), in the very byte order of the LDS tiles, so staging is a
// copy: every lane moves 16 bytes from global memory straight into LDS and the vector unit is left to the tests.
//
// The kernel is persistent: two workgroups per CU take tiles from a per-XCD counter.  When a tile
// ends, the first slab and the per-row data of the next tile are already being fetched while the
// finished tile is written out, so the short tiles of a well-pruned step do not drain the pipeline.
#include "skm_internal.h"

#include <algorithm>
#include <type_traits>

namespace skm {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------- split-fp16 copies of the operands
// Row r of a matrix scaled by split_scale(*absmax): granule g (dims 16 g .. 16 g + 15) is 16 words: 8 words of hi halves
// (fp16 of the scaled value, two per word), then 8 words of lo halves (fp16 of the remainder).  Granule positions 0 and
// ds / 16 + 1 are zero.  Where a granule lies: see skm_internal.h.
__global__ void __launch_bounds__(256) split_rows_kernel(const float *A, int64_t lda, int64_t rows, int32_t ds,
                                                         const unsigned int *absmax, uint32_t *out) {
  const float scale = split_scale(*absmax);
  const int per_row = ds / 4 + 8;   // float4 pieces per output row, pads included
  const int64_t total = rows * per_row;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e / per_row;
    const int piece = (int)(e - r * per_row);      // 4 dims each; pieces 0..3 and the last 4 are padding
    const int gpos = piece >> 2, q = piece & 3;    // granule position, quarter of the granule
    uint2 hi = make_uint2(0u, 0u), lo = hi;
    if (gpos >= 1 && gpos <= ds / 16) {
      const float4 v = *reinterpret_cast<const float4 *>(A + r * lda + 16 * (gpos - 1) + 4 * q);
      const f32x2 p0 = {v.x * scale, v.y * scale}, p1 = {v.z * scale, v.w * scale};
      const f16x2 h0 = __builtin_convertvector(p0, f16x2), h1 = __builtin_convertvector(p1, f16x2);
      const f16x2 l0 = __builtin_convertvector(p0 - __builtin_convertvector(h0, f32x2), f16x2);
      const f16x2 l1 = __builtin_convertvector(p1 - __builtin_convertvector(h1, f32x2), f16x2);
      hi.x = __builtin_bit_cast(unsigned int, h0); hi.y = __builtin_bit_cast(unsigned int, h1);
      lo.x = __builtin_bit_cast(unsigned int, l0); lo.y = __builtin_bit_cast(unsigned int, l1);
    }
    uint32_t *dst = out + split_row(r, split_ld(ds)) + 32 * gpos;
    *reinterpret_cast<uint2 *>(dst + 2 * q) = hi;
    *reinterpret_cast<uint2 *>(dst + 8 + 2 * q) = lo;
  }
}
hipError_t launch_split_rows(const float *A, int64_t lda, int64_t rows, int32_t ds, const unsigned int *absmax,
                             uint32_t *out, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (ds % 16 != 0 || lda % 4 != 0 || (reinterpret_cast<uintptr_t>(A) & 15u) || (reinterpret_cast<uintptr_t>(out) & 15u))
    return hipErrorInvalidValue;
  const int64_t total = rows * (ds / 4 + 8);
  const int64_t blocks = std::min<int64_t>((total + 255) / 256, 1 << 16);
  hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st, A, lda, rows, ds, absmax, out);
  return hipGetLastError();
}

namespace {
constexpr int BM = 128;                             // rows of a workgroup's tile; its columns: 128 NB, NB = 1 or 2
constexpr int TM = 4;                               // 4 wavefronts side by side, each 128 rows x NB blocks of 32 columns
constexpr int NT = 256;
constexpr int ROW_WORDS = 16;                       // a tile row of a unit: 64 bytes (16 hi + 16 lo halves, or 32 hi halves)
template <int NB> constexpr int kStageWords = (BM + 128 * NB) * ROW_WORDS;   // one unit of both operands: 16 or 24 KB
constexpr int NSTAGE = 3;                           // the unit being multiplied and two in flight
constexpr int ROWS_PASS = NT / 4;                   // 4 lanes move one tile row: 64 rows per load instruction
constexpr int A_LD = BM / ROWS_PASS;                // 2 load instructions per thread, unit and operand

// wait until at most n of this wavefront's vector memory operations are outstanding (LDS and export counters untouched)
#define SKM_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))
// barrier behind this wavefront's LDS traffic only: loads in flight stay in flight
#define SKM_BARRIER()                                             \
  do {                                                            \
    asm volatile("" : : : "memory");                              \
    __builtin_amdgcn_s_waitcnt(0xC07F); /* lgkmcnt(0) */          \
    __builtin_amdgcn_s_barrier();                                 \
    asm volatile("" : : : "memory");                              \
  } while (0)

// Sum over the 64 lanes of a wavefront through the data-parallel lane moves: within quads, mirrored
// within half rows and rows, then the row totals handed on to the following rows; lane 63 ends with the result.
#define SKM_WAVE_REDUCE(v, OP)                                                                \
  do {                                                                                        \
    v = v OP __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);  /* quad_perm [1,0,3,2] */ \
    v = v OP __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);  /* quad_perm [2,3,0,1] */ \
    v = v OP __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false); /* row_half_mirror */      \
    v = v OP __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false); /* row_mirror */           \
    v = v OP __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false); /* row_bcast:15 */         \
    v = v OP __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false); /* row_bcast:31 */         \
  } while (0)
__device__ inline int wave_sum_i32(int v) {
  SKM_WAVE_REDUCE(v, +);
  return __builtin_amdgcn_readlane(v, 63);
}

template <int NB> using acc_t = f32x16[TM][NB];

// One unit of 16 dimensions, hi and lo halves: x.y ~ hi.hi' + lo.hi' + hi.lo'.  p0 / p1: word offsets of this lane's
// first and second 16-byte piece inside a tile row.
// Units come in pairs that end on a checkpoint, and the second of a pair adds its largest product last.  The order is
// part of the results: a split leaves two centroids at y (1 +- 1/1024), and which of them a point between them goes to is
// decided by the last bits of the sum.  (1000 fits of 20 000 x 128 points into 100 clusters, 801 of which split one: with the
// first unit's order in both, and the centroids' norms added pairwise, 18 ended with other labels, 12 of them with centroids
// 3e-3 to 3e-2 away.  The uniform branch costs nothing that can be measured: 1M x 1536, k = 4096 240.6 -> 240.9 ms a fit.)
template <int NB>
__device__ inline void unit_three(acc_t<NB> &acc, const uint32_t *Ab, const uint32_t *Bb, int p0, int p1, bool second) {
  f16x8 ah[TM], al[TM], bh[NB], bl[NB];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int b = 0; b < NB; ++b) bh[b] = *reinterpret_cast<const f16x8 *>(Bb + b * 128 * ROW_WORDS + p0);
#pragma unroll
  for (int a = 0; a < TM; ++a) ah[a] = *reinterpret_cast<const f16x8 *>(Ab + a * 32 * ROW_WORDS + p0);
#pragma unroll
  for (int a = 0; a < TM; ++a) al[a] = *reinterpret_cast<const f16x8 *>(Ab + a * 32 * ROW_WORDS + p1);
#pragma unroll
  for (int b = 0; b < NB; ++b) bl[b] = *reinterpret_cast<const f16x8 *>(Bb + b * 128 * ROW_WORDS + p1);
  __builtin_amdgcn_sched_barrier(0);
  auto product = [&](const f16x8 (&x)[TM], const f16x8 (&y)[NB]) {
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[a], y[b], acc[a][b], 0, 0, 0);
  };
  if (!second) product(ah, bh);
  product(al, bh);
  product(ah, bl);
  if (second) product(ah, bh);
  __builtin_amdgcn_sched_barrier(0);
}

// One unit of 32 dimensions, hi halves only.
template <int NB>
__device__ inline void unit_one(acc_t<NB> &acc, const uint32_t *Ab, const uint32_t *Bb, int p0, int p1) {
  f16x8 x[TM], y[NB], x1[TM], y1[NB];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int b = 0; b < NB; ++b) y[b] = *reinterpret_cast<const f16x8 *>(Bb + b * 128 * ROW_WORDS + p0);
#pragma unroll
  for (int a = 0; a < TM; ++a) x[a] = *reinterpret_cast<const f16x8 *>(Ab + a * 32 * ROW_WORDS + p0);
#pragma unroll
  for (int b = 0; b < NB; ++b) y1[b] = *reinterpret_cast<const f16x8 *>(Bb + b * 128 * ROW_WORDS + p1);
#pragma unroll
  for (int a = 0; a < TM; ++a) x1[a] = *reinterpret_cast<const f16x8 *>(Ab + a * 32 * ROW_WORDS + p1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[a], y[b], acc[a][b], 0, 0, 0);
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1[a], y1[b], acc[a][b], 0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
}

}  // namespace

// A workgroup of 4 wavefronts owns 128 points x 128 NB centroids, two workgroups share a CU: while one tests, the other
// multiplies.  A wavefront w owns all 128 rows of the column blocks w and w + 4 (blocks of 32).
//
// The tile advances in units of 64 bytes per tile row: 16 dimensions of both halves, multiplied three ways, or - behind
// the first test of a listed tile, see below - 32 dimensions of the hi halves, multiplied once.  Units are requested two
// ahead, global memory -> LDS directly, 16 bytes per lane, four lanes per row; piece c of row r is kept at position
// c ^ ((r >> 2) & 3), so that the 16-byte fragment reads of 16 consecutive rows fall into 16 different bank groups.
// One barrier per unit.
//
// Listed tiles (g.deep): the first test is exact (three products over d' dimensions: the survivors of the first test are
// counted there).  What follows only has to find the few pairs that can reach the end: one product per dimension
// (a third of the matrix work), and the tests widened by its error bound (screen.hip) over the dimensions behind d'.  A
// pair that passes the exact tests passes the widened ones.  Once few pairs are left, or at the last test, they go to
// the gather kernel, which starts them from dimension 0 again and applies the exact tests (p < 0 marks them): labels,
// distances and counts are those of the exact tests.  A tile most of whose pairs survive the first test, or that ends
// with more pairs than it may hand over, is done in three products throughout.
template <bool LISTED, int NB>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) progressive_kernel(ProgArgs g) {
  constexpr int BN = 128 * NB, TN = NB, STAGE_WORDS = kStageWords<NB>;
  constexpr int B_LD = BN / ROWS_PASS;               // load instructions per thread and unit of the columns' rows
  static_assert(!LISTED || BN == kListCols, "a tile of listed columns");
  extern __shared__ __align__(16) uint32_t smem[];   // [NSTAGE][A: BM rows | B: BN rows][ROW_WORDS]
  // (two copies of the thresholds by tile parity: the previous tile may still be handing pairs over while the next is
  // committed)
  __shared__ __align__(16) float s_tau[2][BM], s_thr[BM], s_xn[BM], s_yn[BN];
  __shared__ int s_ids[LISTED ? 2 : 1][LISTED ? BN : 1];   // by tile parity: the listed centroid ids (-1 = none)
  __shared__ int s_prev[BM];                         // incumbents of the tile being loaded (listed tiles: position in the list)
  __shared__ __align__(16) int s_inc[BM];            // column of every row's incumbent in the tile in work (-1 = another tile's)
  __shared__ int s_any[2];                           // whether there are any, rows 0 .. 63 and 64 .. 127
  __shared__ __align__(16) unsigned int s_wcnt[2][4];   // alive pairs of every wavefront at the last checkpoint (by checkpoint parity)
  __shared__ unsigned int s_base;         // first list slot of a tile that hands its pairs over
  __shared__ int s_q[4];   // ring of tile numbers drawn from the XCD's counter, two tiles ahead of the one in work
  put_stamp(g.stamp);

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, kh = lane >> 5;
  const int swz = (r32 >> 2) & 3;
  const int p0 = (kh ^ swz) << 2, p1 = ((2 + kh) ^ swz) << 2;   // this lane's two pieces of a tile row
  const int nrt = (g.M + BM - 1) / BM, nct = (g.N + BN - 1) / BN;
  // Listed columns (after the low-precision first filter): tile t is row tile tile_rt[t] against the 256 centroids
  // col_list[256 t ..]; the "column tile" of such a tile is its own number.
  const int ntiles = LISTED ? *g.ntiles : nrt * nct;
  // column tiles per panel of the tile walk: in the steady state only d' + a few blocks of every centroid are read,
  // so a panel of 2048 centroids fits one XCD's L2 and every point tile is read once per panel
  constexpr int PC = 2048 / BN;

  // This workgroup's share: the tiles of its XCD (workgroups are dealt round-robin to the 8 XCDs), walked through a per-XCD
  // counter.  Consecutive tiles share rows or columns, so an XCD takes them in runs, long enough that the 64 workgroups at
  // work in it are in one or two runs; and the runs are dealt out in turn, because the tiles of a step are not alike: where the
  // points follow their thresholds the last ones hold most of the pairs that live on.  One contiguous eighth for each XCD, one
  // of them worked (and its part of the hand-over list was gathered) long after the others were done: assignment of 2.5M x 384
  // to 32 768 centroids 39.4 -> 34.9 ms, the gather kernel in it 4.30 -> 1.22.  Runs of 32, 64, 128 and 256 tiles are alike
  // (35.1, 35.5, 34.9, 35.2).  So that there are 16 rounds (from 1024 tiles on), fewer than 16 384 tiles go in shorter ones, 64 tiles from 8192 on,
  // 32 from 4096, 16 from 2048 and 8 below (the last two not measured against others).  What does not fill a round is split evenly.
  const int xcd = blockIdx.x & 7;
  const int run = min(max(31 - __builtin_clz(max(ntiles, 1)) - 7, 3), 7);   // log2 of the tiles in a run
  const int rounds = ntiles >> (run + 3), rest = ntiles - (rounds << (run + 3));
  const int in_rounds = rounds << run;   // tiles of this XCD in whole rounds
  const int tbase = rest >> 3, trem = rest & 7;
  const int xstart = (rounds << (run + 3)) + xcd * tbase + (xcd < trem ? xcd : trem) - in_rounds;
  const int xcount = in_rounds + tbase + (xcd < trem ? 1 : 0);
  unsigned int *ctr = g.tile_counter + xcd * kSubListStride;
  const int panel_sz = PC * nrt;
  auto tile_rc = [&](int q, int &rt, int &ct) {   // q-th tile of this XCD -> (row tile, column tile)
    const int logical = q < in_rounds ? (((q >> run) << 3 | xcd) << run) + (q & ((1 << run) - 1)) : xstart + q;
    if (LISTED) {   // (the list tells the row tile; ct is the tile's place in the list)
      ct = logical;
      return;
    }
    const int p = logical / panel_sz, r = logical - p * panel_sz;   // (uniform)
    const int pc = (nct - p * PC) < PC ? (nct - p * PC) : PC;
    rt = r / pc;
    ct = p * PC + (r - rt * pc);
  };

  unsigned long long *sc = g.scal + (size_t)(blockIdx.x & (kStatReplicas - 1)) * SC_COUNT;

  // Staging: load instruction j of wavefront w moves tile rows 64 j + 16 w .. + 15 of a unit.
  const int ld_row = 16 * wave + (lane >> 2);                       // + 64 j
  const unsigned int ld_piece = 16u * ((lane & 3) ^ ((ld_row >> 2) & 3));   // byte offset of the piece that belongs at this lane's position
  const int ldh = (int)(g.lda >> 1);

  // ---- the tile being loaded.  Rows past the end repeat the last one (their accumulator elements start dead).
  // byte offsets of this lane's pieces from the tile's first row / the first row of the tile's columns
  unsigned int offA[A_LD], offB[B_LD];
  const uint32_t *baseA = g.A, *baseAh = g.Ah, *baseB = g.B;   // first rows (uniform)
  int nrow = 0, ncol = 0;                   // row tid & 127 and column tid, for their prefix norms
  float nxreg = 0.f, nyreg = 0.f, rreg = 0.f;
  float2 wreg = make_float2(0.f, 0.f);
  int2 where = make_int2(0, 0);   // row tile of the next listed tile, and the number of its list's columns before it
  // What the next tile needs is brought to LDS a tile ahead: the list's ids (a missing one loads centroid 0 and starts
  // dead), the rows' thresholds and incumbents.
  auto fetch_ids = [&](int ct, int par) {
    if constexpr (LISTED) {
      const auto *w = reinterpret_cast<const __attribute__((address_space(4))) int *>(reinterpret_cast<uint64_t>(g.tile_rt + ct));
      where = make_int2(w[0], w[1]);   // (scalar loads: written by an earlier kernel)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(uniform_buffer(g.col_list + (int64_t)ct * BN), (lds_words_t)s_ids[par] + 64 * wave, 4,
                                               tid * 4, 0, 0, 0);
    }
  };
  auto fetch_rows = [&](int rt, int par) {
    if (LISTED) rt = where.x;
    const int64_t at = g.row_base + (int64_t)rt * BM;
    if (wave < BM / 64) {
      const int off = 4 * min(tid, g.M - 1 - rt * BM);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(uniform_buffer(g.tau + at), (lds_words_t)s_tau[par] + 64 * wave, 4, off, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(uniform_buffer(g.prev + at), (lds_words_t)s_prev + 64 * wave, 4, off, 0, 0, 0);
    }
  };
  int first_col = 0;   // of the aimed tile: its first column, or for a listed tile its first position in the row tile's list
  auto aim = [&](int &rt, int ct, int par) {
    first_col = ct * BN;
    if (LISTED) {
      rt = where.x;
      first_col = where.y;
    }
    const int row0 = rt * BM;
    baseA = g.A + (int64_t)row0 * g.lda;
    if (LISTED && g.deep) baseAh = g.Ah + (int64_t)row0 * ldh;
    const int limA = g.M - 1 - row0;
#pragma unroll
    for (int j = 0; j < A_LD; ++j) offA[j] = (unsigned int)split_row(min(ld_row + ROWS_PASS * j, limA), (int)g.lda) * 4u + ld_piece;
    nrow = row0 + min(tid & (BM - 1), limA);
    if constexpr (LISTED) {
#pragma unroll
      for (int j = 0; j < B_LD; ++j) offB[j] = (unsigned int)split_row(max(s_ids[par][ld_row + ROWS_PASS * j], 0), (int)g.ldb) * 4u + ld_piece;   // (the launcher checks the range)
      ncol = max(s_ids[par][tid], 0);
    } else {
      const int col0 = ct * BN, limB = g.N - 1 - col0;
      baseB = g.B + (int64_t)col0 * g.ldb;
#pragma unroll
      for (int j = 0; j < B_LD; ++j) offB[j] = (unsigned int)split_row(min(ld_row + ROWS_PASS * j, limB), (int)g.ldb) * 4u + ld_piece;
      ncol = col0 + min(tid, limB);
    }
  };
  // ---- requests: the next unit of the aimed tile -> LDS (asynchronous).  Buffer loads: a uniform base, a uniform offset
  // that moves on by 128 bytes a unit (a unit of two rows), and an offset register per load.  (They are known to be no LDS reads: behind
  // global_load_lds the compiler lets the first matrix instruction of a unit wait for all of its fragments.)  Row pairs of
  // the points' hi plane are half as long as those of the three-product copy: the offsets (128 bytes a granule of two rows,
  // 64 bytes a row) are halved once where a tile changes over.  Where d' is an odd multiple of 16 the plane's units and those
  // of this tile are half a unit apart: a piece comes from the second half of one or the first half of the next.
  int cur = 0;            // word offset of the LDS stage of the unit being multiplied
  int rstage = 0;         // ... of the next request
  int treq = 0, rstep = 16;   // dimensions requested so far of the tile, and those of the next request
  int soff = 0;           // byte offset of the next unit in a row
  const uint32_t *fromA = g.A, *fromB = g.B;
  auto ring = [&](int stage) { return stage == (NSTAGE - 1) * STAGE_WORDS ? 0 : stage + STAGE_WORDS; };
  auto request = [&]() {
    lds_words_t sb = (lds_words_t)smem + rstage + 16 * wave * ROW_WORDS;
    const __amdgpu_buffer_rsrc_t ra = uniform_buffer(fromA), rb = uniform_buffer(fromB);
#pragma unroll
    for (int j = 0; j < A_LD; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, sb + ROWS_PASS * j * ROW_WORDS, 16, (int)offA[j], soff, 0, 0);
#pragma unroll
    for (int j = 0; j < B_LD; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, sb + (BM + ROWS_PASS * j) * ROW_WORDS, 16, (int)offB[j], soff, 0, 0);
    soff += 128;
    treq += rstep;
    rstage = ring(rstage);
  };
  const unsigned int ld_odd = !LISTED || (g.dprime & 16) == 0 ? 0u : ld_piece < 32u ? 32u : 96u;
  auto change_over = [&]() {   // to one product, at dimension d'
    fromA = baseAh;
    fromB = g.Bh;
    soff = 128 * (g.dprime / 32);
#pragma unroll
    for (int j = 0; j < A_LD; ++j) offA[j] = ((offA[j] & ~127u) >> 1) + (offA[j] & 127u) + ld_odd;
    rstep = 32;
  };
  // Checkpoint m's prefix norms (the points' table has a row per 16 dimensions, the centroids' a row per checkpoint of
  // this step), theta ratio and, for the widened tests, the largest centroid norms.
  auto load_norm = [&](int m) {
    m = min(m, g.nb);
    const int px = (min(g.dprime + kBlockDims * m, g.ds) >> 4) - 1;
    nxreg = (g.xnp + ((int64_t)px * g.xn_stride + g.row_base))[nrow];
    nyreg = (g.ynp + (int64_t)m * g.N)[ncol];
    rreg = g.ratio[m];
    if (LISTED && g.deep) wreg = g.widen[m];
  };
  const unsigned int amax = *g.a_absmax, bmax = *g.b_absmax;
  const float m2 = -2.f * split_unscale(amax) * split_unscale(bmax);   // accumulator -> -2 x.y
  auto row_of = [&](int a, int v) { return a * 32 + 8 * (v >> 2) + 4 * kh + (v & 3); };

  // first tile of this workgroup
  __syncthreads();
  if (tid == 0) {
    s_q[0] = (int)atomicAdd(ctr, 1u);
    s_q[1] = (int)atomicAdd(ctr, 1u);
  }
  __syncthreads();
  int q = __builtin_amdgcn_readfirstlane(s_q[0]);
  if (q >= xcount) return;
  int rt = 0, ct = 0;
  tile_rc(q, rt, ct);
  rt = __builtin_amdgcn_readfirstlane(rt);
  ct = __builtin_amdgcn_readfirstlane(ct);
  bool redone = false;   // (listed) the tile is being done again, in three products
  auto start_tile = [&]() {   // first two units of the aimed tile
    load_norm(0);
    fromA = baseA;
    fromB = baseB;
    soff = 128;   // (a granule of zeros leads every row)
    treq = 0;
    rstep = 16;
    rstage = cur;
    request();
    if (treq < g.ds) {
      if (LISTED && g.deep && !redone && treq == g.dprime) change_over();
      request();
    }
  };
  if (LISTED) fetch_ids(ct, 0);
  fetch_rows(rt, 0);
  SKM_VMCNT(0);
  SKM_BARRIER();
  aim(rt, ct, 0);   // (sets rt of a listed tile)
  start_tile();
  // A tile is committed: the incumbents' columns are noted, and the number of the tile after next is drawn (the counter's
  // answer is stored at the end of the tile, so its round trip never stalls the workgroup).
  unsigned int drawn = 0;
  auto commit = [&]() {
    if (wave < BM / 64) {
      const int prev = s_prev[tid], cl = prev - first_col;
      const bool here = prev >= 0 && cl >= 0 && cl < BN;
      s_inc[tid] = here ? cl : -1;
      const bool any = __ballot(here) != 0;
      if (lane == 0) s_any[wave] = any;
    }
    if (tid == 0) drawn = atomicAdd(ctr, 1u);
    SKM_BARRIER();
  };
  commit();

  for (int tile_no = 0;; ++tile_no) {
    const int row0 = rt * BM, col0 = ct * BN;
    const int par = tile_no & 1;
    // the tile after this one: its number is known already, its list of columns is fetched while this one is multiplied
    q = __builtin_amdgcn_readfirstlane(s_q[(tile_no + 1) & 3]);
    const bool more = q < xcount;
    int rt_next = 0, ct_next = 0;
    if (more) {
      tile_rc(q, rt_next, ct_next);
      rt_next = __builtin_amdgcn_readfirstlane(rt_next);
      ct_next = __builtin_amdgcn_readfirstlane(ct_next);
    }
    acc_t<NB> acc;
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    int gc[TN];   // centroid of this lane's accumulator columns (listed tiles: -1 = none)
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      if constexpr (LISTED) gc[b] = s_ids[par][(b * 4 + wave) * 32 + r32];
      else gc[b] = col0 + (b * 4 + wave) * 32 + r32;
    }
    auto is_col = [&](int b) { return (unsigned int)gc[b] < (unsigned int)g.N; };
    if (LISTED && more) fetch_ids(ct_next, par ^ 1);
    if (!LISTED && more) fetch_rows(rt_next, par ^ 1);
    // one alive-bit per accumulator element: word a, bit 16 b + v
    unsigned int bits[TM];
    {
#pragma unroll
      for (int a = 0; a < TM; ++a) bits[a] = NB > 1 ? 0xffffffffu : 0xffffu;
      if (s_any[0] | s_any[1]) {   // incumbents start dead
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int v4 = 0; v4 < 4; ++v4) {
            const int4 c = *reinterpret_cast<const int4 *>(&s_inc[a * 32 + 8 * v4 + 4 * kh]);
            const int cl[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
              for (int b = 0; b < TN; ++b)
                if (cl[u] == (b * 4 + wave) * 32 + r32) bits[a] &= ~(1u << (16 * b + 4 * v4 + u));
          }
      }
      if (row0 + BM > g.M) {   // rows past the end start dead
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (row0 + row_of(a, v) >= g.M) bits[a] &= ~(0x10001u << v);
      }
    }

    int fin_mode = 0, fin_m = 0;   // how the tile ends: 0 = nothing alive, 1 = reached t = d, 2 = handed over at fin_m
    int wave_alive = 0;            // alive pairs of this wavefront at the last checkpoint
    unsigned int slot0 = 0;        // thread 0: reply of the list reservation
    float yn[TN] = {};
    float xn0 = 0.f;               // this thread's row: its norm over the first d' dimensions
    const bool deep = LISTED && __builtin_amdgcn_readfirstlane(g.deep && !redone);
    int t = 0;                     // dimensions multiplied
    int m = 0;                     // next checkpoint, at dimension tcp
    int tcp = g.dprime;
    int ncp = 0;                   // exchanges so far (row of s_wcnt)
    // in one product a test every deep_stride blocks will do, the last one is the last test there is
    auto after = [&](int mm) { return LISTED && deep ? min(mm + g.deep_stride, g.nb - 1) : mm + 1; };
    const int tend = LISTED && deep ? g.dprime + kBlockDims * (g.nb - 1) : g.ds;   // dimensions that may be needed
    unsigned int dims3 = 0, dims1 = 0;
    // Units until the tile ends (0), goes on in one product (1) or has to be done again in three (2); kind: one product
    // or three, a constant.  (Two loops rather than one with both kinds of unit: the accumulators of a loop with two
    // multiply blocks do not stay in place.)
    auto advance = [&](auto kind) -> int {
    constexpr bool one = decltype(kind)::value;
    constexpr int step = one ? 32 : 16;
    while (true) {
      cur = __builtin_amdgcn_readfirstlane(cur);   // (uniform: kept in scalar registers)
      treq = __builtin_amdgcn_readfirstlane(treq);
      rstage = __builtin_amdgcn_readfirstlane(rstage);
      rstep = __builtin_amdgcn_readfirstlane(rstep);
      soff = __builtin_amdgcn_readfirstlane(soff);
      t = __builtin_amdgcn_readfirstlane(t);
      m = __builtin_amdgcn_readfirstlane(m);
      tcp = __builtin_amdgcn_readfirstlane(tcp);
      // the unit has arrived once at most the unit requested after it is outstanding (loads are counted in order)
      if (treq > t + step) SKM_VMCNT(A_LD + B_LD);
      else SKM_VMCNT(0);
      const bool cp = t + step >= tcp, last = !one && t + step >= g.ds;
      if (cp) {
        // the prefix norms fetched one checkpoint ago -> LDS, with the row's threshold theta(t_m, tau) - ||x_t||^2
        if (tid < BM) {
          const float tau = s_tau[par][tid];
          float thr = rreg * tau - nxreg;
          if (one)   // + the error bound of the one product over the dimensions behind d', and guards
            thr += fmaf(wreg.x, sqrtf(fmaxf(nxreg - xn0, 0.f) + 1e-6f * nxreg), fmaf(1e-6f, rreg * tau + nxreg, wreg.y));
          s_xn[tid] = nxreg;
          s_thr[tid] = thr;
          if (LISTED && m == 0) xn0 = nxreg;
        }
        if (NB > 1 || tid < BN) s_yn[tid] = nyreg;
      }
      SKM_BARRIER();   // everyone's share of the unit is there, and the stage before it is free
      if (cp) load_norm(after(m));
      if (treq < tend) {
        if (LISTED && !one && deep && treq == g.dprime) change_over();
        request();
      }
      {
        const uint32_t *Ab = smem + cur + r32 * ROW_WORDS;
        const uint32_t *Bb = smem + cur + (BM + wave * 32 + r32) * ROW_WORDS;
        if constexpr (one) unit_one<NB>(acc, Ab, Bb, p0, p1);
        else unit_three<NB>(acc, Ab, Bb, p0, p1, ((t ^ g.dprime) & 16) != 0);
      }
      cur = ring(cur);
      t += step;
      if (one) dims1 += step;
      else dims3 += step;
      if (!cp) continue;

#pragma unroll
      for (int b = 0; b < TN; ++b) yn[b] = s_yn[(b * 4 + wave) * 32 + r32];
      if (LISTED && !one && m == 0 && more) fetch_rows(0, par ^ 1);
      auto row_thresholds = [&](int a, float (&thr)[16]) {
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
          const float4 f = *reinterpret_cast<const float4 *>(&s_thr[a * 32 + 8 * v4 + 4 * kh]);
          thr[4 * v4] = f.x; thr[4 * v4 + 1] = f.y; thr[4 * v4 + 2] = f.z; thr[4 * v4 + 3] = f.w;
        }
      };
      // the four wavefronts' numbers added up (the next exchange goes through the other row: a wavefront that is already
      // there cannot disturb this read)
      auto tile_sum = [&](int mine) {
        if (lane == 0) s_wcnt[ncp & 1][wave] = (unsigned int)mine;
        SKM_BARRIER();
        const uint4 wc = *reinterpret_cast<const uint4 *>(s_wcnt[ncp & 1]);
        ++ncp;
        return (unsigned int)__builtin_amdgcn_readfirstlane(wc.x + wc.y + wc.z + wc.w);
      };
      // Test theta(t_m, tau_i): drop the pair when its partial distance exceeds it.
      if constexpr (one) {
        // Is anything left?  Per lane and column the smallest distance minus threshold over its 64 rows, a fused
        // multiply and half a minimum per element; the pairs themselves are told apart only once few columns are left
        // (pairs that died at the first test may count here: a column too many then)
        int cols = 0;
        float least[TM][TN];
#pragma unroll
        for (int a = 0; a < TM; ++a) {
          float thr[16];
          row_thresholds(a, thr);
#pragma unroll
          for (int b = 0; b < TN; ++b) {
            least[a][b] = fminf(fmaf(m2, acc[a][b][0], -thr[0]), fmaf(m2, acc[a][b][1], -thr[1]));
#pragma unroll
            for (int v = 2; v < 16; v += 2)
              least[a][b] = fminf(fminf(least[a][b], fmaf(m2, acc[a][b][v], -thr[v])), fmaf(m2, acc[a][b][v + 1], -thr[v + 1]));
          }
        }
#pragma unroll
        for (int b = 0; b < TN; ++b)
          cols += __popcll(__ballot(fminf(fminf(least[0][b], least[1][b]), fminf(least[2][b], least[3][b])) <= -yn[b] && is_col(b)));
        const unsigned int left = tile_sum(cols);
        if (left == 0u) return 0;
        const bool stop = m >= g.nb - 1;   // (the last test there is)
        if (!stop && left > g.emit_deep) {
          m = after(m);
          tcp = min(g.dprime + kBlockDims * m, g.ds);
          continue;
        }
#pragma unroll
        for (int a = 0; a < TM; ++a) {
          float thr[16];
          row_thresholds(a, thr);
          unsigned int kept = 0u;
#pragma unroll
          for (int b = TN - 1; b >= 0; --b) {
            kept <<= 16;
            if (__ballot(least[a][b] <= -yn[b])) {   // (few blocks of 32 x 32 have any)
              unsigned int dropped = 0u;
#pragma unroll
              for (int v = 15; v >= 0; --v) {
                const float margin = thr[v] - fmaf(m2, acc[a][b][v], yn[b]);
                dropped = __builtin_amdgcn_alignbit(dropped, __builtin_bit_cast(unsigned int, margin), 31);
              }
              kept |= ~dropped & 0xffffu;
            }
          }
          bits[a] &= kept;
        }
        wave_alive = wave_sum_i32(__popc(bits[0]) + __popc(bits[1]) + __popc(bits[2]) + __popc(bits[3]));
      } else {
        // The sign of threshold minus distance is the verdict (a difference of two floats is negative exactly when the
        // second is larger); the signs of the 32 elements of an accumulator row block are shifted into one word, last
        // element first, one funnel shift each.
        if (m == 0) {   // columns past the end
          const unsigned int cols = (is_col(0) ? 0xffffu : 0u) | (NB > 1 && is_col(NB - 1) ? 0xffff0000u : 0u);
#pragma unroll
          for (int a = 0; a < TM; ++a) bits[a] &= cols;
        }
        if (!last || g.nb == 0) {
#pragma unroll
          for (int a = 0; a < TM; ++a) {
            unsigned int dropped = 0u;
            float thr[16];
            row_thresholds(a, thr);
#pragma unroll
            for (int b = TN - 1; b >= 0; --b)
#pragma unroll
              for (int v = 15; v >= 0; --v) {
                const float margin = thr[v] - fmaf(m2, acc[a][b][v], yn[b]);
                dropped = __builtin_amdgcn_alignbit(dropped, __builtin_bit_cast(unsigned int, margin), 31);
              }
            bits[a] &= ~dropped;
          }
          static_assert(TN * 16 <= 32, "one word per accumulator row block");
        }
        wave_alive = wave_sum_i32(__popc(bits[0]) + __popc(bits[1]) + __popc(bits[2]) + __popc(bits[3]));
      }
      const unsigned int total = tile_sum(wave_alive);
      // a tile that is sparse hands over; in one product, whose pairs start again at dimension 0, once few columns are left
      const bool redo = LISTED && deep && (one ? m >= g.nb - 1 && total > g.emit_max : m == 0 && total > g.deep_max);
      const bool hand = total != 0u && !last && !redo && total <= (LISTED && !one && deep ? g.emit_first : g.emit_max);
      if (tid == 0) {
        // a tile that hands its pairs over reserves their slots now (one reservation per tile in the sub-list of
        // this workgroup's XCD): the answer is not needed before the next tile's loads have been requested
        if (hand) slot0 = atomicAdd(g.pair_count + xcd * kSubListStride, total);
        if (total) {
          if (m == 0 && !redone) atomicAdd(sc + SC_SURVIVORS, (unsigned long long)total);
          if (!last && g.block_stats) atomicAdd(sc + SC_ENTER + m, (unsigned long long)total);
          if (last) atomicAdd(sc + SC_COMPLETED, (unsigned long long)total);
          if (!last && !hand && !redo) atomicAdd(sc + SC_DENSE_PB, (unsigned long long)total);   // the next block of these pairs is done densely
        }
      }
      if (total == 0u) return 0;
      if (hand) {
        fin_mode = 2;
        fin_m = m;
        return 0;
      }
      if (redo) return 2;
      if (last) {
        fin_mode = 1;
        fin_m = m;
        return 0;
      }
      m = after(m);
      tcp = min(g.dprime + kBlockDims * m, g.ds);
      if (LISTED && !one && deep) return 1;   // behind the first test
    }
    };
    int act = advance(std::false_type());
    if constexpr (LISTED) {
      if (act == 1) act = advance(std::true_type());
    }
    const bool wide = NB > 1 && __ballot(is_col(NB - 1)) != 0;   // (wavefront 0: more than 128 columns)
    if (tid == 0) {   // (in tiles of 128 x 128)
      atomicAdd(sc + SC_DENSE_DIMS, (unsigned long long)dims3 << (wide ? 1 : 0));
      if (LISTED && dims1) atomicAdd(sc + SC_SCREEN_DIMS, (unsigned long long)dims1 << (wide ? 1 : 0));
    }

    // ---- start fetching the next tile before this one is written out (what was requested ahead of this tile's end has
    // to land first: the stages are reused; stage cur - 1, the last one read, stays free for the hand-over below)
    SKM_VMCNT(0);
    if (LISTED && act == 2) {
      // the tile once more, in three products throughout
      redone = true;
      if (rstep == 32) {
#pragma unroll
        for (int j = 0; j < A_LD; ++j) offA[j] = (((offA[j] - ld_odd) & ~127u) << 1) + ((offA[j] - ld_odd) & 127u);
      }
      start_tile();
      --tile_no;
      continue;
    }
    redone = false;   // (of the finished tile: the next one's first requests already ask for it)
    if (more) {
      if (LISTED) SKM_BARRIER();   // (the ids were brought by all wavefronts)
      aim(rt_next, ct_next, par ^ 1);
      start_tile();
    }

    if (!LISTED && fin_mode == 1) {
      // finished distances: offer those below tau_i to the point's packed minimum
#pragma unroll
      for (int h = 0; h < TM; h += 2) {
        const unsigned long long key = reduce_rows32(
            [&](int a, int v) {
              unsigned long long k = ~0ull;
              const int rl = row_of(h + a, v);
              const float xr = s_xn[rl], tr = s_tau[par][rl];
#pragma unroll
              for (int b = 0; b < TN; ++b)
                if ((bits[h + a] >> (b * 16 + v)) & 1u) {
                  float dist = xr + fmaf(m2, acc[h + a][b][v], yn[b]);
                  dist = dist > 0.f ? dist : 0.f;
                  if (dist < tr) {
                    const unsigned long long kb = pack_key(dist, gc[b]);
                    k = kb < k ? kb : k;
                  }
                }
              return k;
            },
            lane);
        const int rl = row_of(h + (r32 >> 4), r32 & 15);
        if (key != ~0ull) atomicMin(g.best + g.row_base + row0 + rl, key);   // (rows past the end are dead: ~0)
      }
    } else if (fin_mode != 0) {
      // sparse enough: hand the alive pairs to the gather kernel, which resumes at block fin_m (or starts over).
      // A listed tile that is finished here walks its distances on the same way and keeps the least of a row in LDS (behind what
      // the lanes park; only the whole-stage tiles of 256 columns have that room), so that a row is offered once: one by one to
      // the points' minima, tiles of poor incumbents waited for each other's atomics (one step without incumbents, 1.3e9 of
      // 3.0e9 pairs finished: 500 000 x 384 on the sphere against 6000 centroids 43.7 -> 15.3 ms, this kernel 40.4 -> 12.6;
      // 1M x 128, normal, k = 4096 67.1 -> 14.5 ms; 2M x 96, a mixture, k = 16 384 124 -> 52 ms).
      static_assert(!LISTED || STAGE_WORDS >= 4 * 16 * 64 + 2 * BM, "room behind the parked values");
      const bool offer = LISTED && fin_mode == 1;
      const int idle = cur == 0 ? (NSTAGE - 1) * STAGE_WORDS : cur - STAGE_WORDS;   // the stage the last unit was read from
      unsigned long long *s_low = reinterpret_cast<unsigned long long *>(smem + idle + 4 * 16 * 64);
      if (offer) {
        if (tid < BM) s_low[tid] = ~0ull;
      } else if (tid == 0) {
        unsigned int base = slot0;
        const unsigned int *w = s_wcnt[(ncp - 1) & 1];
        const unsigned int tot = w[0] + w[1] + w[2] + w[3];
        if ((unsigned long long)base + tot > (unsigned long long)g.sub_capacity) {
          atomicOr(g.overflow, 1u);
          base = 0xffffffffu;
        } else {
          base += xcd * g.sub_capacity;
        }
        s_base = base;
      }
      SKM_BARRIER();
      unsigned int run = offer ? 0u : s_base;
      if (run != 0xffffffffu && wave_alive > 0) {
        for (int w = 0; w < wave; ++w) run += s_wcnt[(ncp - 1) & 1][w];
        // A sparse tile holds one or two alive pairs per lane.  Every lane walks its own alive bits; the accumulator
        // element behind a bit is found through LDS, where the lane parks its 16 values of a block (a register
        // cannot be chosen per lane): the stage the last unit was read from is free, 4 KB per wavefront as [16][64].
        // List slots: the wavefront's range, then lane by lane (prefix sum of the lanes' counts), then bit by bit.
        int upto = __popc(bits[0]) + __popc(bits[1]) + __popc(bits[2]) + __popc(bits[3]);
        const int mine = upto;
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xF, 0xF, false);   // row_shr:1
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xF, 0xF, false);   // row_shr:2
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xF, 0xF, false);   // row_shr:4
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xF, 0xF, false);   // row_shr:8
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x142, 0xA, 0xF, false);   // row_bcast:15
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x143, 0xC, 0xF, false);   // row_bcast:31
        unsigned int pos = run + (unsigned int)(upto - mine);
        const bool over = LISTED && fin_m > 0 && deep;   // the partial sum holds one-product parts: the pair starts over
        float *park = reinterpret_cast<float *>(smem + idle + wave * (16 * 64)) + lane;
        const unsigned int mtag = over ? 0u : (unsigned int)fin_m << 24;
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b) {
            unsigned int left = (bits[a] >> (16 * b)) & 0xffffu;
            if (!__ballot(left)) continue;
            if (!over) {
#pragma unroll
              for (int v = 0; v < 16; ++v) park[v * 64] = acc[a][b][v];
            }
            while (left) {
              const int v = __builtin_ctz(left);
              left &= left - 1u;
              const int rl = a * 32 + 4 * kh + 8 * (v >> 2) + (v & 3);
              float p = -1.f;
              if (!over) {
                p = s_xn[rl] + fmaf(m2, park[v * 64], yn[b]);
                p = p > 0.f ? p : 0.f;
              }
              if (LISTED && offer) {
                if (p < s_tau[par][rl])
                  (void)__hip_atomic_fetch_min(s_low + rl, pack_key(p, gc[b]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                continue;
              }
              Pair pr;
              pr.i = (int32_t)g.row_base + row0 + rl;
              pr.j = (int32_t)((uint32_t)gc[b] | mtag);
              pr.p = p;
              pr.tau = s_tau[par][rl];
              g.pairs[pos++] = pr;
            }
          }
      }
      if (offer) {
        SKM_BARRIER();
        if (tid < BM && s_low[tid] != ~0ull) atomicMin(g.best + g.row_base + row0 + tid, s_low[tid]);
      }
    }

    if (!more) break;
    rt = rt_next;
    ct = ct_next;
    if (tid == 0) s_q[(tile_no + 2) & 3] = (int)drawn;
    commit();   // its barrier also ends this tile: everyone is done with the tile's LDS
  }
}

hipError_t launch_progressive(const ProgArgs &args, hipStream_t st) {
  ProgArgs g = args;
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.ds % 16 != 0 || g.dprime % 16 != 0 || g.dprime < 16 || g.dprime > g.ds || g.lda != split_ld(g.ds) || g.ldb != split_ld(g.ds) ||
      g.nb > kMaxBlocks || (reinterpret_cast<uintptr_t>(g.A) & 15u) || (reinterpret_cast<uintptr_t>(g.B) & 15u) ||
      g.N > (1 << 24))
    return hipErrorInvalidValue;
  // once per process (the initialisation of a function-local static is synchronised between threads): the kernel's LDS
  // size, and two workgroups per CU (LDS and registers allow no more)
  constexpr size_t smem1 = (size_t)NSTAGE * kStageWords<1> * sizeof(uint32_t), smem2 = (size_t)NSTAGE * kStageWords<2> * sizeof(uint32_t);
  struct Setup {
    hipError_t rc;
    int wgs = 0;
    Setup() {
      rc = hipFuncSetAttribute(reinterpret_cast<const void *>(progressive_kernel<false, 1>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem1);
      if (rc == hipSuccess)
        rc = hipFuncSetAttribute(reinterpret_cast<const void *>(progressive_kernel<false, 2>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem2);
      if (rc == hipSuccess)
        rc = hipFuncSetAttribute(reinterpret_cast<const void *>(progressive_kernel<true, 2>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem2);
      int dev = 0, cus = 256;
      (void)hipGetDevice(&dev);
      (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
      wgs = 2 * cus;
    }
  };
  static const Setup setup;
  if (setup.rc != hipSuccess) return setup.rc;
  const int wgs = setup.wgs;
  if (g.col_list && ((int64_t)g.N + 1) * g.ldb >= ((int64_t)1 << 30)) return hipErrorInvalidValue;   // (32-bit byte offsets)
  if ((g.col_list != nullptr) != (g.tile_rt != nullptr) || (g.col_list != nullptr) != (g.ntiles != nullptr))
    return hipErrorInvalidValue;
  if (g.deep && (g.nb < 3 || g.deep_stride < 1 || !g.col_list || !g.Ah || !g.Bh || !g.widen || (reinterpret_cast<uintptr_t>(g.Ah) & 15u) ||
                 (reinterpret_cast<uintptr_t>(g.Bh) & 15u)))
    return hipErrorInvalidValue;
  // Tiles of 128 columns where tiles of 256 would give a CU fewer than eight: what the last round leaves idle then costs
  // more than the narrower tile's extra fragment reads.
  const int64_t nrt = (g.M + BM - 1) / BM;
  const bool narrow = !g.col_list && nrt * ((g.N + 255) / 256) < (int64_t)4 * wgs;
  if (narrow) g.emit_max /= 2;
  const int64_t ntiles = nrt * (narrow ? (g.N + 127) / 128 : (g.N + 255) / 256);
  if (ntiles > 0x7fffffffLL) return hipErrorInvalidValue;
  const int64_t grid = std::max<int64_t>(8, std::min<int64_t>(wgs, (ntiles + 7) / 8 * 8));
  if (g.col_list)
    hipLaunchKernelGGL((progressive_kernel<true, 2>), dim3((unsigned)grid), dim3(NT), smem2, st, g);
  else if (narrow)
    hipLaunchKernelGGL((progressive_kernel<false, 1>), dim3((unsigned)grid), dim3(NT), smem1, st, g);
  else
    hipLaunchKernelGGL((progressive_kernel<false, 2>), dim3((unsigned)grid), dim3(NT), smem2, st, g);
  return hipGetLastError();
}

int64_t progressive_tiles(int64_t rows, int32_t k) { return ((rows + BM - 1) / BM) * (int64_t)((k + 255) / 256); }
int32_t progressive_tile_pairs() { return BM * 256; }

}  // namespace skm
