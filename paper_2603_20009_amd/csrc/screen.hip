// Low-precision first filter (the paper's closing remark of Section 4.14 on GEMM hardware; Algorithm 1's first test
// theta(d', tau) is what it screens for).
//
// The progressive kernel multiplies every (point tile, centroid tile) pair on the first d' dimensions with three fp16
// products per element, although in a well-pruned step all but a few columns of a tile die at the first test.  This
// pass finds those few columns at a third of the price: one fp16 product (the hi halves of the split operands only:
// half the bytes through L2 and LDS, a third of the matrix instructions), and the first test with its threshold
// widened by a bound of the error that the dropped lo halves can cause.  A pair that passes the exact test passes the
// widened one, so a column that no point of a row tile passes here is dead for that whole tile.  The output is one bit
// per (row tile, centroid); compaction turns the bits into a list of centroid ids per row tile, cut into tiles of 256
// listed columns, and the progressive kernel then runs on those tiles only, with the full arithmetic, the exact tests
// and the exact counters.  What is pruned here is pruned by Algorithm 1's first test as well: the result of the step
// does not depend on whether this pass ran.
//
// Error bound.  A scaled value v is hi + lo with |lo| <= 2^-11 |v| (fp16 rounding; values below the smallest normal
// fp16, 2^-14 in scaled units, are instead off by at most 2^-25).  For x.y = sum x_j y_j the dropped terms
// hi*lo' + lo*hi' + lo*lo' sum to at most (2^-10 + 2^-22) ||x|| ||y|| (Cauchy-Schwarz on the front dimensions), so
// the partial distance ||x'||^2 + ||y'||^2 - 2 x'.y' is off by at most 2 * 2^-10 ||x'|| ||y'|| (taken 10 % larger:
// the fp32 accumulation of up to 16384 / 16 matrix instructions adds 1.2e-4 of that product at most) plus a term for
// the subnormal halves; both prefix norms are at hand (they are the ones the exact test uses).  The test's own few
// fp32 operations are covered by a relative guard of 1e-6 on each of its terms.
#include "skm_internal.h"

#include <algorithm>

namespace skm {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int BM = 256, BN = 256, BK = 32;     // workgroup tile; a wavefront owns 128 x 64 of it
constexpr int RT = 128;                         // rows of a row tile of the exact kernel: what a bit of the output speaks for
constexpr int TM = 4, TN = 2;
constexpr int NT = 512;                         // 8 wavefronts: 2 (rows) x 4 (columns)
constexpr int ROW_WORDS = 16;                       // a tile row of a slab: the 32 hi halves = 64 bytes
constexpr int STAGE_WORDS = (BM + BN) * ROW_WORDS;  // one slab of both operands: 32 KB
constexpr int ROWS_PASS = NT / 4;                   // 4 lanes move one tile row: 128 rows per load instruction
constexpr int A_LD = BM / ROWS_PASS;                // 2 load instructions per thread, slab and operand
constexpr int B_LD = BN / ROWS_PASS;
constexpr float kWiden = 2.f * 1.1f / 1024.f;       // 2 * 1.1 * 2^-10, see the error bound above
constexpr float kGuard = 1e-6f;                     // relative guard for the fp32 rounding of the test's own terms

constexpr int DEPTH = 3, NSTAGE = 4;              // slabs requested ahead of the one being multiplied; LDS stages
// wait until at most n of this wavefront's vector memory operations are outstanding (LDS and export counters untouched)
#define SKM_SCREEN_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))

}  // namespace

struct ScreenArgs {
  const uint32_t *A;   // plane of the hi halves of the chunk's points (see launch_split_rows), lda words a row
  int64_t lda;
  int32_t M;
  const uint32_t *B;   // the same of the centroids
  int64_t ldb;
  int32_t N;
  const unsigned int *a_absmax, *b_absmax;
  int32_t dprime;
  const float *arow;       // [M] per point of the chunk: its widened threshold in accumulator units (screen_terms_kernel)
  const float *ycol;       // [N] per centroid: ||y_j[0 : d')||^2 in accumulator units
  uint32_t *colmask;       // [row tiles of 128][maskw]: bit j = some point of the row tile may pass the first test against j
  int32_t maskw;           // words per row tile: 4 per 128 centroids
  unsigned long long *scal;     // step scalars: SC_SCREEN_DIMS
  // exact mode (iteration 1): arow = the band of every row, ycol = ||y_j||^2 in accumulator units
  unsigned int *rowmin;         // [n] running minimum of every point over the tiles done so far (ordered float bits), by row_base + row
  int64_t row_base;
  Pair *pairs;                  // kSubLists parts of sub_capacity slots: the candidates
  unsigned int *pair_count;     // [kSubLists * kSubListStride]
  unsigned int sub_capacity;
  unsigned int *overflow;
  // neighbour modes: rows are queries, columns points, every row of either operand scaled by a power of two of its own
  const float *row_scale, *col_scale;   // [M] (with arow = the row's threshold term), [N] (with ycol = ||x||^2 times scale / 2)
  float *group_min;                     // SCREEN_GROUPS: [M][ngroups] smallest score of every 64 columns
  int32_t ngroups, group0;
  unsigned long long *cand;             // SCREEN_CANDIDATES: [M][cand_cap] (score, point) entries
  unsigned int *cand_count;             // [M]
  unsigned int cand_cap;
  int64_t point0;                       // point of column 0
};

enum { SCREEN_FIRST_TEST = 0, SCREEN_EXACT = 1, SCREEN_GROUPS = 2, SCREEN_CANDIDATES = 3 };

// A workgroup of 8 wavefronts owns 256 points x 256 centroids; a wavefront owns 128 x 64 (4 x 2 accumulators of
// 32 x 32: per matrix instruction three quarters of the fragment bytes of a 64 x 64 arrangement), so the rows of a
// wavefront are exactly one row tile of the exact kernel and its verdict on a column needs no other wavefront.
// LDS rows are 64 bytes (four 16-byte pieces: dims 8 c .. 8 c + 7 of the slab, c = 2 h + kh for half-slab h and lane
// half kh); piece c of row r sits at position c ^ ((r >> 2) & 3), so that the 16-byte fragment reads of 16 consecutive
// rows fall into 16 different bank groups.  Staging is global -> LDS directly, 16 bytes per lane, four lanes per row:
// the lane that fills a position fetches the piece that belongs there.  In global memory (see launch_split_rows) a slab of two
// rows is a line of 128 bytes.  The kernel is persistent: every XCD walks a contiguous range of tiles (column tile fastest inside panels of 8 column tiles), its workgroups take every n-th;
// the first slab of a workgroup's next tile is requested before the finished tile is tested.
//
// EXACT (Algorithm 1, iteration 1, where nothing prunes): the same multiply over ALL dimensions finds, for every point,
// the centroids that can be its nearest.  With v~(i, j) = ||y_j||^2 - 2 (x_i.y_j)~ from the one product and b_i a
// bound of its error (twice the bound of the product: see the top of this file, with the full norms), the true
// nearest j* has v~(i, j*) <= min_j v~(i, j) + 2 b_i.  Every tile takes the minimum of each of its rows over its 256
// columns, lowers the point's running minimum by it (one atomic per row; the tiles of a row run in any order and a
// stale value is only larger), and emits the pairs within 2 b_i of the smaller of the two: j* is among them whenever
// its tile runs.  In random order a row emits in about ln(column tiles) tiles.  The gather kernel then takes the exact
// distance of every emitted pair, and the packed minimum over those is the exact nearest centroid.
//
// SCREEN_GROUPS, SCREEN_CANDIDATES (Section 3.3, ground truth of the recall measurement; see etr.hip): rows are queries,
// columns are points, and the score is ||x_j||^2 - 2 (q_i.x_j)~.  The first mode writes the smallest score of every 64
// columns, the second appends the points whose score does not exceed the row's threshold to the row's list.
template <int MODE>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) screen_kernel(ScreenArgs g) {
  extern __shared__ __align__(16) uint32_t smem[];   // [NSTAGE stages][A: BM rows | B: BN rows][ROW_WORDS]
  __shared__ __align__(16) float s_a[NSTAGE][BM];    // per row of a tile in flight: the widened threshold in accumulator units
  __shared__ __align__(16) float s_y[NSTAGE][BN];    // per column of a tile in flight: its prefix norm in the same units
  constexpr bool EXACT = MODE == SCREEN_EXACT, NEIGH = MODE >= SCREEN_GROUPS;
  __shared__ __align__(16) float s_a2[NEIGH ? NSTAGE : 1][BM], s_y2[NEIGH ? NSTAGE : 1][BN];   // scales of rows and columns
  __shared__ unsigned int s_rmin[EXACT ? BM : 1];    // EXACT: minimum of every row of the tile (ordered float bits)
  __shared__ __align__(16) float s_thr[EXACT ? BM : 1];   // EXACT: emission threshold of every row

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int r32 = lane & 31, kh = lane >> 5;
  const int swz = (r32 >> 2) & 3;
  const int nrt = (g.M + BM - 1) / BM, nct = (g.N + BN - 1) / BN;
  const int ntiles = nrt * nct;
  constexpr int PC = 8;   // column tiles per panel of the tile walk (row tile slowest inside a panel)

  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, nslots = gridDim.x >> 3;
  const int tbase = ntiles >> 3, trem = ntiles & 7;
  const int xstart = xcd * tbase + (xcd < trem ? xcd : trem);
  const int xcount = tbase + (xcd < trem ? 1 : 0);
  const int panel_sz = PC * nrt;
  auto tile_rc = [&](int q, int &rt, int &ct) {   // q-th tile of this XCD -> (row tile, column tile)
    const int logical = xstart + q;
    const int p = logical / panel_sz;
    const int r = logical - p * panel_sz;
    const int pc = (nct - p * PC) < PC ? (nct - p * PC) : PC;
    rt = __builtin_amdgcn_readfirstlane(r / pc);
    ct = __builtin_amdgcn_readfirstlane(p * PC + (r - (r / pc) * pc));
  };

  const int lrow = lane >> 2, lpos = lane & 3;
  const int ld_row = 16 * wave + lrow;                        // + 128 j
  const int ld_c = lpos ^ ((ld_row >> 2) & 3);                // piece that belongs at this lane's position
  const int ld_words = 4 * ld_c;                              // its word offset inside the slab's 16 hi words
  const int nslab = (g.dprime + BK - 1) / BK;                 // (the columns' plane is zero from d' on)

  // ---- the loading side runs DEPTH slabs ahead of the multiplying side, across tile boundaries (a tile of a
  // well-pruned step is two or three slabs: one tile's worth of loads in flight would leave the matrix cores waiting
  // for memory latency most of the time)
  int lq = slot, ls = 0;            // tile (per-XCD number) and slab the next request is for
  int ltile = 0;                    // tiles requested so far (ring slot of the row terms)
  int ljob = 0;                     // slabs requested so far (ring slot of the stage)
  const uint32_t *baseA = g.A, *baseB = g.B;
  unsigned int offA[A_LD], offB[B_LD];   // bytes
  auto aim = [&]() {                // at a tile's first slab: its addresses and its row terms
    if (ls == 0) {
      int rt, ct;
      tile_rc(lq, rt, ct);
      const int row0 = rt * BM, col0 = ct * BN;
      baseA = g.A + (int64_t)row0 * g.lda;
      baseB = g.B + (int64_t)col0 * g.ldb;
      const int limA = g.M - 1 - row0, limB = g.N - 1 - col0;   // rows / columns past the end repeat the last one
#pragma unroll
      for (int j = 0; j < A_LD; ++j) offA[j] = 4u * (unsigned int)((int)split_row(min(ld_row + ROWS_PASS * j, limA), (int)g.lda) + ld_words);
#pragma unroll
      for (int j = 0; j < B_LD; ++j) offB[j] = 4u * (unsigned int)((int)split_row(min(ld_row + ROWS_PASS * j, limB), (int)g.ldb) + ld_words);
      // the tile's row terms (wavefronts 0-3) and column terms (4-7): one more 4-byte load each, straight into LDS
      {
        const int e = tid & (BM - 1);
        const float *src = wave < 4 ? g.arow + row0 + min(e, limA) : g.ycol + col0 + min(e, limB);
        float *dst = (wave < 4 ? s_a[ltile & (NSTAGE - 1)] : s_y[ltile & (NSTAGE - 1)]) + 64 * (wave & 3);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                         (__attribute__((address_space(3))) void *)dst, 4, 0, 0);
        if constexpr (NEIGH) {
          const float *src2 = wave < 4 ? g.row_scale + row0 + min(e, limA) : g.col_scale + col0 + min(e, limB);
          float *dst2 = (wave < 4 ? s_a2[ltile & (NSTAGE - 1)] : s_y2[ltile & (NSTAGE - 1)]) + 64 * (wave & 3);
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src2,
                                           (__attribute__((address_space(3))) void *)dst2, 4, 0, 0);
        }
      }
      ++ltile;
    }
  };
  static_assert(A_LD + B_LD == TM, "one load behind every row block's matrix instructions");
  // one of a slab's loads: a uniform base and a uniform offset, an offset register per load
  auto load = [&](int j) {
    lds_words_t sb = (lds_words_t)smem + (ljob & (NSTAGE - 1)) * STAGE_WORDS + 16 * wave * ROW_WORDS;
    const int at = 128 * ls;
    if (j < A_LD)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(uniform_buffer(baseA), sb + ROWS_PASS * j * ROW_WORDS, 16, (int)offA[j < A_LD ? j : 0], at, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(uniform_buffer(baseB), sb + ROWS_PASS * j * ROW_WORDS, 16, (int)offB[j < A_LD ? 0 : j - A_LD], at, 0, 0);
  };
  auto requested = [&]() {
    ++ljob;
    if (++ls == nslab) {
      ls = 0;
      lq += nslots;
    }
  };

  if (slot >= xcount) return;
  if constexpr (EXACT) {
    if (tid < BM) s_rmin[tid] = 0xffffffffu;
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < DEPTH; ++i)
    if (lq < xcount) {
      aim();
#pragma unroll
      for (int j = 0; j < TM; ++j) load(j);
      requested();
    }

  // Fragments of a slab's two halves of 16 dimensions, read half a slab ahead: those of the second half are requested
  // before the first half is multiplied, those of the next slab's first half behind the barrier in the middle of this
  // slab, before its second half is multiplied.  The matrix cores have work on both sides of the barrier.
  f16x8 a0[TM], b0[TN], a1[TM], b1[TN];
  auto fragments = [&](int job, int h, f16x8 (&x)[TM], f16x8 (&y)[TN]) {
    const uint32_t *st = smem + (job & (NSTAGE - 1)) * STAGE_WORDS;
    const uint32_t *Ab = st + (wm * 128 + r32) * ROW_WORDS + (((2 * h + kh) ^ swz) << 2);
    const uint32_t *Bb = st + (BM + wn * 64 + r32) * ROW_WORDS + (((2 * h + kh) ^ swz) << 2);
#pragma unroll
    for (int t = 0; t < TN; ++t) y[t] = *reinterpret_cast<const f16x8 *>(Bb + t * 32 * ROW_WORDS);
#pragma unroll
    for (int t = 0; t < TM; ++t) x[t] = *reinterpret_cast<const f16x8 *>(Ab + t * 32 * ROW_WORDS);
  };
  // Slab `job` has arrived, for every wavefront's share of it, and the stage of slab job - 2 is free.  Only the requests
  // made after it may be outstanding: one slab of loads (counted in order; the tile terms in between only make the wait
  // stricter); near the end fewer requests follow, so everything is awaited.  (A bare barrier: a fenced one would first
  // wait for every load in flight.  The reads of slab job - 2 have been consumed by matrix instructions before this
  // point, those of slab job - 1 concern a stage that stays as it is.)
  auto arrived = [&](int later) {
    if (lq < xcount) {
      if (later == 2) SKM_SCREEN_VMCNT(2 * (A_LD + B_LD));
      else SKM_SCREEN_VMCNT(A_LD + B_LD);
    } else {
      SKM_SCREEN_VMCNT(0);
    }
    asm volatile("" : : : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
  };
  arrived(2);
  fragments(0, 0, a0, b0);

  unsigned long long dims_done = 0ull;
  int cjob = 0, ctile = 0;
  for (int q = slot; q < xcount; q += nslots, ++ctile) {
    int rt, ct;
    tile_rc(q, rt, ct);
    const int col0 = ct * BN;
    bool colok[TN];
#pragma unroll
    for (int b = 0; b < TN; ++b) colok[b] = col0 + wn * 64 + b * 32 + r32 < g.N;
    f32x16 acc[TM][TN];
    for (int s = 0; s < nslab; ++s, ++cjob) {
      if (s == 0 && (EXACT || NEIGH)) {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
      }
      if (s == 0 && MODE == SCREEN_FIRST_TEST) {      // every accumulator element starts from its row's term
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {   // accumulator elements 4 q4 .. 4 q4 + 3 are four consecutive rows
            const float4 a4 = *reinterpret_cast<const float4 *>(&s_a[ctile & (NSTAGE - 1)][wm * 128 + a * 32 + 8 * q4 + 4 * kh]);
#pragma unroll
            for (int b = 0; b < TN; ++b) {
              acc[a][b][4 * q4 + 0] = a4.x;
              acc[a][b][4 * q4 + 1] = a4.y;
              acc[a][b][4 * q4 + 2] = a4.z;
              acc[a][b][4 * q4 + 3] = a4.w;
            }
          }
      }
      fragments(cjob, 1, a1, b1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0[a], b0[b], acc[a][b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      const bool next = s + 1 < nslab || q + nslots < xcount;
      arrived(1);
      // Slab cjob + DEPTH -> the stage slab cjob - 1 was in (NSTAGE = DEPTH + 1).  Its loads go between the matrix
      // instructions: a wavefront whose load has to queue for the address unit issues nothing else meanwhile.  (All four
      // ahead of them, 1000 queries against 1M x 768: 3.02 instead of 2.93 ms; 128 x 64 a wavefront in 16 dimensions is
      // 256 cycles of matrix work, so there is room for a load behind every two instructions.)
      const bool more = lq < xcount;
      if (more) aim();
      if (next) fragments(cjob + 1, 0, a0, b0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int a = 0; a < TM; ++a) {
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1[a], b1[b], acc[a][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (more) load(a);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) requested();
    }
    dims_done += (unsigned long long)(BK * nslab);

    if constexpr (NEIGH) {
      // score of (row, column) = (rq ct - acc) 2 / (rq sj), rq and sj the two scales, ct = ||x||^2 sj / 2
      const int slot_t = ctile & (NSTAGE - 1);
      const float c0 = s_y[slot_t][wn * 64 + r32], c1 = s_y[slot_t][wn * 64 + 32 + r32];
      const float j0 = s_y2[slot_t][wn * 64 + r32], j1 = s_y2[slot_t][wn * 64 + 32 + r32];
      int zero = 0;   // (renewed every four rows so that their terms are fetched four at a time: see the EXACT form)
      if constexpr (MODE == SCREEN_GROUPS) {
        const float i0 = colok[0] ? 1.f / j0 : 0.f, i1 = colok[1] ? 1.f / j1 : 0.f;   // (powers of two: exact)
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            if ((v & 3) == 0) asm volatile("" : "+v"(zero) : : "memory");
            const int rl = wm * 128 + a * 32 + 8 * (v >> 2) + 4 * kh + (v & 3) + zero;
            const float rq = s_a2[slot_t][rl];
            float m = 3.0e38f;
            if (colok[0]) m = fmaf(rq, c0, -acc[a][0][v]) * i0;
            if (colok[1]) m = fminf(m, fmaf(rq, c1, -acc[a][1][v]) * i1);
            m = fminf(m, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, m), 0xB1, 0xF, 0xF, false)));
            m = fminf(m, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, m), 0x4E, 0xF, 0xF, false)));
            m = fminf(m, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, m), 0x141, 0xF, 0xF, false)));
            m = fminf(m, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, m), 0x140, 0xF, 0xF, false)));
            m = fminf(m, __shfl_xor(m, 16, 64));
            const int row = rt * BM + rl, grp = g.group0 + ct * (BN / 64) + wn;
            if (r32 == 0 && row < g.M && col0 + wn * 64 < g.N) g.group_min[(int64_t)row * g.ngroups + grp] = m * (2.f / rq);
          }
      } else {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            if ((v & 3) == 0) asm volatile("" : "+v"(zero) : : "memory");
            const int rl = wm * 128 + a * 32 + 8 * (v >> 2) + 4 * kh + (v & 3) + zero;
            const float rq = s_a2[slot_t][rl], rterm = s_a[slot_t][rl];
            const bool e0 = colok[0] && acc[a][0][v] >= fmaf(rq, c0, rterm * j0);
            const bool e1 = colok[1] && acc[a][1][v] >= fmaf(rq, c1, rterm * j1);
            if (__ballot(e0 || e1)) {
              const int row = rt * BM + rl;
              if (row < g.M) {
                if (e0) {
                  const unsigned int p = atomicAdd(g.cand_count + row, 1u);
                  const float sc = fmaf(rq, c0, -acc[a][0][v]) * (2.f / rq) * (1.f / j0);
                  if (p < g.cand_cap)
                    g.cand[(int64_t)row * g.cand_cap + p] =
                        ((unsigned long long)f2ord(sc) << 32) | (unsigned int)(g.point0 + col0 + wn * 64 + r32);
                }
                if (e1) {
                  const unsigned int p = atomicAdd(g.cand_count + row, 1u);
                  const float sc = fmaf(rq, c1, -acc[a][1][v]) * (2.f / rq) * (1.f / j1);
                  if (p < g.cand_cap)
                    g.cand[(int64_t)row * g.cand_cap + p] =
                        ((unsigned long long)f2ord(sc) << 32) | (unsigned int)(g.point0 + col0 + wn * 64 + 32 + r32);
                }
              }
            }
          }
      }
      continue;
    }
    if constexpr (EXACT) {
      // The rows are shared out among the lanes on the way to their minima, and the candidates are counted before room
      // for all of a wavefront's is taken at once: five lane moves and an LDS exchange per row, and a trip to the list's
      // counter for every row with a candidate, were 27 of the 54 us of a tile of 768 dimensions.
      const int slot_t = ctile & (NSTAGE - 1);
      // ---- minimum of every row over the tile's columns
      const float *yc = s_y[slot_t] + wn * 64 + r32;
      const float y0 = colok[0] ? yc[0] : 3.0e38f, y1 = colok[1] ? yc[32] : 3.0e38f;
      const int my_row = rt * BM + tid;   // (wavefronts 0 to 3)
#pragma unroll
      for (int h = 0; h < TM; h += 2) {
        const float m = reduce_rows32_f32([&](int a, int v) { return fminf(y0 - acc[h + a][0][v], y1 - acc[h + a][1][v]); }, lane);
        const int v = r32 & 15;
        atomicMin(&s_rmin[wm * 128 + (h + (r32 >> 4)) * 32 + 8 * (v >> 2) + 4 * kh + (v & 3)], f2ord(m));
      }
      __syncthreads();
      // ---- the point's running minimum takes it; the threshold is the smaller of the two plus the band
      if (tid < BM) {
        float thr = -3.0e38f;
        if (my_row < g.M) {
          const unsigned int local = s_rmin[tid];
          // (not a read ahead of the minimum: the tiles of a row that end together would not see each other's)
          const unsigned int old = atomicMin(g.rowmin + g.row_base + my_row, local);
          thr = ord2f(old < local ? old : local) + s_a[slot_t][tid];
        }
        s_thr[tid] = thr;
        s_rmin[tid] = 0xffffffffu;   // for the next tile
      }
      __syncthreads();
      // ---- emit the pairs at or below the threshold of their row: bit 2 v + b of word a
      unsigned int bits[TM];
#pragma unroll
      for (int a = 0; a < TM; ++a) {
        asm volatile("" : : : "memory");   // (one block's thresholds at a time: all 64 would not fit the registers)
        bits[a] = 0u;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const float4 t4 = *reinterpret_cast<const float4 *>(&s_thr[wm * 128 + a * 32 + 8 * q4 + 4 * kh]);
          const float thr[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
          for (int u = 0; u < 4; ++u) {   // (v~ <= thr written from the accumulator's side)
            const int v = 4 * q4 + u;
            bits[a] |= acc[a][0][v] >= y0 - thr[u] ? 1u << (2 * v) : 0u;
            bits[a] |= acc[a][1][v] >= y1 - thr[u] ? 2u << (2 * v) : 0u;
          }
        }
      }
      int mine = 0;
#pragma unroll
      for (int a = 0; a < TM; ++a) mine += __popc(bits[a]);
      if (__ballot(mine != 0)) {
        int upto = mine;   // list slots: lane by lane (prefix sum of the lanes' counts), then bit by bit
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xF, 0xF, false);   // row_shr:1
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xF, 0xF, false);   // row_shr:2
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xF, 0xF, false);   // row_shr:4
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xF, 0xF, false);   // row_shr:8
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x142, 0xA, 0xF, false);   // row_bcast:15
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x143, 0xC, 0xF, false);   // row_bcast:31
        const unsigned int tot = (unsigned int)__builtin_amdgcn_readlane(upto, 63);
        const int xsub = blockIdx.x & 7;
        unsigned int base = 0;
        if (lane == 0) base = atomicAdd(g.pair_count + xsub * kSubListStride, tot);
        base = __builtin_amdgcn_readfirstlane(base);
        if ((unsigned long long)base + tot > (unsigned long long)g.sub_capacity) {
          if (lane == 0) atomicOr(g.overflow, 1u);
        } else {
          Pair *dst = g.pairs + (size_t)xsub * g.sub_capacity + base + (unsigned int)(upto - mine);
          Pair pr;
          pr.p = 0.f;
          pr.tau = 3.0e38f;
#pragma unroll
          for (int a = 0; a < TM; ++a)
            while (bits[a]) {
              const int e = __builtin_ctz(bits[a]), v = e >> 1;
              bits[a] &= bits[a] - 1u;
              pr.i = (int32_t)(g.row_base + rt * BM + wm * 128 + a * 32 + 8 * (v >> 2) + 4 * kh + (v & 3));
              pr.j = col0 + wn * 64 + 32 * (e & 1) + r32;
              *dst++ = pr;
            }
        }
      }
      continue;
    }

    // ---- widened first test: a column stays if any row of this wavefront's row tile may pass theta(d', tau) against it
    bool alive[TN];
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      float best = acc[0][b][0];
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) best = fmaxf(best, acc[a][b][v]);
      alive[b] = best >= s_y[ctile & (NSTAGE - 1)][wn * 64 + b * 32 + r32];
    }
    const int rtile = rt * (BM / RT) + wm;   // the row tile of 128 this wavefront speaks for
    if (rtile * RT < g.M) {
#pragma unroll
      for (int b = 0; b < TN; ++b) {
        const unsigned long long bal = __ballot(alive[b] && colok[b]);
        const unsigned int w = (unsigned int)bal | (unsigned int)(bal >> 32);   // column r32: lanes r32 and r32 + 32
        const int word = ct * (BN / 32) + wn * 2 + b;
        if (lane == 0 && word < g.maskw) g.colmask[(int64_t)rtile * g.maskw + word] = w;
      }
    }
  }
  if (!NEIGH && tid == 0 && dims_done)   // (in units of the exact kernel's 128 x 128 tiles: four per tile of this kernel)
    atomicAdd(g.scal + (size_t)(blockIdx.x & (kStatReplicas - 1)) * SC_COUNT + SC_SCREEN_DIMS, 4ull * dims_done);
}

// ---------------------------------------------------------------- bits -> lists of listed columns per row tile
// cnt[rt] = set bits of row tile rt (one wavefront per row tile)
__global__ void __launch_bounds__(256) mask_count_kernel(const uint32_t *mask, int32_t nrt, int32_t maskw, int32_t *cnt) {
  const int lane = threadIdx.x & 63;
  const int rt = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (rt >= nrt) return;
  int c = 0;
  for (int w = lane; w < maskw; w += 64) c += __popc(mask[(int64_t)rt * maskw + w]);
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) c += __shfl_xor(c, m, 64);
  if (lane == 0) cnt[rt] = c;
}

// every column of every row tile (the columns past the last one stay out)
__global__ void __launch_bounds__(256) mask_all_kernel(uint32_t *mask, int64_t words, int32_t maskw, int32_t N) {
  for (int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x; w < words; w += (int64_t)gridDim.x * 256) {
    const int left = N - 32 * (int)(w % maskw);
    mask[w] = left >= 32 ? 0xffffffffu : left > 0 ? (1u << left) - 1u : 0u;
  }
}

// first[rt] = first tile of row tile rt (tiles of kListCols listed columns, row tiles in order), *ntiles = their number
__global__ void __launch_bounds__(1024) mask_scan_kernel(const int32_t *cnt, int32_t nrt, int32_t *first, int32_t *ntiles,
                                                         unsigned long long *scal) {
  __shared__ int s_part[1024];
  const int tid = threadIdx.x;
  const int per = (nrt + 1023) / 1024;
  const int lo = min(tid * per, nrt), hi = min(lo + per, nrt);
  int sum = 0, listed = 0;
  for (int r = lo; r < hi; ++r) {
    sum += (cnt[r] + kListCols - 1) / kListCols;
    listed += (cnt[r] + 127) >> 7;
  }
  s_part[tid] = sum;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {   // inclusive scan of the per-thread sums
    const int v = tid >= off ? s_part[tid - off] : 0;
    __syncthreads();
    s_part[tid] += v;
    __syncthreads();
  }
  int run = s_part[tid] - sum;
  for (int r = lo; r < hi; ++r) {
    first[r] = run;
    run += (cnt[r] + kListCols - 1) / kListCols;
  }
  if (tid == 1023) *ntiles = s_part[1023];
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) listed += __shfl_xor(listed, m, 64);
  if ((tid & 63) == 0 && listed) atomicAdd(scal + SC_LISTED_TILES, (unsigned long long)listed);   // (in tiles of 128)
}

// One workgroup per row tile: the ids of its set bits in ascending order, padded with -1 to a multiple of kListCols, one
// tile of kListCols after the other.  Tiles are placed so that the tiles in work at a time share rows and centroids:
// kListGroup row tiles together, tile 0 of each, then tile 1 of each, ... (all lists ascend, so the c-th tiles of two row
// tiles name mostly the same centroids).  Row tile after row tile every centroid came from outside the XCD's L2 once per
// row tile: 5.4 TB/s of misses in an assignment of 2.5M x 384 to 32768 centroids.
__global__ void __launch_bounds__(256) mask_fill_kernel(const uint32_t *mask, int32_t nrt, int32_t maskw, const int32_t *cnt,
                                                        const int32_t *first, int32_t *col_list, int2 *tile_rt,
                                                        const int32_t *prev, int32_t *list_pos, int64_t row_base, int32_t M) {
  __shared__ int s_wave[4];
  __shared__ int s_pos[256];   // positions of the chunk's words
  __shared__ unsigned int s_bits[256];
  __shared__ unsigned short s_ids[256 * 32];   // the chunk's ids, from its first
  __shared__ int s_base;
  const int rt = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int total = cnt[rt];
  const int nt = (total + kListCols - 1) / kListCols;
  const int g0 = rt / kListGroup * kListGroup;
  int others[kListGroup];   // tiles of the group's row tiles
#pragma unroll
  for (int r = 0; r < kListGroup; ++r) others[r] = g0 + r < nrt ? (cnt[g0 + r] + kListCols - 1) / kListCols : 0;
  const int start = first[g0];
  auto place = [&](int c) {   // of tile c of this row tile
    int p = start;
#pragma unroll
    for (int r = 0; r < kListGroup; ++r) p += min(others[r], c) + (g0 + r < rt && others[r] > c ? 1 : 0);
    return p;
  };
  const int inc = tid < RT && rt * RT + tid < M ? prev[row_base + rt * RT + tid] : -1;   // incumbent of row tid of the row tile
  int at_pos = -1;
  if (tid == 0) s_base = 0;
  __syncthreads();
  for (int w0 = 0; w0 < maskw; w0 += 256) {
    const int w = w0 + tid;
    unsigned int bits = w < maskw ? mask[(int64_t)rt * maskw + w] : 0u;
    const int mine = __popc(bits);
    int incl = mine;   // inclusive prefix inside the wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(incl, off, 64);
      if (lane >= off) incl += v;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int pos = incl - mine;
    for (int ww = 0; ww < wave; ++ww) pos += s_wave[ww];
    const int base = s_base, here = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    s_pos[tid] = base + pos;
    s_bits[tid] = bits;
    while (bits) {
      s_ids[pos++] = (unsigned short)(32 * tid + __builtin_ctz(bits));
      bits &= bits - 1u;
    }
    __syncthreads();
    // (through LDS, 256 ids a store: each thread storing its own word's ids, the lists of 2.5M x 384 against 32768 centroids took
    // 1.25 ms a launch)
    for (int e = tid; e < here; e += 256) {
      const int p = base + e;
      col_list[(int64_t)place(p / kListCols) * kListCols + p % kListCols] = 32 * w0 + s_ids[e];
    }
    if (inc >= 32 * w0 && inc < 32 * (w0 + 256)) {   // the row's incumbent is in this chunk of words
      const unsigned int b = s_bits[(inc >> 5) - w0], bit = 1u << (inc & 31);
      if (b & bit) at_pos = s_pos[(inc >> 5) - w0] + __popc(b & (bit - 1u));
    }
    __syncthreads();
    if (tid == 0) s_base = base + here;
    __syncthreads();
  }
  if (nt > 0) {
    int32_t *out = col_list + (int64_t)place(nt - 1) * kListCols;
    for (int p = total - (nt - 1) * kListCols + tid; p < kListCols; p += 256) out[p] = -1;
  }
  for (int t = tid; t < nt; t += 256) tile_rt[place(t)] = make_int2(rt, t * kListCols);
  if (inc >= 0) list_pos[row_base + rt * RT + tid] = at_pos;
}

// The test of a pair, theta + widening - ||x'||^2 >= ||y'||^2 - 2 x'.y', in accumulator units (the accumulator holds
// x'.y' times the two scales; K = 2 / scales > 0):   acc + a_i >= y_j   with
//   a_i = (theta_i - ||x'_i||^2 + slack + guard + widening ||x'_i|| max_j ||y'_j||) / K,   y_j = ||y'_j||^2 (1 - guard) / K.
// a_i is what the row's accumulator elements START from, so after the last slab the verdict on a column is one maximum
// over its rows against one number.  (The widening uses the largest centroid norm instead of the column's own: looser
// only for centroids whose front part is small.)  slack: halves below the smallest normal fp16 (off by up to 2^-25
// scaled = 2^-39 of the bound each, times the other operand, two operands, d' terms, times 2 for the distance).
__global__ void __launch_bounds__(256) screen_terms_kernel(const float *tau, const float *xn, int64_t row_base, int32_t M,
                                                           const float *yn, int32_t N, const float *ynmax, float ratio0,
                                                           int32_t dprime, const unsigned int *a_absmax,
                                                           const unsigned int *b_absmax, float *arow, float *ycol,
                                                           int exact) {
  const float ax = __builtin_bit_cast(float, *a_absmax), ay = __builtin_bit_cast(float, *b_absmax);
  const float slack = (float)dprime * ax * ay * (1.f / 8589934592.f);   // d' * max|x| * max|y| * 2^-33
  const float inv_k = 0.5f * split_scale(*a_absmax) * split_scale(*b_absmax);
  const float symax = sqrtf(fmaxf(*ynmax, 0.f));
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (exact) {
    // exact mode: the band 2 b_i around the smallest v~ of a row inside which the true nearest centroid must lie:
    // b_i = 2 * (bound of the product's error) = widening ||x_i|| max_j ||y_j||, plus the slack and a guard for the
    // rounding of the values compared (their size is at most ||y||^2 + 2 ||x|| ||y||); y_j = ||y_j||^2 / K
    if (i < M) {
      const float xs = sqrtf(fmaxf(xn[row_base + i], 0.f));
      arow[i] = (2.f * kWiden * xs * symax + 2.f * slack + 4.f * kGuard * (symax * symax + 2.f * xs * symax)) * inv_k;
    }
    if (i < N) ycol[i] = yn[i] * inv_k;
    return;
  }
  if (i < M) {
    const float x2 = xn[row_base + i];
    const float th = ratio0 * tau[row_base + i];
    arow[i] = (th - x2 + slack + kGuard * (th + x2) + kWiden * sqrtf(fmaxf(x2, 0.f)) * symax) * inv_k;
  }
  if (i < N) ycol[i] = yn[i] * (1.f - kGuard) * inv_k;
}

// Workgroup 0: *out = max of yn[0 .. n) (non-negative values: their bit patterns order like the numbers).
// Workgroup 1 + m (with ynp): the terms of the widened test at checkpoint m, widen[m] = (widening 1.1 2^-9 times the
// largest centroid norm over the dimensions d' .. t_m, slack for halves below the smallest normal fp16 + guard for the
// rounding of values of the centroids' size).
__global__ void __launch_bounds__(1024) max_value_kernel(const float *yn, const float *ynp, int32_t n, float *out,
                                                         float2 *widen, int32_t ds, const unsigned int *a_absmax,
                                                         const unsigned int *b_absmax, stamp_t *stamp) {
  put_stamp(stamp);
  __shared__ float red[16], red2[16];
  const float *v = blockIdx.x == 0 ? yn : ynp + (int64_t)(blockIdx.x - 1) * n;
  float m = 0.f, p = 0.f;
  for (int i = threadIdx.x; i < n; i += 1024) {
    m = fmaxf(m, v[i]);
    p = fmaxf(p, v[i] - yn[i]);
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    m = fmaxf(m, __shfl_xor(m, off, 64));
    p = fmaxf(p, __shfl_xor(p, off, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = m;
    red2[threadIdx.x >> 6] = p;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) {
      m = fmaxf(m, red[w]);
      p = fmaxf(p, red2[w]);
    }
    if (blockIdx.x == 0) {
      *out = m;
    } else {
      const float slack = (float)ds * __builtin_bit_cast(float, *a_absmax) * __builtin_bit_cast(float, *b_absmax) * (1.f / 8589934592.f);
      widen[blockIdx.x - 1] = make_float2(kWiden * sqrtf(p + kGuard * m), slack + 2.f * kGuard * m);
    }
  }
}

namespace {
// LDS size and grid, once per process (the initialisation of a function-local static is synchronised between threads)
struct ScreenSetup {
  hipError_t rc;
  int wgs = 0;
  ScreenSetup() {
    constexpr int smem = NSTAGE * STAGE_WORDS * (int)sizeof(uint32_t);
    const void *forms[4] = {reinterpret_cast<const void *>(screen_kernel<SCREEN_FIRST_TEST>),
                            reinterpret_cast<const void *>(screen_kernel<SCREEN_EXACT>),
                            reinterpret_cast<const void *>(screen_kernel<SCREEN_GROUPS>),
                            reinterpret_cast<const void *>(screen_kernel<SCREEN_CANDIDATES>)};
    rc = hipSuccess;
    for (const void *f : forms)
      if (rc == hipSuccess) rc = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    wgs = cus;   // one workgroup of eight wavefronts per CU
  }
};
const ScreenSetup &screen_setup() {
  static const ScreenSetup setup;
  return setup;
}
}  // namespace

hipError_t launch_neighbour_screen(const NeighbourLaunch &a, bool groups, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (a.ds % 32 != 0 || (reinterpret_cast<uintptr_t>(a.A) & 15u) || (reinterpret_cast<uintptr_t>(a.B) & 15u)) return hipErrorInvalidValue;
  constexpr size_t smem = (size_t)NSTAGE * STAGE_WORDS * sizeof(uint32_t);
  const ScreenSetup &setup = screen_setup();
  if (setup.rc != hipSuccess) return setup.rc;
  const int64_t ntiles = (int64_t)((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  if (ntiles > 0x7fffffffLL) return hipErrorInvalidValue;
  ScreenArgs g{};
  g.A = a.A; g.lda = a.ds / 2; g.M = a.M;
  g.B = a.B; g.ldb = a.ds / 2; g.N = a.N;
  g.dprime = a.ds;
  g.arow = a.row_term; g.ycol = a.col_term; g.row_scale = a.row_scale; g.col_scale = a.col_scale;
  g.group_min = a.group_min; g.ngroups = a.ngroups; g.group0 = a.group0;
  g.cand = a.cand; g.cand_count = a.cand_count; g.cand_cap = a.cand_cap; g.point0 = a.point0;
  const int64_t grid = std::max<int64_t>(8, std::min<int64_t>(setup.wgs, (ntiles + 7) / 8 * 8));
  if (groups) hipLaunchKernelGGL(screen_kernel<SCREEN_GROUPS>, dim3((unsigned)grid), dim3(NT), smem, st, g);
  else hipLaunchKernelGGL(screen_kernel<SCREEN_CANDIDATES>, dim3((unsigned)grid), dim3(NT), smem, st, g);
  return hipGetLastError();
}

hipError_t launch_screen(const ScreenLaunch &a, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (a.dprime % 16 != 0 || a.dprime < 16 || a.dprime > a.ds || a.lda != split_ld(a.ds) / 2 || a.ldb != split_ld(a.ds) / 2 ||
      (reinterpret_cast<uintptr_t>(a.A) & 15u) || (reinterpret_cast<uintptr_t>(a.B) & 15u) || a.N > (1 << 24))
    return hipErrorInvalidValue;
  if (a.exact && (!a.rowmin || !a.pairs || !a.pair_count || !a.overflow)) return hipErrorInvalidValue;
  constexpr size_t smem = (size_t)NSTAGE * STAGE_WORDS * sizeof(uint32_t);
  const ScreenSetup &setup = screen_setup();
  if (setup.rc != hipSuccess) return setup.rc;
  const int nrt = (a.M + RT - 1) / RT, nct = (a.N + 127) / 128;   // row tiles and column tiles of the exact kernel
  const int64_t ntiles = (int64_t)((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  if (ntiles > 0x7fffffffLL) return hipErrorInvalidValue;
  ScreenArgs g{};
  g.A = a.A; g.lda = a.lda; g.M = a.M; g.B = a.B; g.ldb = a.ldb; g.N = a.N;
  g.a_absmax = a.a_absmax; g.b_absmax = a.b_absmax;
  g.dprime = a.dprime;
  float *ynmax = reinterpret_cast<float *>(a.ntiles + 1);   // (the word after the tile count)
  hipLaunchKernelGGL(max_value_kernel, dim3(a.widen ? (unsigned)a.nb + 2 : 1), dim3(1024), 0, st, a.yn, a.ynp, a.N, ynmax,
                     a.widen, a.ds, a.a_absmax, a.b_absmax, a.stamp);
  if (!a.all)
    hipLaunchKernelGGL(screen_terms_kernel, dim3((unsigned)((std::max<int64_t>(a.M, a.N) + 255) / 256)), dim3(256), 0, st,
                     a.tau, a.xn, a.row_base, a.M, a.yn, a.N, (const float *)ynmax, a.ratio0, a.dprime, a.a_absmax,
                     a.b_absmax, a.arow, a.ycol, a.exact ? 1 : 0);
  g.arow = a.arow; g.ycol = a.ycol; g.colmask = a.colmask; g.maskw = 4 * nct;
  g.scal = a.scal;
  g.rowmin = a.rowmin; g.row_base = a.row_base; g.pairs = a.pairs; g.pair_count = a.pair_count;
  g.sub_capacity = a.sub_capacity; g.overflow = a.overflow;
  const int64_t grid = std::max<int64_t>(8, std::min<int64_t>(setup.wgs, (ntiles + 7) / 8 * 8));
  if (a.exact) {
    hipLaunchKernelGGL(screen_kernel<SCREEN_EXACT>, dim3((unsigned)grid), dim3(NT), smem, st, g);
    return hipGetLastError();
  }
  if (a.all) {
    const int64_t words = (int64_t)nrt * 4 * nct;
    hipLaunchKernelGGL(mask_all_kernel, dim3((unsigned)std::min<int64_t>((words + 255) / 256, (int64_t)setup.wgs * 8)), dim3(256), 0, st, a.colmask,
                       words, 4 * nct, a.N);
  } else {
    hipLaunchKernelGGL(screen_kernel<SCREEN_FIRST_TEST>, dim3((unsigned)grid), dim3(NT), smem, st, g);
  }
  hipError_t rc = hipGetLastError();
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(mask_count_kernel, dim3((unsigned)((nrt + 3) / 4)), dim3(256), 0, st, a.colmask, nrt, 4 * nct, a.cnt);
  hipLaunchKernelGGL(mask_scan_kernel, dim3(1), dim3(1024), 0, st, a.cnt, nrt, a.first, a.ntiles, a.scal);
  hipLaunchKernelGGL(mask_fill_kernel, dim3((unsigned)nrt), dim3(256), 0, st, a.colmask, nrt, 4 * nct, a.cnt, a.first,
                     a.col_list, a.tile_rt, a.prev, a.list_pos, a.row_base, a.M);
  return hipGetLastError();
}

}  // namespace skm
