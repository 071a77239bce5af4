// Random orthogonal matrix on the device (Algorithm 1, GenerateRandomRotationMatrix; Section 3.1).
//
// The rows of a d x d matrix of independent standard normals are orthonormalised by Gram-Schmidt, which
// gives a Haar-distributed orthogonal matrix.  Everything is fp64 (the result is rounded to fp32 at the
// end) and runs in panels of 64 rows (the chain of small dependent kernels per panel is what the run time is made of,
// so fewer, fatter panels are faster):
//   1. the panel is cleared of all finished rows (coefficients C = W Q^T, then W -= C Q);
//   2. the panel is orthonormalised in itself by Cholesky QR: G = W W^T = L L^T, W <- L^-1 W,
//      which is Gram-Schmidt inside the panel written as three dense steps.
// Both steps are done twice in the last 256 rows, where the complement of the finished rows gets small.
// The normals come from a counter-based generator (splitmix64 of seed and element index, Box-Muller), so
// the matrix depends on (d, seed) only and no kernel uses atomics: the result is reproducible bit by bit.
#include "skm_internal.h"

namespace skm {

namespace {
constexpr int PB = 64;  // panel rows

__device__ inline uint64_t mix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ULL;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

__global__ void gauss_fill_kernel(double *Q, int64_t n_pairs, uint64_t seed) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_pairs) return;
  const uint64_t a = mix64(seed + 2 * (uint64_t)t), b = mix64(seed + 2 * (uint64_t)t + 1);
  double u1 = (double)(a >> 11) * (1.0 / 9007199254740992.0);
  const double u2 = (double)(b >> 11) * (1.0 / 9007199254740992.0);
  if (u1 < 1e-300) u1 = 1e-300;
  const double m = sqrt(-2.0 * log(u1));
  Q[2 * t] = m * cos(6.283185307179586 * u2);
  Q[2 * t + 1] = m * sin(6.283185307179586 * u2);
}

// All products of a panel run on the fp64 matrix instruction v_mfma_f64_16x16x4_f64: one operand pair of doubles per lane
// feeds 16 multiply-adds where the vector form read a double from LDS for each, and LDS reads were what the products
// waited for.  Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds D[l / 16 + 4 v][l % 16] in element v.
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ inline f64x4 mma_f64(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
// LDS row strides (doubles): operands read by rows of 16 lanes along k (stride 66: the 32 lanes of half a read hit 64
// different banks), operands read along the row (stride 80: two rows are 32 banks apart)
constexpr int SK = 66, SR = 80;
// (the same for a whole wavefront: row addresses stay in scalar registers)
__device__ inline int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// C = W Q_done^T as a small tiled product: workgroup (jt, ks) owns 32 finished rows j0 .. j0+31 and the
// ks-th part of the columns; Cpart[ks][r][j] holds its share of <W_r, Q_j>.  Wavefront w: panel rows 16 w .. + 15.
// What bounds it is latency: a workgroup's few slabs of 64 columns one after the other, so a slab's values are
// requested while the one before it is multiplied.
constexpr int KS = 6;    // column splits of the coefficient product
constexpr int JR = 128;  // finished rows per workgroup of the update (the row range is split into ceil(p0 / JR) parts)
__global__ void __launch_bounds__(256) coeff_kernel(const double *Q, int d, int p0, int nr, double *Cpart) {
  __shared__ double s_w[PB * SK], s_q[32 * SK];
  const int j0 = blockIdx.x * 32, ks = blockIdx.y;
  const int kchunk = ((d + KS - 1) / KS + 63) / 64 * 64;
  const int kbeg = ks * kchunk, kend = min(d, kbeg + kchunk);
  const int lane = threadIdx.x & 63, w = wave_id(), l16 = lane & 15, lk = lane >> 4;
  f64x4 acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
  double vw[16], vq[8];
  auto fetch = [&](int c0) {
    const int cc = min(c0 + lane, d - 1);
#pragma unroll
    for (int u = 0; u < 16; ++u) vw[u] = Q[(int64_t)min(p0 + 4 * u + w, p0 + nr - 1) * d + cc];
#pragma unroll
    for (int u = 0; u < 8; ++u) vq[u] = Q[(int64_t)min(j0 + 4 * u + w, p0 - 1) * d + cc];
  };
  if (kbeg < kend) fetch(kbeg);
  for (int c0 = kbeg; c0 < kend; c0 += 64) {
    const double live = c0 + lane < kend ? 1.0 : 0.0;   // (loads unconditional at valid addresses; what lies outside counts as zero)
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; ++u) s_w[(4 * u + w) * SK + lane] = vw[u] * (4 * u + w < nr ? live : 0.0);
#pragma unroll
    for (int u = 0; u < 8; ++u) s_q[(4 * u + w) * SK + lane] = vq[u];
    __syncthreads();
    if (c0 + 64 < kend) fetch(c0 + 64);
#pragma unroll
    for (int k = 0; k < 64; k += 4) {
      const double a = s_w[(16 * w + l16) * SK + k + lk];
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[b] = mma_f64(a, s_q[(16 * b + l16) * SK + k + lk], acc[b]);
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int j = j0 + 16 * b + l16;
    if (j < p0)
#pragma unroll
      for (int v = 0; v < 4; ++v) Cpart[((int64_t)ks * PB + 16 * w + lk + 4 * v) * p0 + j] = acc[b][v];
  }
}

// acc[b] += A (rows 16 w .. + 15, 64 values of k) x B (64 values of k, columns 16 b .. + 15), both in LDS
__device__ inline void mma_64x64(const double *s_a, const double *s_b, int w, int l16, int lk, f64x4 (&acc)[4]) {
#pragma unroll
  for (int k = 0; k < 64; k += 4) {
    const double a = s_a[(16 * w + l16) * SK + k + lk];
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = mma_f64(a, s_b[(k + lk) * SR + 16 * b + l16], acc[b]);
  }
}

// Wpart[js][r][c] = sum over the js-th JR rows of the finished rows j of C[r][j] Q[j][c], with
// C[r][j] = sum_ks Cpart[ks][r][j], on a tile of 64 columns.  (The second 64 rows are requested while the first are
// multiplied.)
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) apply_kernel(const double *Q, int d, int p0, int nr, const double *Cpart,
                                                    double *Wpart) {
  __shared__ double s_c[PB * SK], s_q[64 * SR];
  const int cb = blockIdx.x * 64, js = blockIdx.y;
  const int jbeg = js * JR, jend = min(p0, jbeg + JR);
  const int t = threadIdx.x & 63, w = wave_id(), l16 = t & 15, lk = t >> 4;
  f64x4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
  double vc[KS][16], vq[16];
  auto fetch = [&](int j0) {
    // (every load unconditional at a valid address, so that all of them are in flight together; what lies outside counts
    // as zero through C)
    const int jc = min(j0 + t, p0 - 1), cc = min(cb + t, d - 1);
#pragma unroll
    for (int u = 0; u < 16; ++u) vq[u] = Q[(int64_t)min(j0 + 4 * u + w, p0 - 1) * d + cc];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int u = 0; u < 16; ++u) vc[ks][u] = Cpart[((int64_t)ks * PB + 4 * u + w) * p0 + jc];
  };
  fetch(jbeg);
  for (int j0 = jbeg; j0 < jend; j0 += 64) {
    const double live = j0 + t < jend ? 1.0 : 0.0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      double c = 0.0;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) c += vc[ks][u];
      s_q[(4 * u + w) * SR + t] = vq[u];
      s_c[(4 * u + w) * SK + t] = c * live;
    }
    __syncthreads();
    if (j0 + 64 < jend) fetch(j0 + 64);
    mma_64x64(s_c, s_q, w, l16, lk, acc);
  }
#pragma unroll
  for (int b = 0; b < 4; ++b)
    if (cb + 16 * b + l16 < d)
#pragma unroll
      for (int v = 0; v < 4; ++v) Wpart[((int64_t)js * PB + 16 * w + lk + 4 * v) * d + cb + 16 * b + l16] = acc[b][v];
}

// Takes the projection off the panel, W[r][c] -= sum_js Wpart[js][r][c] (fixed order; njs = 0: nothing to take off), and
// writes the partial Gram matrices: workgroup `chunk` covers GC columns and writes W_chunk W_chunk^T (PB x PB).
constexpr int GC = 64;
// out = T T^T (PB x PB) of a panel tile T of GC columns in LDS (row stride SK)
__device__ inline void gram_tile(const double *s_w, int w, int l16, int lk, double *out) {
  f64x4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
  for (int k = 0; k < GC; k += 4) {
    const double a = s_w[(16 * w + l16) * SK + k + lk];
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = mma_f64(a, s_w[(16 * b + l16) * SK + k + lk], acc[b]);
  }
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) out[(16 * w + lk + 4 * q) * PB + 16 * b + l16] = acc[b][q];
}
__global__ void __launch_bounds__(256) gram_partial_kernel(double *Q, int d, int p0, int nr, const double *Wpart, int njs,
                                                           double *part) {
  __shared__ double s_w[PB * SK];
  const int c0 = blockIdx.x * GC;
  const int t = threadIdx.x & 63, w = wave_id(), l16 = t & 15, lk = t >> 4;
  const bool cok = c0 + t < d;
  double v[16];   // rows 4 u + w of column c0 + t: the loads of all of them are in flight together
#pragma unroll
  for (int u = 0; u < 16; ++u) v[u] = (cok && 4 * u + w < nr) ? Q[(int64_t)(p0 + 4 * u + w) * d + c0 + t] : 0.0;
  const double live = cok ? 1.0 : 0.0;
#pragma unroll 2
  for (int js = 0; js < njs; ++js)   // (rows past nr are rows of zeros in Wpart)
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] -= live * Wpart[((int64_t)js * PB + 4 * u + w) * d + min(c0 + t, d - 1)];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    s_w[(4 * u + w) * SK + t] = v[u];
    if (njs > 0 && cok && 4 * u + w < nr) Q[(int64_t)(p0 + 4 * u + w) * d + c0 + t] = v[u];
  }
  __syncthreads();
  gram_tile(s_w, w, l16, lk, part + (int64_t)blockIdx.x * PB * PB);
}
static_assert(PB == 64 && GC == 64, "four wavefronts of 16 panel rows each");

__device__ inline double bcast_lane(double v, int src) {   // (src uniform)
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned int lo = __builtin_amdgcn_readlane((int)(unsigned int)u, src);
  const unsigned int hi = __builtin_amdgcn_readlane((int)(unsigned int)(u >> 32), src);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// 1 / sqrt(v) for v > 0 to fp64 rounding: the hardware's estimate and two Newton steps
__device__ inline double rsqrt_f64(double v) {
  double r = __builtin_amdgcn_rsq(v);
#pragma unroll
  for (int i = 0; i < 2; ++i) r = fma(0.5 * r, fma(-(v * r), r, 1.0), r);
  return r;
}

// Cholesky factor and its inverse of a 32 x 32 matrix inside one wavefront, both in one elimination: lanes 0 .. 31 hold the
// rows of the matrix, lanes 32 .. 63 the columns of the unit matrix, and a step does the same to all 64 of them (scale
// element k, take its multiple of column k of L off the elements behind it).  At the end lane 32 + t holds column t of
// L^-1 (v[i] = Linv[i][t]).
// One wavefront works alone here, and everything it waits for is run time of the whole panel.  Column k of L, an element a
// lane, is copied to all rows of 16 lanes (elements 0 .. 15 and 16 .. 31), and the multiply-adds take their element from
// there by the lane broadcast that is part of the instruction: through LDS, 30 ns to come back and 15 broadcast reads a
// column, the 64 columns of a panel took 15 us, now 7.5.  The chain of nine dependent operations to the next column's
// reciprocal root (which replaces a square root and all divisions) runs between them; its operands are broadcast before
// the column is scaled.  The empty asm statements keep the operations in the order written.
constexpr int HB = 32;
#define SKM_PIN(x) asm volatile("" : "+v"(x))
// v[j] -= l[j] c for j = J .. J + COUNT - 1, l[j] in lane j % 16 of every row of lo or hi.  (A lane broadcast reads its
// register two wait states after it was written at the earliest.)
template <int J, int COUNT>
__device__ inline void chol_behind(double (&v)[HB], double lo, double hi, double c) {
  if constexpr (COUNT > 0 && J < HB) {
    constexpr int n = (COUNT < 4 ? COUNT : 4) < HB - J ? (COUNT < 4 ? COUNT : 4) : HB - J;
    constexpr int j1 = n > 1 ? J + 1 : J, j2 = n > 2 ? J + 2 : J, j3 = n > 3 ? J + 3 : J;
    const double l0 = J < 16 ? lo : hi, l1 = j1 < 16 ? lo : hi, l2 = j2 < 16 ? lo : hi, l3 = j3 < 16 ? lo : hi;
#define SKM_FMAC(o, l, at) "v_fmac_f64_dpp " o ", -" l ", %[c] row_newbcast:" at " row_mask:0xf bank_mask:0xf\n"
    if constexpr (n == 1)
      asm volatile("s_nop 1\n" SKM_FMAC("%0", "%[l0]", "%[n0]") : "+v"(v[J]) : [l0] "v"(l0), [c] "v"(c), [n0] "n"(J % 16));
    else if constexpr (n == 2)
      asm volatile("s_nop 1\n" SKM_FMAC("%0", "%[l0]", "%[n0]") SKM_FMAC("%1", "%[l1]", "%[n1]")
                   : "+v"(v[J]), "+v"(v[j1]) : [l0] "v"(l0), [l1] "v"(l1), [c] "v"(c), [n0] "n"(J % 16), [n1] "n"(j1 % 16));
    else if constexpr (n == 3)
      asm volatile("s_nop 1\n" SKM_FMAC("%0", "%[l0]", "%[n0]") SKM_FMAC("%1", "%[l1]", "%[n1]") SKM_FMAC("%2", "%[l2]", "%[n2]")
                   : "+v"(v[J]), "+v"(v[j1]), "+v"(v[j2])
                   : [l0] "v"(l0), [l1] "v"(l1), [l2] "v"(l2), [c] "v"(c), [n0] "n"(J % 16), [n1] "n"(j1 % 16), [n2] "n"(j2 % 16));
    else
      asm volatile("s_nop 1\n" SKM_FMAC("%0", "%[l0]", "%[n0]") SKM_FMAC("%1", "%[l1]", "%[n1]") SKM_FMAC("%2", "%[l2]", "%[n2]")
                       SKM_FMAC("%3", "%[l3]", "%[n3]")
                   : "+v"(v[J]), "+v"(v[j1]), "+v"(v[j2]), "+v"(v[j3])
                   : [l0] "v"(l0), [l1] "v"(l1), [l2] "v"(l2), [l3] "v"(l3), [c] "v"(c), [n0] "n"(J % 16), [n1] "n"(j1 % 16),
                     [n2] "n"(j2 % 16), [n3] "n"(j3 % 16));
#undef SKM_FMAC
    chol_behind<J + n, COUNT - n>(v, lo, hi, c);
  }
}
// lo, hi: elements 0 .. 15 and 16 .. 31 of lanes 0 .. 31, in every row of 16 lanes
__device__ inline void copy_to_rows(double v, double &lo, double &hi) {
  const uint2 u = __builtin_bit_cast(uint2, v);
  uint2 a, b;
  const auto x0 = __builtin_amdgcn_permlane32_swap(u.x, u.x, false, false), x1 = __builtin_amdgcn_permlane32_swap(u.y, u.y, false, false);
  const auto y0 = __builtin_amdgcn_permlane16_swap(x0[0], x0[0], false, false), y1 = __builtin_amdgcn_permlane16_swap(x1[0], x1[0], false, false);
  a = make_uint2(y0[0], y1[0]);
  b = make_uint2(y0[1], y1[1]);
  lo = __builtin_bit_cast(double, a);
  hi = __builtin_bit_cast(double, b);
}
// column K; r: its reciprocal root; a, b: elements K and K + 1 of row K + 1
template <int K>
__device__ inline void chol_column(double (&v)[HB], double r, double a, double b) {
  v[K] *= r;   // column K of L (rows above K hold values nothing reads); row K of L^-1
  SKM_PIN(v[K]);
  if constexpr (K + 1 < HB) {
    constexpr int J = K + 3;
    double l1 = a * r;
    SKM_PIN(l1);
    double lo, hi;
    copy_to_rows(v[K], lo, hi);
    double dd = fma(-l1, l1, b);
    SKM_PIN(dd);
    double q = __builtin_amdgcn_rsq(dd);
    SKM_PIN(q);
    chol_behind<K + 1, 2>(v, lo, hi, v[K]);
    chol_behind<J, 1>(v, lo, hi, v[K]);
    double t = dd * q, h = 0.5 * q;
    SKM_PIN(t);
    SKM_PIN(h);
    chol_behind<J + 1, 4>(v, lo, hi, v[K]);
    double e = fma(-t, q, 1.0);
    SKM_PIN(e);
    if constexpr (K + 2 < HB) {
      a = bcast_lane(v[K + 1], K + 2);
      b = bcast_lane(v[K + 2], K + 2);
    }
    chol_behind<J + 5, 4>(v, lo, hi, v[K]);
    q = fma(h, e, q);
    SKM_PIN(q);
    chol_behind<J + 9, 4>(v, lo, hi, v[K]);
    t = dd * q;
    h = 0.5 * q;
    SKM_PIN(t);
    SKM_PIN(h);
    chol_behind<J + 13, 4>(v, lo, hi, v[K]);
    e = fma(-t, q, 1.0);
    SKM_PIN(e);
    chol_behind<J + 17, 4>(v, lo, hi, v[K]);
    q = fma(h, e, q);
    SKM_PIN(q);
    chol_behind<J + 21, 8>(v, lo, hi, v[K]);
    chol_column<K + 1>(v, q, a, b);
  }
}
__device__ inline void chol_inv32(double (&v)[HB]) {
  chol_column<0>(v, rsqrt_f64(bcast_lane(v[0], 0)), bcast_lane(v[0], 1), bcast_lane(v[1], 1));
}

// The partial Gram matrices added up in their order, one element a thread (entries above the diagonal are not read later, and
// not added).  Many partials are a chain of loads for whoever needs the sum: 12 us of a panel's factor at 24.
__global__ void __launch_bounds__(256) gram_sum_kernel(const double *part, int nchunks, double *out) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if ((e & (PB - 1)) > e / PB) return;
  double a = 0.0;
  for (int c0 = 0; c0 < nchunks; c0 += 24) {
    double p[24];
#pragma unroll
    for (int u = 0; u < 24; ++u) p[u] = part[(int64_t)min(c0 + u, nchunks - 1) * (PB * PB) + e];   // (all in flight together)
#pragma unroll
    for (int u = 0; u < 24; ++u)
      if (c0 + u < nchunks) a += p[u];
  }
  out[e] = a;
}

// Second half of a panel's Cholesky-QR.  Every workgroup takes the Cholesky factor of G = sum of the partials (fixed
// order) = [G11 G21^T; G21 G22] in blocks of 32, and its inverse:
//   L11 = chol(G11), X11 = L11^-1;  L21 = G21 X11^T;  L22 = chol(G22 - L21 L21^T), X22 = L22^-1;
//   L^-1 = [X11 0; -X22 L21 X11, X22],
// and multiplies its own tile of 64 columns, W <- L^-1 W, in place.  (The factor is the same chain of dependent steps
// whether one workgroup takes it or all of them do; done by all, nobody waits for another launch.)  Where the panel is
// factorised once more, the tile's part of the next Gram matrix follows (TC = GC columns a tile; part_next, another buffer:
// other workgroups may still read `part`).  Otherwise tiles are narrow (the fp64 products of 64 columns take 3 us, those of
// 16 columns one); R_out (optional) receives the panel rounded to fp32.
// The two 32 x 32 factorisations run in the registers of the first wavefront; the products use all four.
constexpr int kAreaDoubles = 64 * SR + 96;               // G, then L21; later the tile of W (row stride SR, then SK)
static_assert(PB * (PB + 1) + HB * (HB + 1) <= kAreaDoubles && PB * SK <= kAreaDoubles, "what shares the area");
constexpr size_t kFactorLds = sizeof(double) * (size_t)(kAreaDoubles + PB * SK);
template <int TC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) factor_apply_kernel(double *Q, int d, int p0, int nr, const double *part, int nchunks,
                                                           double *part_next, float *R_out) {
  extern __shared__ __align__(16) double s_mem[];
  double (*s_g)[PB + 1] = reinterpret_cast<double (*)[PB + 1]>(s_mem);   // G; its diagonal blocks become X11 and X22, its upper right block L21 X11
  double (*s_l21)[HB + 1] = reinterpret_cast<double (*)[HB + 1]>(s_mem + PB * (PB + 1));   // L21
  double *s_w = s_mem;                        // the tile of W, once G is not needed any more
  double *s_l = s_mem + kAreaDoubles;            // L^-1, row stride SK
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = wave_id(), l16 = lane & 15, lk = lane >> 4;
  const int c0 = blockIdx.x * TC;
  constexpr int VW = TC / 4, RW = 256 / TC;   // elements of the tile a thread, rows a step of the workgroup
  const int wcol = tid % TC, wrow = tid / TC;
  double vw[VW];   // rows RW u + wrow of the tile's column wcol: wanted only behind the factor
#pragma unroll
  for (int u = 0; u < VW; ++u) vw[u] = Q[(int64_t)(p0 + min(RW * u + wrow, nr - 1)) * d + min(c0 + wcol, d - 1)];
  {
    double a[16];   // element (4 u + w, lane) of G; nothing above the diagonal is read (those lanes repeat the diagonal)
#pragma unroll
    for (int u = 0; u < 16; ++u) a[u] = 0.0;
#pragma unroll 4
    for (int ch = 0; ch < nchunks; ++ch)   // fixed order; the loads of several chunks are in flight together
#pragma unroll
      for (int u = 0; u < 16; ++u) a[u] += part[(int64_t)ch * (PB * PB) + (4 * u + w) * PB + min(lane, 4 * u + w)];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      // rows past nr are padding: make them the identity so that the factorisation stays defined
      const int row = 4 * u + w, col = lane;
      s_g[row][col] = (row >= nr || col >= nr) ? ((row == col) ? 1.0 : 0.0) : a[u];
    }
  }
  __syncthreads();
  // block products: wavefront w holds a 16 x 16 quarter, rows rq .. + 15 and columns cq .. + 15, of the 32 x 32 result
  const int rq = 16 * (w >> 1), cq = 16 * (w & 1);
#pragma unroll 1
  for (int o = 0; o < PB; o += HB) {
    if (tid < 64) {   // the diagonal block at o: its factor's inverse takes its place
      const int t = lane & 31;
      double v[HB];
#pragma unroll
      for (int j = 0; j < HB; ++j) v[j] = s_g[o + t][o + j];
      if (lane >= HB)
#pragma unroll
        for (int j = 0; j < HB; ++j) v[j] = j == t ? 1.0 : 0.0;
      chol_inv32(v);
      if (lane >= HB)
#pragma unroll
        for (int i = 0; i < HB; ++i) s_g[o + i][o + t] = v[i];
    }
    if (o > 0) {   // (beside X22) L21 X11 into the unused upper right block
      f64x4 acc = {0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < HB; k += 4) acc = mma_f64(s_l21[rq + l16][k + lk], s_g[k + lk][cq + l16], acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) s_g[rq + lk + 4 * v][HB + cq + l16] = acc[v];
    }
    __syncthreads();
    if (o > 0) break;
    {   // L21 = G21 X11^T
      f64x4 acc = {0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < HB; k += 4) acc = mma_f64(s_g[HB + rq + l16][k + lk], s_g[cq + l16][k + lk], acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) s_l21[rq + lk + 4 * v][cq + l16] = acc[v];
    }
    __syncthreads();
    {   // G22 - L21 L21^T, in place
      f64x4 acc;
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = s_g[HB + rq + lk + 4 * v][HB + cq + l16];
#pragma unroll
      for (int k = 0; k < HB; k += 4) acc = mma_f64(-s_l21[rq + l16][k + lk], s_l21[cq + l16][k + lk], acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) s_g[HB + rq + lk + 4 * v][HB + cq + l16] = acc[v];
    }
    __syncthreads();
  }
  {   // L^-1 = [X11 0; -X22 (L21 X11), X22]
    f64x4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < HB; k += 4) acc = mma_f64(-s_g[HB + rq + l16][HB + k + lk], s_g[k + lk][HB + cq + l16], acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = rq + lk + 4 * v, col = cq + l16;
      s_l[(HB + row) * SK + col] = acc[v];
      s_l[row * SK + col] = s_g[row][col];
      s_l[row * SK + HB + col] = 0.0;
      s_l[(HB + row) * SK + HB + col] = s_g[HB + row][HB + col];
    }
  }
  __syncthreads();
  const bool cok = c0 + wcol < d;
#pragma unroll
  for (int u = 0; u < VW; ++u) s_w[(RW * u + wrow) * SR + wcol] = RW * u + wrow < nr && cok ? vw[u] : 0.0;
  __syncthreads();
  constexpr int NB = TC / 16;
  f64x4 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = f64x4{0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < PB; k += 4) {
    const double a = s_l[(16 * w + l16) * SK + k + lk];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = mma_f64(a, s_w[(k + lk) * SR + 16 * b + l16], acc[b]);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * w + lk + 4 * v, c = c0 + 16 * b + l16;
      if (r < nr && c < d) {
        Q[(int64_t)(p0 + r) * d + c] = acc[b][v];
        if (R_out) R_out[(int64_t)(p0 + r) * d + c] = (float)acc[b][v];
      }
    }
  if constexpr (TC == GC) {
    __syncthreads();   // (the tile's last readers)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * w + lk + 4 * v, c = 16 * b + l16;
        s_w[r * SK + c] = r < nr && c0 + c < d ? acc[b][v] : 0.0;
      }
    __syncthreads();
    gram_tile(s_w, w, l16, lk, part_next + (int64_t)blockIdx.x * PB * PB);
  }
}
static_assert(PB == 64 && HB * 2 == PB, "factor_apply_kernel: two blocks of 32");
}  // namespace

// Qwork: d*d + 2 doubles; Cwork: max(12 * 64 * d, (2 * ceil(d/64) + 1) * 64 * 64); Wwork: ceil(d/64) * 64 * d.
hipError_t launch_make_rotation(int32_t d, uint64_t seed, double *Qwork, double *Cwork, double *Wwork, float *R_out,
                                hipStream_t st) {
  struct Setup {   // (once per process: the kernel's LDS size)
    hipError_t rc;
    Setup() {
      rc = hipFuncSetAttribute(reinterpret_cast<const void *>(factor_apply_kernel<GC>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kFactorLds);
      if (rc == hipSuccess)
        rc = hipFuncSetAttribute(reinterpret_cast<const void *>(factor_apply_kernel<16>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)kFactorLds);
    }
  };
  static const Setup setup;
  if (setup.rc != hipSuccess) return setup.rc;
  const int64_t pairs = ((int64_t)d * d + 1) / 2;
  hipLaunchKernelGGL(gauss_fill_kernel, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, st, Qwork, pairs, seed);
  for (int p0 = 0; p0 < d; p0 += PB) {
    const int nr = d - p0 < PB ? d - p0 : PB;
    // The rows are Gaussian: what a panel keeps after the projection has norm sqrt((d - p0) / d) of what it had, so one
    // projection and one Cholesky-QR already leave errors near fp64 rounding while the complement is large.  In the
    // last 256 rows, where the complement gets small and the panel ill-conditioned (10^2 to 10^5 in the last one), both
    // steps are done twice.  The largest |Q Q^T - I| before rounding, median and maximum of 40 matrices: 7e-15 and 7e-14 at
    // d = 128, 5e-15 and 6e-14 at d = 384; with one projection everywhere and the second factorisation only where
    // d - p0 < 2 nr 4e-14 and 4e-13, 8e-14 and 1e-12.
    const int passes = d - p0 <= 256 ? 2 : 1;
    const int njs = p0 > 0 ? (p0 + JR - 1) / JR : 0;
    const int nchunks = (d + GC - 1) / GC;
    for (int pass = 0; p0 > 0 && pass < passes; ++pass) {
      if (pass > 0)   // takes the first projection off the panel (the Gram matrix of a panel that is projected again is not used)
        hipLaunchKernelGGL(gram_partial_kernel, dim3((unsigned)nchunks), dim3(256), 0, st, Qwork, d, p0, nr,
                           (const double *)Wwork, njs, Cwork);
      hipLaunchKernelGGL(coeff_kernel, dim3((unsigned)((p0 + 31) / 32), KS), dim3(256), 0, st, Qwork, d, p0, nr, Cwork);
      hipLaunchKernelGGL(apply_kernel, dim3((unsigned)((d + 63) / 64), (unsigned)njs), dim3(256), 0, st, Qwork, d, p0, nr,
                         Cwork, Wwork);
    }
    // the last projection off the panel, and its Gram matrix in parts
    hipLaunchKernelGGL(gram_partial_kernel, dim3((unsigned)nchunks), dim3(256), 0, st, Qwork, d, p0, nr,
                       (const double *)Wwork, njs, Cwork);
    // Several partials are added up by a kernel of their own.  The whole generator with 2, 4, 6, 8, 10 partials as the line (us):
    // d = 128 146, 131 and as that; d = 256 324, 319, 347 and as that; d = 384 450, 443, 447, 486; d = 512 563, 558, 561, 570,
    // 641; d = 1536 1622 each, 2077 without it.
    constexpr int kSumParts = 4;
    double *sum = Cwork + (int64_t)2 * nchunks * PB * PB;
    for (int pass = 0; pass < passes; ++pass) {
      const double *part = Cwork + (int64_t)pass * nchunks * PB * PB;
      int parts = nchunks;
      if (nchunks >= kSumParts) {
        hipLaunchKernelGGL(gram_sum_kernel, dim3(PB * PB / 256), dim3(256), 0, st, part, nchunks, sum);
        part = sum;
        parts = 1;
      }
      if (pass < passes - 1)
        hipLaunchKernelGGL(factor_apply_kernel<GC>, dim3((unsigned)nchunks), dim3(256), kFactorLds, st, Qwork, d, p0, nr, part,
                           parts, Cwork + (int64_t)nchunks * PB * PB, (float *)nullptr);
      else
        hipLaunchKernelGGL(factor_apply_kernel<16>, dim3((unsigned)((d + 15) / 16)), dim3(256), kFactorLds, st, Qwork, d, p0, nr,
                           part, parts, (double *)nullptr, R_out);
    }
  }
  return hipGetLastError();
}

}  // namespace skm
