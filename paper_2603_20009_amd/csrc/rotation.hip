// Random orthogonal matrix on the device (Algorithm 1, GenerateRandomRotationMatrix; Section 3.1).
//
// The rows of a d x d matrix of independent standard normals are orthonormalised by Gram-Schmidt, which
// gives a Haar-distributed orthogonal matrix.  Everything is fp64 (the result is rounded to fp32 at the
// end) and runs in panels of 64 rows (the chain of small dependent kernels per panel is what the run time is made of,
// so fewer, fatter panels are faster):
//   1. the panel is cleared of all finished rows (coefficients C = W Q^T, then W -= C Q);
//   2. the panel is orthonormalised in itself by Cholesky QR: G = W W^T = L L^T, W <- L^-1 W,
//      which is Gram-Schmidt inside the panel written as three dense steps.
// Both steps are done twice in the last 128 rows, where the complement of the finished rows gets small.  Up to 128 rows it is
// one kernel.
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
// Finished rows per workgroup of the update (the row range is split into ceil(p0 / JR) parts).  The whole generator with 64, 128, 192,
// 256 (us): d = 200 190, 211, 221, 220; d = 384 274, 302, 327, 349; d = 768 569, 617, 666, 721; d = 1536 1441, 1436, 1465, 1576.
constexpr int JR = 64;
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
// C[r][j] = sum_ks Cpart[ks][r][j], on a tile of 64 columns.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) apply_kernel(const double *Q, int d, int p0, int nr, const double *Cpart,
                                                    double *Wpart) {
  __shared__ double s_c[PB * SK], s_q[JR * SR];
  const int cb = blockIdx.x * 64, js = blockIdx.y, j0 = js * JR;
  const int t = threadIdx.x & 63, w = wave_id(), l16 = t & 15, lk = t >> 4;
  f64x4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
  double vc[KS][16], vq[16];
  // (every load unconditional at a valid address, so that all of them are in flight together; what lies outside counts
  // as zero through C)
  const int jc = min(j0 + t, p0 - 1), cc = min(cb + t, d - 1);
  const double live = j0 + t < p0 ? 1.0 : 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) vq[u] = Q[(int64_t)min(j0 + 4 * u + w, p0 - 1) * d + cc];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int u = 0; u < 16; ++u) vc[ks][u] = Cpart[((int64_t)ks * PB + 4 * u + w) * p0 + jc];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    double c = 0.0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) c += vc[ks][u];
    s_q[(4 * u + w) * SR + t] = vq[u];
    s_c[(4 * u + w) * SK + t] = c * live;
  }
  __syncthreads();
  mma_64x64(s_c, s_q, w, l16, lk, acc);
#pragma unroll
  for (int b = 0; b < 4; ++b)
    if (cb + 16 * b + l16 < d)
#pragma unroll
      for (int v = 0; v < 4; ++v) Wpart[((int64_t)js * PB + 16 * w + lk + 4 * v) * d + cb + 16 * b + l16] = acc[b][v];
}
static_assert(JR == 64, "apply_kernel: one round of 64 rows");

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
__device__ __forceinline__ void chol_behind(double (&v)[HB], double lo, double hi, double c) {
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
__device__ __forceinline__ void copy_to_rows(double v, double &lo, double &hi) {
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
__device__ __forceinline__ void chol_column(double (&v)[HB], double r, double a, double b) {
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
__device__ __forceinline__ void chol_inv32(double (&v)[HB]) {
  chol_column<0>(v, rsqrt_f64(bcast_lane(v[0], 0)), bcast_lane(v[0], 1), bcast_lane(v[1], 1));
}

// The Gram matrix of a panel that has been factorised once is next to the unit matrix, and the inverse of its factor needs no
// eliminations: I + E = L L^T with L = I + low(E) + O(|E|^2), low(E) = the part of E below the diagonal and half of its
// diagonal, so L^-1 W = W - low(E) W + O(|E|^2).  With no element of E beyond kNearUnit the norm of E is at most 64 of these,
// and its square below the rounding of the unit matrix; an element that is larger, in three to six of a
// hundred last panels of 64 rows (fp64 model of the step, 150 to 400 seeds each of d = 64, 128, 192), makes the panel take the eliminations.  Returns the element of -low(E) for element (r, c) of the Gram matrix; far: whether
// that is so.
constexpr double kNearUnit = 1.0 / (1ull << 33);
__device__ inline double minus_low(double g, int r, int c, bool &far) {
  const double e = r == c ? g - 1.0 : g;
  if (r >= c && !(fabs(e) <= kNearUnit)) far = true;
  return r > c ? -e : r == c ? -0.5 * e : 0.0;
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
// and multiplies its own tile of 16 columns, W <- L^-1 W, in place (the fp64 products of 64 columns take 3 us, those of 16
// columns one).  (The factor is the same chain of dependent steps whether one workgroup takes it or all of them do; done by all,
// nobody waits for another launch.)  R_out (optional) receives the panel rounded to fp32.
// NEAR: the panel has been factorised once, G is next to the unit matrix, and its factor's inverse is taken without the
// eliminations (they remain for a G that is not).
// The two 32 x 32 factorisations run in the registers of the first wavefront; the products use all four.
constexpr int kAreaDoubles = PB * SR + 96;               // G and L21; later the tile of W (row stride SR)
static_assert(PB * (PB + 1) + HB * (HB + 1) <= kAreaDoubles, "what shares the area");
constexpr size_t kFactorLds = sizeof(double) * (size_t)(kAreaDoubles + PB * SK);
template <bool NEAR>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) factor_apply_kernel(double *Q, int d, int p0, int nr, const double *part, int nchunks,
                                                           float *R_out) {
  extern __shared__ __align__(16) double s_mem[];
  double (*s_g)[PB + 1] = reinterpret_cast<double (*)[PB + 1]>(s_mem);   // G; its diagonal blocks become X11 and X22, its upper right block L21 X11
  double (*s_l21)[HB + 1] = reinterpret_cast<double (*)[HB + 1]>(s_mem + PB * (PB + 1));   // L21
  double *s_w = s_mem;                        // the tile of W, once G is not needed any more
  double *s_l = s_mem + kAreaDoubles;            // L^-1, row stride SK
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = wave_id(), l16 = lane & 15, lk = lane >> 4;
  constexpr int TC = 16;   // columns of the tile
  const int c0 = blockIdx.x * TC;
  constexpr int VW = TC / 4, RW = 256 / TC;   // elements of the tile a thread, rows a step of the workgroup
  const int wcol = tid % TC, wrow = tid / TC;
  double vw[VW];   // rows RW u + wrow of the tile's column wcol: wanted only behind the factor
#pragma unroll
  for (int u = 0; u < VW; ++u) vw[u] = Q[(int64_t)(p0 + min(RW * u + wrow, nr - 1)) * d + min(c0 + wcol, d - 1)];
  bool full = true;
  {
    double a[16];   // element (4 u + w, lane) of G; nothing above the diagonal is read (those lanes repeat the diagonal)
#pragma unroll
    for (int u = 0; u < 16; ++u) a[u] = 0.0;
#pragma unroll 4
    for (int ch = 0; ch < nchunks; ++ch)   // fixed order; the loads of several chunks are in flight together
#pragma unroll
      for (int u = 0; u < 16; ++u) a[u] += part[(int64_t)ch * (PB * PB) + (4 * u + w) * PB + min(lane, 4 * u + w)];
    // rows past nr are padding: make them the identity so that the factorisation stays defined
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (4 * u + w >= nr || lane >= nr) a[u] = 4 * u + w == lane ? 1.0 : 0.0;
    if constexpr (NEAR) {
      bool far = false;
#pragma unroll
      for (int u = 0; u < 16; ++u) s_l[(4 * u + w) * SK + lane] = minus_low(a[u], 4 * u + w, lane, far);
      full = __syncthreads_or(far) != 0;
    }
    if (full) {
#pragma unroll
      for (int u = 0; u < 16; ++u) s_g[4 * u + w][lane] = a[u];
    }
  }
  if (full) {
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
  }
  const bool cok = c0 + wcol < d;
#pragma unroll
  for (int u = 0; u < VW; ++u) s_w[(RW * u + wrow) * SR + wcol] = RW * u + wrow < nr && cok ? vw[u] : 0.0;
  __syncthreads();
  constexpr int NB = TC / 16;
  f64x4 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[b][v] = full ? 0.0 : s_w[(16 * w + lk + 4 * v) * SR + 16 * b + l16];
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
}
static_assert(PB == 64 && HB * 2 == PB, "factor_apply_kernel: two blocks of 32");
// The whole chain for up to 128 rows in one workgroup, the matrix in its LDS: two panels of 64 rows, each cleared of the
// finished rows and factorised twice, as above.  The chain of kernels waits for a launch and for its loads in each of its
// twelve kernels; here a step waits for a barrier, and what bounds it are the fp64 products on one CU (3.4 us for 64 x 64 x 128)
// and the two eliminations of a panel (4.2 us each).  The generator at d = 64 41 -> 30 us, at d = 128 113 -> 77.
constexpr int kSmallDim = 2 * PB, kSmallThreads = 512;
constexpr int SW = 130, SB = 34;   // LDS row strides (doubles) of the matrix and of the blocks of the factor
constexpr size_t kSmallLds = sizeof(double) * (size_t)(kSmallDim * SW + 3 * HB * SB);
__global__ void __launch_bounds__(kSmallThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) rotation_small_kernel(const double *G, int d, float *R_out) {
  extern __shared__ __align__(16) double s_mem[];
  double *s_w = s_mem;                      // [128][SW], zero past d
  double *s_b = s_mem + kSmallDim * SW;     // blocks (0, 0), (1, 0), (1, 1) of 32 x 32 of a panel's Gram matrix; later of L^-1
  double *s_b1 = s_b + HB * SB, *s_b2 = s_b + 2 * HB * SB;
  const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
  int l16 = lane & 15, lk = lane >> 4;
  const int kend = (d + 31) & ~31;
  auto at = [&](int r, int c) { return s_b + ((r >> 5) + (c >> 5)) * (HB * SB) + (r & 31) * SB + (c & 31); };   // r >= c / 32 * 32
  auto each_row = [&](double *row0) { return row0 + l16 * SW + lk; };   // this lane's place in 16 rows read along k
  {
    double v[2][kSmallDim / 8];   // (every load unconditional at a valid address, so that all of them are in flight together)
#pragma unroll
    for (int u = 0; u < kSmallDim / 8; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) v[h][u] = G[min(8 * u + w, d - 1) * d + min(64 * h + lane, d - 1)];
    const double live[2] = {lane < d ? 1.0 : 0.0, 64 + lane < d ? 1.0 : 0.0};
#pragma unroll
    for (int u = 0; u < kSmallDim / 8; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) s_w[(8 * u + w) * SW + 64 * h + lane] = v[h][u] * (8 * u + w < d ? live[h] : 0.0);
  }
  __syncthreads();
  for (int p0 = 0; p0 < d; p0 += PB) {
    const int nr = min(d - p0, PB);
    double *panel = s_w + p0 * SW;
    for (int pass = 0; pass < 2; ++pass) {
      asm volatile("" : "+v"(l16), "+v"(lk));   // (addresses are made where they are used: kept over the loops, they spill)
      if (p0 > 0) {
        // C = W Q^T, two blocks of 16 x 16 a wavefront; W -= C Q in two halves of the finished rows (the blocks' room holds 32 of 64)
        const int rb = w >> 1, ch = w & 1;
        f64x4 c[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
        const double *pa = each_row(panel + 16 * rb * SW), *pb = each_row(s_w + 32 * ch * SW);
        for (int k0 = 0; k0 < kend; k0 += 32)
#pragma unroll
          for (int k = k0; k < k0 + 32; k += 4)
#pragma unroll
            for (int b = 0; b < 2; ++b) c[b] = mma_f64(pa[k], pb[16 * b * SW + k], c[b]);
        f64x4 acc[4];   // columns 64 ch .. + 63 of row block rb
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[b][v] = panel[(16 * rb + lk + 4 * v) * SW + 64 * ch + 16 * b + l16];
        for (int h = 0; h < 2; ++h) {
          if (ch == h)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
              for (int v = 0; v < 4; ++v) s_b[(16 * rb + lk + 4 * v) * SB + 16 * b + l16] = -c[b][v];
          __syncthreads();
#pragma unroll
          for (int k = 0; k < 32; k += 4) {
            const double a = s_b[(16 * rb + l16) * SB + k + lk];
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[b] = mma_f64(a, s_w[(32 * h + k + lk) * SW + 64 * ch + 16 * b + l16], acc[b]);
          }
          __syncthreads();
        }
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int v = 0; v < 4; ++v) panel[(16 * rb + lk + 4 * v) * SW + 64 * ch + 16 * b + l16] = acc[b][v];
        __syncthreads();
      }
      asm volatile("" : "+v"(l16), "+v"(lk));
      // Gram matrix, its lower triangle in blocks of 16 x 16 (the blocks of 32 on the diagonal get both sides)
      bool far = pass == 0;
      f64x4 g[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};   // blocks w and (of wavefronts 0 and 1) 8 + w
      int rb[2], cb[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int i = w + 8 * u;
        rb[u] = i >= 6 ? 3 : i >= 3 ? 2 : i >= 1 ? 1 : 0;
        cb[u] = i - rb[u] * (rb[u] + 1) / 2;
      }
      const bool two = w < 2;
      const double *pa0 = each_row(panel + 16 * rb[0] * SW), *pb0 = each_row(panel + 16 * cb[0] * SW);
      const double *pa1 = each_row(panel + 16 * (two ? rb[1] : 0) * SW), *pb1 = each_row(panel + 16 * (two ? cb[1] : 0) * SW);
      for (int k0 = 0; k0 < kend; k0 += 32)
#pragma unroll
        for (int k = k0; k < k0 + 32; k += 4) {
          g[0] = mma_f64(pa0[k], pb0[k], g[0]);
          if (two) g[1] = mma_f64(pa1[k], pb1[k], g[1]);
        }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (u > 0 && !two) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {   // (rows past nr: the identity)
          const int r = 16 * rb[u] + lk + 4 * v, c = 16 * cb[u] + l16;
          if (r >= nr) g[u][v] = r == c ? 1.0 : 0.0;
          if (pass > 0) *at(r, c) = minus_low(g[u][v], r, c, far);
        }
      }
      const bool full = __syncthreads_or(far) != 0;
      if (full) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          if (u > 0 && !two) continue;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int r = 16 * rb[u] + lk + 4 * v, c = 16 * cb[u] + l16;
            *at(r, c) = g[u][v];
            if (rb[u] != cb[u] && rb[u] >> 1 == cb[u] >> 1) *at(c, r) = g[u][v];
          }
        }
        __syncthreads();
        asm volatile("" : "+v"(l16), "+v"(lk));
        const int t = lane & 31;
        auto factor = [&](double *blk) {   // one wavefront: its factor's inverse takes the place of a diagonal block
          double v[HB];
#pragma unroll
          for (int j = 0; j < HB; ++j) v[j] = blk[t * SB + j];
          if (lane >= HB)
#pragma unroll
            for (int j = 0; j < HB; ++j) v[j] = j == t ? 1.0 : 0.0;
          chol_inv32(v);
          if (lane >= HB)
#pragma unroll
            for (int i = 0; i < HB; ++i) blk[i * SB + t] = v[i];
        };
        // 32 x 32 products by four wavefronts, a quarter of 16 x 16 each
        const int rq = 16 * ((w >> 1) & 1), cq = 16 * (w & 1);
        f64x4 q = {0, 0, 0, 0};
        auto store = [&](double *blk) {
#pragma unroll
          for (int v = 0; v < 4; ++v) blk[(rq + lk + 4 * v) * SB + cq + l16] = q[v];
        };
#pragma unroll 1
        for (int o = 0;; ++o) {
          if (w == 0) {
            factor(o == 0 ? s_b : s_b2);
          } else if (o > 0 && w >= 4) {   // (beside it) L21 X11
            q = f64x4{0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < HB; k += 4) q = mma_f64(s_b1[(rq + l16) * SB + k + lk], s_b[(k + lk) * SB + cq + l16], q);
          }
          __syncthreads();
          if (o > 0) break;
          if (w < 4)   // L21 = G21 X11^T
#pragma unroll
            for (int k = 0; k < HB; k += 4) q = mma_f64(s_b1[(rq + l16) * SB + k + lk], s_b[(cq + l16) * SB + k + lk], q);
          __syncthreads();
          if (w < 4) store(s_b1);
          __syncthreads();
          if (w < 4) {   // G22 - L21 L21^T
#pragma unroll
            for (int v = 0; v < 4; ++v) q[v] = s_b2[(rq + lk + 4 * v) * SB + cq + l16];
#pragma unroll
            for (int k = 0; k < HB; k += 4) q = mma_f64(-s_b1[(rq + l16) * SB + k + lk], s_b1[(cq + l16) * SB + k + lk], q);
            store(s_b2);
          }
          __syncthreads();
        }
        if (w >= 4) store(s_b1);
        __syncthreads();
        if (w < 4) {   // -X22 (L21 X11)
          q = f64x4{0, 0, 0, 0};
#pragma unroll
          for (int k = 0; k < HB; k += 4) q = mma_f64(-s_b2[(rq + l16) * SB + k + lk], s_b1[(k + lk) * SB + cq + l16], q);
        }
        __syncthreads();
        if (w < 4) store(s_b1);
        __syncthreads();
      }
      asm volatile("" : "+v"(l16), "+v"(lk));
      // W <- L^-1 W, 16 columns a wavefront
      f64x4 x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int v = 0; v < 4; ++v) x[r][v] = full ? 0.0 : panel[(16 * r + lk + 4 * v) * SW + 16 * w + l16];
#pragma unroll
      for (int k = 0; k < PB; k += 4) {
        const double b = panel[(k + lk) * SW + 16 * w + l16];
#pragma unroll
        for (int r = k / 16; r < 4; ++r) x[r] = mma_f64(*at(16 * r + l16, k + lk), b, x[r]);
      }
      // (a wavefront reads and writes its own columns only)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int v = 0; v < 4; ++v) panel[(16 * r + lk + 4 * v) * SW + 16 * w + l16] = x[r][v];
      __syncthreads();
    }
  }
  for (int e = tid; e < d * d; e += kSmallThreads) {
    const int r = e / d;
    R_out[e] = (float)s_w[r * SW + (e - r * d)];
  }
}
static_assert(3 * HB >= PB && kSmallThreads == 512, "half of the coefficients in the room of the three blocks; eight wavefronts");
}  // namespace

// Qwork: d*d + 2 doubles; Cwork: rotation_cwork(d); Wwork: ceil(d/64) * 64 * d.
static_assert(KS == 6 && PB == 64 && GC == 64, "rotation_cwork");
hipError_t launch_make_rotation(int32_t d, uint64_t seed, double *Qwork, double *Cwork, double *Wwork, float *R_out,
                                hipStream_t st) {
  struct Setup {   // (once per process: the kernel's LDS size)
    hipError_t rc;
    Setup() {
      rc = hipFuncSetAttribute(reinterpret_cast<const void *>(factor_apply_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kFactorLds);
      if (rc == hipSuccess)
        rc = hipFuncSetAttribute(reinterpret_cast<const void *>(factor_apply_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)kFactorLds);
      if (rc == hipSuccess)
        rc = hipFuncSetAttribute(reinterpret_cast<const void *>(rotation_small_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)kSmallLds);
    }
  };
  static const Setup setup;
  if (setup.rc != hipSuccess) return setup.rc;
  const int64_t pairs = ((int64_t)d * d + 1) / 2;
  hipLaunchKernelGGL(gauss_fill_kernel, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, st, Qwork, pairs, seed);
  if (d <= kSmallDim) {
    hipLaunchKernelGGL(rotation_small_kernel, dim3(1), dim3(kSmallThreads), kSmallLds, st, (const double *)Qwork, d, R_out);
    return hipGetLastError();
  }
  for (int p0 = 0; p0 < d; p0 += PB) {
    const int nr = d - p0 < PB ? d - p0 : PB;
    // The rows are Gaussian: what a panel keeps after the projection has norm sqrt((d - p0) / d) of what it had, and while it
    // has more than twice as many dimensions as rows its condition is at most 6, so one projection and one Cholesky-QR leave
    // errors near fp64 rounding.  Behind that it gets up to 10^5, and both steps are done twice, the second projection behind
    // the first factor: what the factor's inverse has blown up of the first one's rounding goes with it.  The largest |Q Q^T - I|
    // before rounding, median and maximum of 60 matrices, and the time of the generator, all three forms with 128 rows a workgroup
    // of the update: this one d = 200 2e-15, 2e-15 and 208 us, 384 2e-15, 3e-15 and 301, 1536 4e-15, 5e-15 and 1433; with both projections
    // before both factorisations, in the last 256 rows, d = 200 1e-15, 9e-14 and 299 us, 384 5e-15, 8e-14 and 422, 1536 5e-15, 2e-13 and
    // 1593; in this order for the last 256 rows the same errors, 248, 366 and 1527.
    const int passes = d - p0 <= 2 * PB ? 2 : 1;
    const int njs = p0 > 0 ? (p0 + JR - 1) / JR : 0;
    const int nchunks = (d + GC - 1) / GC;
    for (int pass = 0; pass < passes; ++pass) {   // (the first panel, of more than 128 rows, has one)
      if (p0 > 0) {
        hipLaunchKernelGGL(coeff_kernel, dim3((unsigned)((p0 + 31) / 32), KS), dim3(256), 0, st, Qwork, d, p0, nr, Cwork);
        hipLaunchKernelGGL(apply_kernel, dim3((unsigned)((d + 63) / 64), (unsigned)njs), dim3(256), 0, st, Qwork, d, p0, nr,
                           Cwork, Wwork);
      }
      // the projection off the panel, and its Gram matrix in parts
      hipLaunchKernelGGL(gram_partial_kernel, dim3((unsigned)nchunks), dim3(256), 0, st, Qwork, d, p0, nr,
                         (const double *)Wwork, njs, Cwork);
      // Several partials are added up by a kernel of their own.  The whole generator with 4, 6, 8, 10 partials as the line (us), when
      // it did both steps twice in the last 256 rows: d = 256 319, 347 and as that; d = 384 443, 447, 486; d = 512 558, 561, 570,
      // 641; d = 1536 1622 each, 2077 without it.
      constexpr int kSumParts = 4;
      const double *part = Cwork;
      int parts = nchunks;
      if (nchunks >= kSumParts) {
        double *sum = Cwork + (int64_t)nchunks * PB * PB;
        hipLaunchKernelGGL(gram_sum_kernel, dim3(PB * PB / 256), dim3(256), 0, st, part, nchunks, sum);
        part = sum;
        parts = 1;
      }
      const dim3 grid((unsigned)((d + 15) / 16));
      float *out = pass < passes - 1 ? nullptr : R_out;
      if (pass == 0) hipLaunchKernelGGL(factor_apply_kernel<false>, grid, dim3(256), kFactorLds, st, Qwork, d, p0, nr, part, parts, out);
      else hipLaunchKernelGGL(factor_apply_kernel<true>, grid, dim3(256), kFactorLds, st, Qwork, d, p0, nr, part, parts, out);
    }
  }
  return hipGetLastError();
}

}  // namespace skm
