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
constexpr int KS = 6;    // column splits of the coefficient product
constexpr int JR = 128;  // finished rows per workgroup of the update (the row range is split into ceil(p0 / JR) parts)
__global__ void __launch_bounds__(256) coeff_kernel(const double *Q, int d, int p0, int nr, double *Cpart) {
  __shared__ double s_w[PB * SK], s_q[32 * SK];
  const int j0 = blockIdx.x * 32, ks = blockIdx.y;
  const int kchunk = ((d + KS - 1) / KS + 63) / 64 * 64;
  const int kbeg = ks * kchunk, kend = min(d, kbeg + kchunk);
  const int lane = threadIdx.x & 63, w = wave_id(), l16 = lane & 15, lk = lane >> 4;
  f64x4 acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
  for (int c0 = kbeg; c0 < kend; c0 += 64) {
    double vw[16], vq[8];
    const int c = threadIdx.x & 63, cc = min(c0 + c, d - 1);
    const double live = c0 + c < kend ? 1.0 : 0.0;   // (loads unconditional at valid addresses; what lies outside counts as zero)
#pragma unroll
    for (int u = 0; u < 16; ++u) vw[u] = Q[(int64_t)min(p0 + 4 * u + w, p0 + nr - 1) * d + cc];
#pragma unroll
    for (int u = 0; u < 8; ++u) vq[u] = Q[(int64_t)min(j0 + 4 * u + w, p0 - 1) * d + cc];
#pragma unroll
    for (int u = 0; u < 16; ++u) vw[u] *= 4 * u + w < nr ? live : 0.0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; ++u) s_w[(4 * u + w) * SK + c] = vw[u];
#pragma unroll
    for (int u = 0; u < 8; ++u) s_q[(4 * u + w) * SK + c] = vq[u];
    __syncthreads();
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
__global__ void __launch_bounds__(256) apply_kernel(const double *Q, int d, int p0, int nr, const double *Cpart,
                                                    double *Wpart) {
  __shared__ double s_c[PB * SK], s_q[64 * SR];
  const int cb = blockIdx.x * 64, js = blockIdx.y;
  const int jbeg = js * JR, jend = min(p0, jbeg + JR);
  const int t = threadIdx.x & 63, w = wave_id(), l16 = t & 15, lk = t >> 4;
  f64x4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
  for (int j0 = jbeg; j0 < jend; j0 += 64) {
    double vc[16], vq[16];
    // (every load unconditional at a valid address, so that all of them are in flight together; what lies outside counts
    // as zero through C)
    const int jc = min(j0 + t, p0 - 1), cc = min(cb + t, d - 1);
    const double live = j0 + t < jend ? 1.0 : 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      vq[u] = Q[(int64_t)min(j0 + 4 * u + w, p0 - 1) * d + cc];
      vc[u] = 0.0;
    }
#pragma unroll 3
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int u = 0; u < 16; ++u) vc[u] += Cpart[((int64_t)ks * PB + 4 * u + w) * p0 + jc];
#pragma unroll
    for (int u = 0; u < 16; ++u) vc[u] *= live;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      s_q[(4 * u + w) * SR + t] = vq[u];
      s_c[(4 * u + w) * SK + t] = vc[u];
    }
    __syncthreads();
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
    for (int q = 0; q < 4; ++q) part[((int64_t)blockIdx.x * PB + 16 * w + lk + 4 * q) * PB + 16 * b + l16] = acc[b][q];
}
static_assert(PB == 64 && GC == 64, "four wavefronts of 16 panel rows each");

__device__ inline double bcast_lane(double v, int src) {   // src is a compile-time constant after unrolling
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

// Cholesky factor and its inverse of a 32 x 32 matrix inside one wavefront.  Lane t (and its mirror t + 32) holds row
// t of the matrix in g[].  On return x[] holds column t of L^-1 (x[i] = Linv[i][t]); g[] is used up.  One wavefront works
// alone here, and everything it waits for is run time of the whole panel: a finished column goes to LDS (s_l, column
// after column) and comes back as broadcast reads of two values, so the multiply-adds of a step are independent of each
// other (values broadcast through lane reads filled the scalar registers and were spilled), and a reciprocal square root
// per column replaces a square root and all divisions.
constexpr int HB = 32;
__device__ inline void chol_inv32(double (&g)[HB], double (&x)[HB], int t, double *s_l) {
  double r = rsqrt_f64(bcast_lane(g[0], 0));
#pragma unroll
  for (int k = 0; k < HB; ++k) {
    g[k] *= r;                              // column k of L (rows above k hold values nothing reads)
    s_l[k * HB + t] = t == k ? r : g[k];    // (the diagonal's place holds its reciprocal)
    __builtin_amdgcn_wave_barrier();
    if (k + 1 < HB) {   // the next column first: its reciprocal root is the longest chain of the step
      g[k + 1] = fma(-g[k], bcast_lane(g[k], k + 1), g[k + 1]);
      r = rsqrt_f64(bcast_lane(g[k + 1], k + 1));
    }
#pragma unroll
    for (int j = (k + 2) & ~1; j < HB; j += 2) {
      const double2 l = *reinterpret_cast<const double2 *>(s_l + k * HB + j);
      if (j > k + 1) g[j] = fma(-g[k], l.x, g[j]);
      g[j + 1] = fma(-g[k], l.y, g[j + 1]);
    }
  }
  // forward substitution: lane t builds column t of L^-1
#pragma unroll
  for (int i = 0; i < HB; ++i) x[i] = (i == t) ? 1.0 : 0.0;
#pragma unroll
  for (int m = 0; m < HB; ++m) {
    x[m] *= s_l[m * HB + m];
#pragma unroll
    for (int i = (m + 1) & ~1; i < HB; i += 2) {
      const double2 l = *reinterpret_cast<const double2 *>(s_l + m * HB + i);
      if (i > m) x[i] = fma(-l.x, x[m], x[i]);
      x[i + 1] = fma(-l.y, x[m], x[i + 1]);
    }
  }
}

// One workgroup: G = sum of the partials (fixed order) = [G11 G21^T; G21 G22] in blocks of 32, and the inverse of its
// Cholesky factor L = [L11 0; L21 L22] by blocks:
//   L11 = chol(G11), X11 = L11^-1;  L21 = G21 X11^T;  L22 = chol(G22 - L21 L21^T), X22 = L22^-1;
//   L^-1 = [X11 0; -X22 L21 X11, X22].
// The two 32 x 32 factorisations run in the registers of the first wavefront; the block products use all four.
__global__ void __launch_bounds__(256) chol_inv_kernel(const double *part, int nchunks, int nr, double *Linv_out) {
  __shared__ double s_g[PB][PB + 1];    // G; its diagonal blocks become X11 and X22, its upper right block L21 X11
  __shared__ double s_l21[HB][HB + 1];  // L21
  __shared__ __align__(16) double s_fac[HB * HB];   // columns of the factor in work
  const int tid = threadIdx.x;
  {
    double a[16];   // entries tid, tid + 256, ..
#pragma unroll
    for (int u = 0; u < 16; ++u) a[u] = 0.0;
#pragma unroll 4
    for (int ch = 0; ch < nchunks; ++ch)   // fixed order; the loads of several chunks are in flight together
#pragma unroll
      for (int u = 0; u < 16; ++u) a[u] += part[(int64_t)ch * (PB * PB) + 256 * u + tid];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      // rows past nr are padding: make them the identity so that the factorisation stays defined
      const int row = (256 * u + tid) / PB, col = tid % PB;
      s_g[row][col] = (row >= nr || col >= nr) ? ((row == col) ? 1.0 : 0.0) : a[u];
    }
  }
  __syncthreads();
  const int t = tid & 31;
  // block products: wavefront w holds a 16 x 16 quarter, rows rq .. + 15 and columns cq .. + 15, of the 32 x 32 result
  const int lane = tid & 63, w = wave_id(), l16 = lane & 15, lk = lane >> 4;
  const int rq = 16 * (w >> 1), cq = 16 * (w & 1);
  auto factor = [&](int o) {   // the diagonal block at o: its factor's inverse takes its place
    double g[HB], x[HB];
#pragma unroll
    for (int j = 0; j < HB; ++j) g[j] = s_g[o + t][o + j];
    chol_inv32(g, x, t, s_fac);
    if (tid < HB)
#pragma unroll
      for (int i = 0; i < HB; ++i) s_g[o + i][o + t] = x[i];
  };
  if (tid < 64) factor(0);   // X11
  __syncthreads();
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
  if (tid < 64) factor(HB);   // X22
  {   // meanwhile, by the other wavefronts too: L21 X11 into the unused upper right block
    f64x4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < HB; k += 4) acc = mma_f64(s_l21[rq + l16][k + lk], s_g[k + lk][cq + l16], acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) s_g[rq + lk + 4 * v][HB + cq + l16] = acc[v];
  }
  __syncthreads();
  {   // the result: [X11 0; -X22 (L21 X11), X22]
    f64x4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < HB; k += 4) acc = mma_f64(-s_g[HB + rq + l16][HB + k + lk], s_g[k + lk][HB + cq + l16], acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = rq + lk + 4 * v, col = cq + l16;
      Linv_out[(HB + row) * PB + col] = acc[v];
      Linv_out[row * PB + col] = s_g[row][col];
      Linv_out[row * PB + HB + col] = 0.0;
      Linv_out[(HB + row) * PB + HB + col] = s_g[HB + row][HB + col];
    }
  }
}
static_assert(PB == 64 && HB * 2 == PB, "chol_inv_kernel: two blocks of 32");

// W <- Linv W on a tile of 64 columns, in place (the tile is read into LDS first).
__global__ void __launch_bounds__(256) tri_apply_kernel(double *Q, int d, int p0, int nr, const double *Linv) {
  __shared__ double s_l[PB * SK], s_w[64 * SR];
  const int c0 = blockIdx.x * 64;
  const int t = threadIdx.x & 63, w = wave_id(), l16 = t & 15, lk = t >> 4;
  double vl[16], vw[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int r = 4 * u + w;
    vl[u] = Linv[r * PB + t];
    vw[u] = (r < nr && c0 + t < d) ? Q[(int64_t)(p0 + r) * d + c0 + t] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    s_l[(4 * u + w) * SK + t] = vl[u];
    s_w[(4 * u + w) * SR + t] = vw[u];
  }
  __syncthreads();
  f64x4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
  mma_64x64(s_l, s_w, w, l16, lk, acc);
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * w + lk + 4 * v, c = c0 + 16 * b + l16;
      if (r < nr && c < d) Q[(int64_t)(p0 + r) * d + c] = acc[b][v];
    }
}

__global__ void to_float_kernel(const double *Q, int64_t n, float *R) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) R[t] = (float)Q[t];
}
}  // namespace

// Qwork: d*d + 2 doubles; Cwork: max(12 * 64 * d, ceil(d/64) * 64 * 64); Wwork: ceil(d/64) * 64 * d; Lwork: 64 * 64.
hipError_t launch_make_rotation(int32_t d, uint64_t seed, double *Qwork, double *Cwork, double *Wwork, double *Lwork,
                                float *R_out, hipStream_t st) {
  const int64_t nel = (int64_t)d * d;
  const int64_t pairs = (nel + 1) / 2;
  hipLaunchKernelGGL(gauss_fill_kernel, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, st, Qwork, pairs, seed);
  for (int p0 = 0; p0 < d; p0 += PB) {
    const int nr = d - p0 < PB ? d - p0 : PB;
    // The rows are Gaussian: what a panel keeps after the projection has norm sqrt((d - p0) / d) of what it had, so one
    // projection and one Cholesky-QR already leave errors near fp64 rounding while the complement is large.  In the
    // last 256 rows, where the complement gets small and the panel ill-conditioned (10^2 to 10^5 in the last one), both
    // steps are done twice.  The largest |Q Q^T - I| before rounding, median and maximum of 40 matrices: 7e-15 and 7e-14 at
    // d = 128, 5e-15 and 6e-14 at d = 384; with one projection everywhere and the second factorisation only where
    // d - p0 < 2 nr 4e-14 and 4e-13, 8e-14 and 1e-12, for 116 instead of 165 us and 350 instead of 550.
    const int passes = d - p0 <= 256 ? 2 : 1;
    const int njs = p0 > 0 ? (p0 + JR - 1) / JR : 0;
    const int nchunks = (d + GC - 1) / GC;
    auto gram = [&](int take_off) {   // takes the last projection off the panel, then its Gram matrix in parts
      hipLaunchKernelGGL(gram_partial_kernel, dim3((unsigned)nchunks), dim3(256), 0, st, Qwork, d, p0, nr,
                         (const double *)Wwork, take_off, Cwork);
    };
    for (int pass = 0; p0 > 0 && pass < passes; ++pass) {
      if (pass > 0) gram(njs);   // (the Gram matrix of a panel that is projected again is not used)
      hipLaunchKernelGGL(coeff_kernel, dim3((unsigned)((p0 + 31) / 32), KS), dim3(256), 0, st, Qwork, d, p0, nr, Cwork);
      hipLaunchKernelGGL(apply_kernel, dim3((unsigned)((d + 63) / 64), (unsigned)njs), dim3(256), 0, st, Qwork, d, p0, nr,
                         Cwork, Wwork);
    }
    for (int pass = 0; pass < passes; ++pass) {
      gram(pass == 0 ? njs : 0);
      hipLaunchKernelGGL(chol_inv_kernel, dim3(1), dim3(256), 0, st, Cwork, nchunks, nr, Lwork);
      hipLaunchKernelGGL(tri_apply_kernel, dim3((unsigned)((d + 63) / 64)), dim3(256), 0, st, Qwork, d, p0, nr, Lwork);
    }
  }
  hipLaunchKernelGGL(to_float_kernel, dim3((unsigned)((nel + 255) / 256)), dim3(256), 0, st, Qwork, nel, R_out);
  return hipGetLastError();
}

}  // namespace skm
