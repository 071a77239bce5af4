// Selection kernels for Early Termination by Recall (Section 3.3): exact top-K ground truth of the
// queries over the points, and the recall of an IVF search that probes the nearest centroids.
// The score matrices come from the MFMA GEMM; these kernels only select.
#include "skm_internal.h"

#include <algorithm>

namespace skm {

__device__ inline unsigned long long block_min_u64(unsigned long long v, unsigned long long *red) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    const unsigned long long o = __shfl_xor(v, m, 64);
    v = o < v ? o : v;
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  unsigned long long r = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = red[w] < r ? red[w] : r;
  return r;
}

// Keys are (order-preserving distance bits << 32 | index); the running list of each query and the new
// score row are treated as one candidate set, from which the K smallest keys are drawn one at a time
// (each round takes the smallest key above the previous one: ties resolve to the lowest index).
// Once the running list is full, a column can only enter it with a key below the list's largest: one pass over the
// row collects those columns in LDS (after the first chunks there are few) and the K rounds run over them instead of
// over the whole row; a row with more candidates than the buffer holds falls back to rounds over the row.
constexpr int TOPK_CAND = 4096;
__global__ void __launch_bounds__(256) topk_merge_kernel(const float *S, int64_t lds, int32_t m, int64_t col_base,
                                                         const float *colnorm, int32_t K, unsigned long long *top) {
  __shared__ unsigned long long red[4];
  __shared__ unsigned long long s_new[256];
  __shared__ unsigned long long s_cand[TOPK_CAND];
  __shared__ unsigned int s_ncand;
  const int q = blockIdx.x;
  const float *row = S + (int64_t)q * lds;
  unsigned long long *mine = top + (int64_t)q * K;
  auto key_of = [&](int c) {
    const float v = colnorm[col_base + c] - 2.f * row[c];
    return ((unsigned long long)f2ord(v) << 32) | (unsigned long long)(uint32_t)(col_base + c);
  };
  const unsigned long long kth = mine[K - 1];   // ~0 while the list is not full: then every column is a candidate
  if (threadIdx.x == 0) s_ncand = 0u;
  __syncthreads();
  bool filtered = false;
  if (kth != ~0ull) {
    for (int c = threadIdx.x; c < m; c += 256) {
      const unsigned long long key = key_of(c);
      if (key < kth) {
        const unsigned int pos = atomicAdd(&s_ncand, 1u);
        if (pos < (unsigned int)TOPK_CAND) s_cand[pos] = key;
      }
    }
    __syncthreads();
    filtered = s_ncand <= (unsigned int)TOPK_CAND;
  }
  const int ncand = filtered ? (int)s_ncand : m;
  unsigned long long last = 0ull;
  bool first = true;
  for (int r = 0; r < K; ++r) {
    unsigned long long best = ~0ull;
    for (int c = threadIdx.x; c < ncand; c += 256) {
      const unsigned long long key = filtered ? s_cand[c] : key_of(c);
      if ((first || key > last) && key < best) best = key;
    }
    if ((int)threadIdx.x < K) {
      const unsigned long long key = mine[threadIdx.x];
      if ((first || key > last) && key < best) best = key;
    }
    best = block_min_u64(best, red);
    if (threadIdx.x == 0) s_new[r] = best;
    last = best;
    first = false;
    if (best == ~0ull) {
      for (int rr = r + 1; rr < K; ++rr)
        if (threadIdx.x == 0) s_new[rr] = ~0ull;
      break;
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < K) mine[threadIdx.x] = s_new[threadIdx.x];
}

hipError_t launch_topk_merge(const float *S, int64_t lds, int32_t nq, int32_t m, int64_t col_base,
                             const float *colnorm, int32_t K, unsigned long long *top, hipStream_t st) {
  if (K > 256 || K < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(topk_merge_kernel, dim3(nq), dim3(256), 0, st, S, lds, m, col_base, colnorm, K, top);
  return hipGetLastError();
}

// One workgroup per query.  S[q][c] = q . y_c; the centroid order by distance is the order of
// ynorm[c] - 2 S[q][c].  The nprobe nearest centroids are drawn one at a time into LDS, then every
// ground-truth neighbour is looked up: it is retrieved iff its cluster is probed.
constexpr int MAX_PROBE = kMaxProbe;
// NK > 0: at most 256 NK centroids, whose keys every thread keeps in registers over the rounds of the selection (read again in
// every round, 1000 queries against 4096 centroids took 173 us, forty rounds of dependent loads).
template <int NK>
__global__ void __launch_bounds__(256) recall_kernel(const float *S, int64_t lds, int32_t k, const float *ynorm,
                                                     int32_t nprobe, const unsigned long long *gt_keys, int32_t K,
                                                     const int32_t *assign, unsigned long long *hits,
                                                     unsigned long long *total) {
  __shared__ unsigned long long red[4];
  __shared__ int32_t s_probe[MAX_PROBE];
  __shared__ unsigned int s_hits, s_total;
  const int q = blockIdx.x;
  const float *row = S + (int64_t)q * lds;
  if (threadIdx.x == 0) { s_hits = 0; s_total = 0; }
  unsigned long long last = 0ull;
  auto key_of = [&](int c) {
    return ((unsigned long long)f2ord(ynorm[c] - 2.f * row[c]) << 32) | (unsigned long long)(uint32_t)c;
  };
  unsigned long long keys[NK > 0 ? NK : 1];
#pragma unroll
  for (int u = 0; u < NK; ++u) keys[u] = (int)threadIdx.x + 256 * u < k ? key_of((int)threadIdx.x + 256 * u) : ~0ull;
  for (int r = 0; r < nprobe; ++r) {
    unsigned long long best = ~0ull;
    if constexpr (NK > 0) {
#pragma unroll
      for (int u = 0; u < NK; ++u)
        if ((r == 0 || keys[u] > last) && keys[u] < best) best = keys[u];
    } else {
      for (int c = threadIdx.x; c < k; c += 256) {
        const unsigned long long key = key_of(c);
        if ((r == 0 || key > last) && key < best) best = key;
      }
    }
    best = block_min_u64(best, red);
    if (threadIdx.x == 0) s_probe[r] = (int32_t)(best & 0xffffffffull);
    last = best;
  }
  __syncthreads();
  for (int g = 0; g < K; ++g) {
    const unsigned long long key = gt_keys[(int64_t)q * K + g];
    if (key == ~0ull) continue;
    const int32_t cl = assign[(int64_t)(key & 0xffffffffull)];
    bool found = false;
    for (int s = threadIdx.x; s < nprobe; s += 256) found |= (s_probe[s] == cl);
    if (__any(found) && (threadIdx.x & 63) == 0) atomicAdd(&s_hits, 1u);   // a cluster appears once in the list
    if (threadIdx.x == 0) s_total += 1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    atomicAdd(hits, (unsigned long long)s_hits);
    atomicAdd(total, (unsigned long long)s_total);
  }
}

hipError_t launch_recall_scores(const float *S, int64_t lds, int32_t nq, int32_t k, const float *ynorm, int32_t nprobe,
                                const unsigned long long *gt_keys, int32_t K, const int32_t *assign,
                                unsigned long long *hits, unsigned long long *total, hipStream_t st) {
  if (nprobe > MAX_PROBE || nprobe < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k <= 256 ? recall_kernel<1> : k <= 1024 ? recall_kernel<4> : k <= 4096 ? recall_kernel<16> : recall_kernel<0>,
                     dim3(nq), dim3(256), 0, st, S, lds, k, ynorm, nprobe, gt_keys, K, assign, hits,
                     total);
  return hipGetLastError();
}

// ---------------------------------------------------------------- ground truth through a one-product multiply
// The K nearest points of a query need exact scores only near the K-th smallest: the score matrix of all pairs, in full
// arithmetic and through memory, was nine tenths of the time (1000 queries over 1M x 768: 10.1 ms, of it 5.7 ms of
// three-product multiply, 4.2 GB of scores written and read again, 1.4 ms for two passes that bound and norm the rows).
// Here
//   1. a sample of the points, spread evenly, is multiplied in one fp16 product; the K-th smallest of the minima over groups
//      of 64 points is an upper bound of the K-th smallest score (K different points have scores at or below it), up to
//      the error of a one-product score;
//   2. all points are multiplied the same way, in chunks whose fp16 copy stays in the Infinity Cache; a pair whose score
//      is within twice the error bound of that threshold becomes a candidate (K n / sample and a few per query);
//   3. of a query's candidates, those within twice the bound of their own K-th smallest score get their exact distance
//      (direct form, fp32), and the K smallest (distance, index) are the result.
// Error bound: a row is scaled by the power of two that brings its largest value into [2^14, 2^15) and rounded to fp16, a
// relative error of 2^-11 per value (absolute 2^-25 below 2^-14), so q.x is off by at most (2^-10 + 2^-22) ||q|| ||x|| plus
// d 2^-38 max|q| max|x| (Cauchy-Schwarz), taken 10 % larger for the fp32 accumulation; the score by twice that.  The
// largest norm stands for ||x||.  A list that runs over its capacity makes the caller take the full path instead.
__device__ inline float gt_band(float qnorm2, float maxnorm2, int d) {
  const float q = sqrtf(fmaxf(qnorm2, 0.f)), x = sqrtf(fmaxf(maxnorm2, 0.f));
  return (2.f * 1.1f / 1024.f + (float)d * (1.f / 68719476736.f)) * q * x + (1e-6f + 1e-9f * (float)d) * (maxnorm2 + 2.f * q * x);
}

// one wavefront per row; NV > 0: the row in registers (ds <= 256 NV), 0: two passes over it
template <int NV, bool ALIGNED>
__global__ void __launch_bounds__(256) gt_convert_kernel(const float *X, int64_t ldx, int64_t n, int64_t nsel, int64_t row0,
                                                         int64_t rows, int32_t d, int32_t ds, uint32_t *plane, float *scale,
                                                         float *term, unsigned int *maxnorm) {
  __shared__ float s_m[4];
  const int lane = threadIdx.x & 63;
  float most = 0.f;
  auto load = [&](const float *x, int c) {
    if (!ALIGNED) return load4_any(x + c, d - c);
    return c < d ? *reinterpret_cast<const float4 *>(x + c) : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  auto emit = [&](uint32_t *dst, int c, const float4 &v, float sc) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t p0 = {v.x * sc, v.y * sc}, p1 = {v.z * sc, v.w * sc};
    *reinterpret_cast<uint2 *>(dst + 32 * (c / 32) + (c % 32) / 2) =
        make_uint2(__builtin_bit_cast(unsigned int, __builtin_convertvector(p0, f16x2_t)),
                   __builtin_bit_cast(unsigned int, __builtin_convertvector(p1, f16x2_t)));
  };
  for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < rows; i += (int64_t)gridDim.x * 4) {
    const int64_t src = nsel == n ? row0 + i : (int64_t)(((double)(row0 + i) + 0.5) * ((double)n / (double)nsel));
    const float *x = X + (src < n ? src : n - 1) * ldx;
    float4 v[NV > 0 ? NV : 1];
    float s = 0.f, m = 0.f;
    auto take = [&](const float4 &w) {
      s = fmaf(w.x, w.x, fmaf(w.y, w.y, fmaf(w.z, w.z, fmaf(w.w, w.w, s))));
      m = fmaxf(m, fmaxf(fmaxf(fabsf(w.x), fabsf(w.y)), fmaxf(fabsf(w.z), fabsf(w.w))));
    };
    if (NV > 0) {
#pragma unroll
      for (int u = 0; u < NV; ++u) v[u] = load(x, 256 * u + 4 * lane);
#pragma unroll
      for (int u = 0; u < NV; ++u) take(v[u]);
    } else {
      for (int c = 4 * lane; c < ds; c += 256) take(load(x, c));
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      s += __shfl_xor(s, o, 64);
      m = fmaxf(m, __shfl_xor(m, o, 64));
    }
    const float sc = m > 0.f ? split_scale(__builtin_bit_cast(unsigned int, m)) : 1.f;
    uint32_t *dst = plane + split_row(i, ds / 2);
    if (NV > 0) {
#pragma unroll
      for (int u = 0; u < NV; ++u)
        if (256 * u + 4 * lane < ds) emit(dst, 256 * u + 4 * lane, v[u], sc);
    } else {
      for (int c = 4 * lane; c < ds; c += 256) emit(dst, c, load(x, c), sc);
    }
    if (lane == 0) {
      scale[i] = sc;
      term[i] = 0.5f * s * sc;
    }
    most = fmaxf(most, s);
  }
  if (lane == 0) s_m[threadIdx.x >> 6] = most;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned int b = __builtin_bit_cast(unsigned int, fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3])));
    if (b > __atomic_load_n(maxnorm, __ATOMIC_RELAXED)) atomicMax(maxnorm, b);
  }
}

hipError_t launch_gt_convert(const float *X, int64_t ldx, int64_t n, int64_t nsel, int64_t row0, int64_t rows, int32_t d,
                             int32_t ds, uint32_t *plane, float *scale, float *term, unsigned int *maxnorm, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (ds % 32 != 0 || ds < d) return hipErrorInvalidValue;
  const bool al = (reinterpret_cast<uintptr_t>(X) & 15u) == 0 && ldx % 4 == 0 && d % 4 == 0;
  const int64_t blocks = std::min<int64_t>((rows + 3) / 4, 256 * 32);
#define SKM_GT_CONVERT(NV)                                                                                                 \
  do {                                                                                                                     \
    if (al) hipLaunchKernelGGL((gt_convert_kernel<NV, true>), dim3((unsigned)blocks), dim3(256), 0, st, X, ldx, n, nsel,    \
                               row0, rows, d, ds, plane, scale, term, maxnorm);                                            \
    else hipLaunchKernelGGL((gt_convert_kernel<NV, false>), dim3((unsigned)blocks), dim3(256), 0, st, X, ldx, n, nsel, row0, \
                            rows, d, ds, plane, scale, term, maxnorm);                                                     \
  } while (0)
  if (ds <= 256) SKM_GT_CONVERT(1);
  else if (ds <= 512) SKM_GT_CONVERT(2);
  else if (ds <= 768) SKM_GT_CONVERT(3);
  else if (ds <= 1024) SKM_GT_CONVERT(4);
  else if (ds <= 1536) SKM_GT_CONVERT(6);
  else if (ds <= 2048) SKM_GT_CONVERT(8);
  else SKM_GT_CONVERT(0);
#undef SKM_GT_CONVERT
  return hipGetLastError();
}

// ascending bitonic sort of N (a power of two) items in LDS by all threads of the workgroup
template <typename T>
__device__ inline void lds_sort(T *s, int n) {
  for (int k = 2; k <= n; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      __syncthreads();
      for (int t = threadIdx.x; t < n / 2; t += blockDim.x) {
        const int i = 2 * t - (t & (j - 1)), p = i + j;   // the t-th pair at distance j
        const T a = s[i], b = s[p];
        if ((a > b) == ((i & k) == 0)) {
          s[i] = b;
          s[p] = a;
        }
      }
    }
  __syncthreads();
}

__global__ void __launch_bounds__(256) gt_threshold_kernel(const float *group_min, int32_t ngroups, int32_t np2, int32_t K,
                                                           const float *q_scale, const float *q_term,
                                                           const unsigned int *maxnorm, int32_t d, float *tq) {
  extern __shared__ float s_g[];
  const int q = blockIdx.x;
  for (int t = threadIdx.x; t < np2; t += 256) s_g[t] = t < ngroups ? group_min[(int64_t)q * ngroups + t] : 3.4e38f;
  lds_sort(s_g, np2);
  if (threadIdx.x == 0)
    tq[q] = s_g[K - 1] + gt_band(2.f * q_term[q] / q_scale[q], __builtin_bit_cast(float, *maxnorm), d);
}
hipError_t launch_gt_threshold(const float *group_min, int32_t ngroups, int32_t nq, int32_t K, const float *q_scale,
                               const float *q_term, const unsigned int *maxnorm, int32_t d, float *tq, hipStream_t st) {
  if (K < 1 || K > ngroups || ngroups > kGtMaxGroups) return hipErrorInvalidValue;
  static const hipError_t attr_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(gt_threshold_kernel),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, kGtMaxGroups * 4);
  if (attr_rc != hipSuccess) return attr_rc;
  int np2 = 2;
  while (np2 < ngroups) np2 <<= 1;
  hipLaunchKernelGGL(gt_threshold_kernel, dim3((unsigned)nq), dim3(256), (size_t)np2 * sizeof(float), st, group_min, ngroups, np2,
                     K, q_scale, q_term, maxnorm, d, tq);
  return hipGetLastError();
}

__global__ void gt_terms_kernel(const float *tq, const float *q_scale, const float *q_term, int32_t nq,
                                const unsigned int *maxnorm, int32_t d, float *row_term) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nq) return;
  const float band = gt_band(2.f * q_term[q] / q_scale[q], __builtin_bit_cast(float, *maxnorm), d);
  row_term[q] = -0.5f * (tq[q] + band) * q_scale[q];
}
hipError_t launch_gt_terms(const float *tq, const float *q_scale, const float *q_term, int32_t nq, const unsigned int *maxnorm,
                           int32_t d, float *row_term, hipStream_t st) {
  hipLaunchKernelGGL(gt_terms_kernel, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, st, tq, q_scale, q_term, nq, maxnorm, d,
                     row_term);
  return hipGetLastError();
}

// One workgroup per query.  The candidates are ordered by their one-product score; those within twice the bound of the
// K-th get their exact distance, a wavefront each, and are ordered by (distance, index).
__global__ void __launch_bounds__(256) gt_select_kernel(const unsigned long long *cand, const unsigned int *count, unsigned int cap,
                                                        int32_t K, const float *X, int64_t ldx, const float *Q, int32_t d,
                                                        const float *q_scale, const float *q_term, const unsigned int *maxnorm,
                                                        unsigned long long *keys, volatile unsigned int *overflow) {
  extern __shared__ unsigned long long s_k[];
  __shared__ int s_m;
  const int q = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned int total = count[q];
  if (total > cap || (int)total < K) {   // (fewer than K: only where a score is not finite)
    if (threadIdx.x == 0) *overflow = 1u;
    return;
  }
  int np2 = 2;
  while (np2 < (int)total) np2 <<= 1;
  for (int t = threadIdx.x; t < np2; t += 256) s_k[t] = t < (int)total ? cand[(int64_t)q * cap + t] : ~0ull;
  if (threadIdx.x == 0) s_m = 0;
  lds_sort(s_k, np2);
  const float band = gt_band(2.f * q_term[q] / q_scale[q], __builtin_bit_cast(float, *maxnorm), d);
  const unsigned long long lim =
      ((unsigned long long)f2ord(ord2f((unsigned int)(s_k[K - 1] >> 32)) + 2.f * band) << 32) | 0xffffffffull;
  for (int t = threadIdx.x; t < (int)total; t += 256)
    if (s_k[t] <= lim && (t + 1 == (int)total || s_k[t + 1] > lim)) s_m = t + 1;   // (sorted: one thread finds the end)
  __syncthreads();
  const int m = s_m;
  const float *qr = Q + (int64_t)q * d;
  for (int t = wave; t < m; t += 4) {
    const unsigned int id = (unsigned int)(s_k[t] & 0xffffffffull);
    const float *x = X + (int64_t)id * ldx;
    float s = 0.f;
    for (int c = lane; c < d; c += 64) {
      const float df = x[c] - qr[c];
      s = fmaf(df, df, s);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) s_k[t] = ((unsigned long long)f2ord(s) << 32) | id;
  }
  __syncthreads();
  int mp2 = 2;
  while (mp2 < m) mp2 <<= 1;
  for (int t = m + threadIdx.x; t < mp2; t += 256) s_k[t] = ~0ull;
  lds_sort(s_k, mp2);
  for (int t = threadIdx.x; t < K; t += 256) keys[(int64_t)q * K + t] = t < m ? s_k[t] : ~0ull;
}
hipError_t launch_gt_select(const unsigned long long *cand, const unsigned int *count, unsigned int cap, int32_t nq, int32_t K,
                            const float *X, int64_t ldx, const float *Q, int32_t d, const float *q_scale, const float *q_term,
                            const unsigned int *maxnorm, unsigned long long *keys, unsigned int *overflow, hipStream_t st) {
  if (cap > kGtMaxCand || (cap & (cap - 1)) != 0 || cap < 2) return hipErrorInvalidValue;
  static const hipError_t attr_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(gt_select_kernel),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGtMaxCand * 8);
  if (attr_rc != hipSuccess) return attr_rc;
  hipLaunchKernelGGL(gt_select_kernel, dim3((unsigned)nq), dim3(256), (size_t)cap * 8, st, cand, count, cap, K, X, ldx, Q, d,
                     q_scale, q_term, maxnorm, keys, overflow);
  return hipGetLastError();
}

// ||row||^2 for n rows of length d (any alignment): one wavefront per row.
__global__ void __launch_bounds__(256) row_norms_kernel(const float *X, int64_t ldx, int64_t n, int32_t d, float *out) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * 4;
  for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += nw) {
    const float *x = X + i * ldx;
    float s = 0.f;
    for (int j = lane; j < d; j += 64) s = fmaf(x[j], x[j], s);
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) s += __shfl_xor(s, m, 64);
    if (lane == 0) out[i] = s;
  }
}
hipError_t launch_row_norms(const float *X, int64_t ldx, int64_t n, int32_t d, float *out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 3) / 4;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(row_norms_kernel, dim3((unsigned)blocks), dim3(256), 0, st, X, ldx, n, d, out);
  return hipGetLastError();
}

// keys (distance bits << 32 | index) -> int64 indices, -1 for missing
__global__ void keys_to_index_kernel(const unsigned long long *keys, int64_t n, int64_t *idx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) idx[i] = keys[i] == ~0ull ? -1 : (int64_t)(keys[i] & 0xffffffffull);
}
__global__ void index_to_keys_kernel(const int64_t *idx, int64_t n, unsigned long long *keys) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) keys[i] = idx[i] < 0 ? ~0ull : (unsigned long long)idx[i];
}
hipError_t launch_keys_to_index(const unsigned long long *keys, int64_t n, int64_t *idx, hipStream_t st) {
  hipLaunchKernelGGL(keys_to_index_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, keys, n, idx);
  return hipGetLastError();
}
hipError_t launch_index_to_keys(const int64_t *idx, int64_t n, unsigned long long *keys, hipStream_t st) {
  hipLaunchKernelGGL(index_to_keys_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, idx, n, keys);
  return hipGetLastError();
}

}  // namespace skm
