// PRUNING phase (Algorithm 1, loop over PDX blocks; Section 3.4 "Progressive Pruning").
//
// Input is the list of (point, centroid) pairs that passed the first test.  A pair is owned by a
// group of 8 lanes: one 64-dimension block of the point (256 contiguous bytes of the rotated row)
// and of the centroid (256 contiguous bytes of the block-major centroid copy) is two float4 per
// lane, taken so that each load instruction moves a full 128-byte line per pair.  After each
// block the group adds the block's squared distance, compares with theta(t, tau) and either drops
// the pair, goes on to the next block, or - at t = d - offers the finished distance to the point's
// packed (distance, centroid) minimum.  A group that is done with a pair takes the next one of its
// stride at once (its list entry was requested one pair earlier), so lanes do not idle while other
// groups of the wavefront are still busy.  The kernel is bound by memory latency times the number
// of pairs in flight: eight pairs per wavefront instead of four took a steady step of the 1M x 1536, k = 1024
// workload from 1.38 to 1.24 ms.
#include "skm_internal.h"

#include <algorithm>

namespace skm {

// Sum over 8 consecutive lanes; every lane receives the same bits (symmetric butterfly: swap within
// pairs, within quads, mirror the half row).
__device__ inline float row8_sum(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));  // row_half_mirror
  return v;
}

constexpr int PRUNE_THREADS = 256;
constexpr int PAIR_LANES = 8;

template <bool STATS>
__global__ void __launch_bounds__(PRUNE_THREADS) prune_kernel(PruneArgs a) {
  __shared__ float s_ratio[kMaxBlocks + 1];
  __shared__ unsigned int s_enter[kMaxBlocks + 1];
  __shared__ unsigned int s_completed, s_steps, s_pairs;
  put_stamp(a.stamp);
  const int tid = threadIdx.x;
  for (int m = tid; m <= a.nb; m += PRUNE_THREADS) {
    s_ratio[m] = a.ratio[m];
    s_enter[m] = 0u;
  }
  if (tid == 0) {
    s_completed = 0u;
    s_steps = 0u;
    s_pairs = 0u;
  }
  __syncthreads();
  unsigned int my_steps = 0u, my_pairs = 0u;   // (lane 0 of a group) block steps gathered and pairs taken: the kernel's traffic

  // The list is kSubLists parts, one per XCD of the kernel that made it (workgroup id mod 8), each in the order in
  // which that XCD walked its tiles: neighbouring entries share point rows and centroid blocks.  A workgroup reads
  // the part of its own XCD, so those rows and blocks are fetched into one L2 only and found there again.
  static_assert(kSubLists == 8, "one part per XCD");
  const unsigned int part = blockIdx.x & 7u;
  // (a producer that ran out of room has still counted what it could not write: never read past the part's end)
  const unsigned int total = min(a.count[part * kSubListStride], a.sub_capacity);
  const Pair *list = a.pairs + (size_t)part * a.sub_capacity;
  const unsigned int ngroups = (gridDim.x >> 3) * (PRUNE_THREADS / PAIR_LANES);
  const int q = tid & (PAIR_LANES - 1);
  unsigned int p = (blockIdx.x >> 3) * (PRUNE_THREADS / PAIR_LANES) + (tid / PAIR_LANES);
  bool active = p < total;
  int i = 0, j = 0, m = 0, front = 0;
  float acc = 0.f, tau = 0.f;
  auto unpack = [&](const Pair &pr) {
    const unsigned int jm = (unsigned int)pr.j;
    i = pr.i;
    j = (int)(jm & 0xffffffu);
    m = (int)(jm >> 24);   // first block still to be added
    acc = fmaxf(pr.p, 0.f);
    tau = pr.tau;
    front = pr.p < 0.f ? 0 : a.dprime;   // p < 0: the pair starts over, its first d' dimensions come first
    // An entry that names no point or centroid is skipped (finished at once, offering nothing).  Every producer
    // writes valid entries only; but after a producer's overflow, which the host answers by redoing the step another
    // way, slots inside the counted range may never have been written.
    if ((unsigned int)i >= (unsigned int)a.n || j >= a.k || m > a.nb) {
      i = 0;
      j = 0;
      m = a.nb;
      acc = 1.f;
      tau = 0.f;
      front = a.dprime;
    }
  };
  if (active) {
    unpack(list[p]);
    ++my_pairs;
  }
  unsigned int pn = p + ngroups;   // the entry after this one, requested ahead of its use
  Pair nx = {0, 0, 0.f, 0.f};
  if (pn < total) nx = list[pn];
  while (__any(active)) {
    if (active) {
      const bool ahead = front < a.dprime;
      if (ahead || m < a.nb) {
        // lane q holds float4 q and float4 q + 8 of the 16 in a block
        const int col = (ahead ? front : a.dprime + kBlockDims * m) + 4 * q;
        const int end = ahead ? a.dprime : a.ds;
        const float *xp = a.Xr + (int64_t)i * a.ldx + col;
        const float *yp = ahead ? a.Y + (int64_t)j * a.ds + col : a.Ypdx + ((int64_t)m * a.k + j) * kBlockDims + 4 * q;
        float4 x0 = make_float4(0.f, 0.f, 0.f, 0.f), x1 = x0, y0 = x0, y1 = x0;
        if (col < end) {
          x0 = *reinterpret_cast<const float4 *>(xp);
          y0 = *reinterpret_cast<const float4 *>(yp);
        }
        if (col + 32 < end) {
          x1 = *reinterpret_cast<const float4 *>(xp + 32);
          y1 = *reinterpret_cast<const float4 *>(yp + 32);
        }
        float dx = x0.x - y0.x, dy = x0.y - y0.y, dz = x0.z - y0.z, dw = x0.w - y0.w;
        float s = dx * dx;
        s = fmaf(dy, dy, s);
        s = fmaf(dz, dz, s);
        s = fmaf(dw, dw, s);
        dx = x1.x - y1.x; dy = x1.y - y1.y; dz = x1.z - y1.z; dw = x1.w - y1.w;
        s = fmaf(dx, dx, s);
        s = fmaf(dy, dy, s);
        s = fmaf(dz, dz, s);
        s = fmaf(dw, dw, s);
        acc += row8_sum(s);
        front += kBlockDims;
        m += ahead ? 0 : 1;
        ++my_steps;
      }
      // (behind the first d' dimensions of a pair that starts over there is no test: it has passed it)
      const bool done = !ahead && m >= a.nb;
      bool drop = false;
      if (ahead) {
      } else if (done) {
        if (q == 0) {
          atomicAdd(&s_completed, 1u);
          if (acc < tau) atomicMin(a.best + i, pack_key(acc, j));
        }
      } else {
        drop = acc > s_ratio[m] * tau;   // checkpoint m: t = d' + 64 m dimensions seen
        if (STATS && !drop && q == 0) atomicAdd(&s_enter[m], 1u);
      }
      if (done || drop) {
        p = pn;
        active = p < total;
        if (active) {
          unpack(nx);
          ++my_pairs;
          pn = p + ngroups;
          if (pn < total) nx = list[pn];
        }
      }
    }
  }
  if (q == 0) {
    if (my_steps) atomicAdd(&s_steps, my_steps);
    if (my_pairs) atomicAdd(&s_pairs, my_pairs);
  }
  __syncthreads();
  unsigned long long *sc = a.scal + (size_t)(blockIdx.x & (kStatReplicas - 1)) * SC_COUNT;
  if (tid == 0 && s_completed) atomicAdd(sc + SC_COMPLETED, (unsigned long long)s_completed);
  if (tid == 0 && s_steps) atomicAdd(sc + SC_GATHER_PB, (unsigned long long)s_steps);
  if (tid == 0 && s_pairs) atomicAdd(sc + SC_GATHER_PAIRS, (unsigned long long)s_pairs);
  if (STATS) {
    for (int mm = tid; mm < a.nb; mm += PRUNE_THREADS)
      if (s_enter[mm]) atomicAdd(sc + SC_ENTER + mm, (unsigned long long)s_enter[mm]);
  }
}

hipError_t launch_prune(const PruneArgs &a, hipStream_t st) {
  if (a.nb > kMaxBlocks) return hipErrorInvalidValue;
  int dev = 0, cus = 256;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const unsigned grid = (unsigned)cus * 8u;  // 8 workgroups of 4 waves per CU = full occupancy at <= 64 VGPRs; a multiple of 8
  if (a.block_stats)
    hipLaunchKernelGGL(prune_kernel<true>, dim3(grid), dim3(PRUNE_THREADS), 0, st, a);
  else
    hipLaunchKernelGGL(prune_kernel<false>, dim3(grid), dim3(PRUNE_THREADS), 0, st, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------- candidates of the one-product search, row by row
// The pairs of a search in which nothing is dropped on the way (launch_screen's exact form): a point has a few candidates, found
// by different workgroups at different times.  With a list entry a group of lanes, every entry fetches its point's row again:
// 2.4 entries a point of 1M x 1536 were 19 GB from beyond the L2s, 2.69 ms at 7.2 TB/s.  Here the entries are dealt out to
// their points first (up to `slots` each; more stay in a list, behind the middle of their part, for the kernel above), and a
// group of 8 lanes then takes a point with all of them: the rows stream through once, in a few launches that each take the
// blocks of 64 dimensions whose centroids' part fits an L2 (7.7 GB from beyond the L2s, 1.93 ms; 4.0 entries a point of k = 4096
// 6.76 -> 2.80 ms; in one launch 2.17 and 4.00).  The sums are those of the kernel above.
constexpr int DEAL_THREADS = 256;

__global__ void __launch_bounds__(DEAL_THREADS) deal_pairs_kernel(RowPairsArgs a) {
  const unsigned int part = blockIdx.x & 7u, half = a.sub_capacity / 2, room = a.sub_capacity - half - (unsigned int)a.rows;
  Pair *list = a.pairs + (size_t)part * a.sub_capacity;
  const unsigned int total = a.count[part * kSubListStride];
  if (total > room) {   // no room for what may be left over: reported like a list that is too short
    if (threadIdx.x == 0) atomicOr(a.overflow, 1u);
    return;
  }
  for (unsigned int p0 = (blockIdx.x >> 3) * DEAL_THREADS; p0 < total; p0 += (gridDim.x >> 3) * DEAL_THREADS) {
    const unsigned int p = p0 + threadIdx.x;
    bool left = false;
    Pair pr = {0, 0, 0.f, 0.f};
    if (p < total) {
      pr = list[p];
      const unsigned int r = (unsigned int)((int64_t)pr.i - a.row_base);
      if (r < (unsigned int)a.rows && (unsigned int)pr.j < (unsigned int)a.k) {   // (see the kernel above: never written)
        const unsigned int rank = atomicAdd(a.row_count + r, 1u);
        if (rank < (unsigned int)a.slots) a.cand[(size_t)r * a.slots + rank] = pr.j;
        else left = true;
      }
    }
    const unsigned long long mask = __ballot(left);
    if (mask) {
      const int lane = threadIdx.x & 63, first = __builtin_ctzll(mask);
      unsigned int base = 0;
      if (lane == first) base = atomicAdd(a.left_count + part * kSubListStride, (unsigned int)__popcll(mask));
      base = __shfl(base, first, 64);
      if (left) list[half + base + __popcll(mask & ((1ull << lane) - 1))] = pr;
    }
  }
}

// Blocks [m0, m1) of all points' candidates: the sums so far come from memory and go back there, four to a vector.
__global__ void __launch_bounds__(PRUNE_THREADS) row_pairs_kernel(RowPairsArgs a, int m0, int m1) {
  __shared__ unsigned int s_pairs;
  if (threadIdx.x == 0) s_pairs = 0u;
  __syncthreads();
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  constexpr int U = 4;   // candidates at a time
  const int q = threadIdx.x & (PAIR_LANES - 1);
  unsigned int my_pairs = 0u;
  const int ngroups = gridDim.x * (PRUNE_THREADS / PAIR_LANES);
  // a row's number of candidates and its first four are asked for a row ahead
  int r = blockIdx.x * (PRUNE_THREADS / PAIR_LANES) + threadIdx.x / PAIR_LANES;
  unsigned int count = 0u;
  int4 four = make_int4(0, 0, 0, 0);
  if (r < a.rows) {
    count = a.row_count[r];
    four = *reinterpret_cast<const int4 *>(a.cand + (size_t)r * a.slots);
  }
  for (int next; r < a.rows; r = next) {
    next = r + ngroups;
    const int c = (int)min(count, (unsigned int)a.slots);
    int4 cand = four;
    if (next < a.rows) {
      count = a.row_count[next];
      four = *reinterpret_cast<const int4 *>(a.cand + (size_t)next * a.slots);
    }
    const float *x = a.Xr + (a.row_base + r) * a.ldx + 4 * q;
    unsigned long long best = ~0ull;
    for (int c0 = 0; c0 < c; c0 += U) {
      const int nu = min(U, c - c0);
      float4 *sums = reinterpret_cast<float4 *>(a.pairs + (size_t)(c0 / U + 1) * a.sub_capacity - a.rows) + r;
      if (c0 > 0) cand = *reinterpret_cast<const int4 *>(a.cand + (size_t)r * a.slots + c0);
      const int j[U] = {cand.x, cand.y, cand.z, cand.w};   // (those past the row's last are not looked at)
      float acc[U] = {0.f, 0.f, 0.f, 0.f};
      if (m0 > 0) {
        const float4 v = *sums;
        acc[0] = v.x; acc[1] = v.y; acc[2] = v.z; acc[3] = v.w;
      }
      f32x4_t x0, x1, n0, n1;
      // (the rows pass through once: they are not to displace the centroids' blocks)
      auto fetch = [&](int m, f32x4_t &v0, f32x4_t &v1) {
        const int col = kBlockDims * m + 4 * q;
        v0 = v1 = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (col < a.K) v0 = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(x + kBlockDims * m));
        if (col + 32 < a.K) v1 = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(x + kBlockDims * m + 32));
      };
      fetch(m0, n0, n1);
      for (int m = m0; m < m1; ++m) {
        float4 y0[U], y1[U];
        const float *y = a.Ypdx + (int64_t)m * a.k * kBlockDims + 4 * q;
        x0 = n0;
        x1 = n1;
        if (m + 1 < m1) fetch(m + 1, n0, n1);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (u < nu) {   // (zeros past the K dimensions)
            y0[u] = *reinterpret_cast<const float4 *>(y + (int64_t)j[u] * kBlockDims);
            y1[u] = *reinterpret_cast<const float4 *>(y + (int64_t)j[u] * kBlockDims + 32);
          }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (u < nu) {
            float dx = x0.x - y0[u].x, dy = x0.y - y0[u].y, dz = x0.z - y0[u].z, dw = x0.w - y0[u].w;
            float s = dx * dx;
            s = fmaf(dy, dy, s);
            s = fmaf(dz, dz, s);
            s = fmaf(dw, dw, s);
            dx = x1.x - y1[u].x; dy = x1.y - y1[u].y; dz = x1.z - y1[u].z; dw = x1.w - y1[u].w;
            s = fmaf(dx, dx, s);
            s = fmaf(dy, dy, s);
            s = fmaf(dz, dz, s);
            s = fmaf(dw, dw, s);
            acc[u] += row8_sum(s);
          }
      }
      if (m1 < a.nb) {
        if (q == 0) *sums = make_float4(acc[0], acc[1], acc[2], acc[3]);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (u < nu && acc[u] < kFarAway) {
            const unsigned long long key = pack_key(acc[u], j[u]);
            best = key < best ? key : best;
          }
        my_pairs += nu;
      }
    }
    if (q == 0 && best != ~0ull) atomicMin(a.best + a.row_base + r, best);   // (pairs left in the list come on top)
  }
  if (q == 0 && my_pairs) atomicAdd(&s_pairs, my_pairs);
  __syncthreads();
  if (threadIdx.x == 0 && s_pairs) {
    unsigned long long *sc = a.scal + (size_t)(blockIdx.x & (kStatReplicas - 1)) * SC_COUNT;
    atomicAdd(sc + SC_COMPLETED, (unsigned long long)s_pairs);
    atomicAdd(sc + SC_GATHER_PB, (unsigned long long)s_pairs * a.nb);
    atomicAdd(sc + SC_GATHER_PAIRS, (unsigned long long)s_pairs);
  }
}

hipError_t launch_row_pairs(const RowPairsArgs &a, hipStream_t st) {
  if (a.rows <= 0) return hipSuccess;
  if ((a.slots != 4 && a.slots != 8) || a.nb < 1 || a.K % 16 != 0 || a.sub_capacity < 8u * (unsigned int)a.rows) return hipErrorInvalidValue;
  hipError_t rc = launch_fill_u32(a.row_count, a.rows, 0u, st);
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(deal_pairs_kernel, dim3((unsigned)num_cus() * 4u / 8u * 8u), dim3(DEAL_THREADS), 0, st, a);
  const int64_t blocks = ((int64_t)a.rows * PAIR_LANES + PRUNE_THREADS - 1) / PRUNE_THREADS;
  const dim3 grid((unsigned)std::min<int64_t>(blocks, (int64_t)num_cus() * 8));
  // as many blocks a launch as keep the centroids' part of them within one L2 (4 MB): 1M x 1536, k = 4096 with a launch of 1 MB
  // 16.1 ms for the whole stage, 2 MB 15.0, 4 MB 14.8, 8 MB 15.0, all blocks 16.0
  const int step = (int)std::max<int64_t>(1, std::min<int64_t>(a.nb, ((int64_t)4 << 20) / ((int64_t)a.k * kBlockDims * 4)));
  for (int m0 = 0; m0 < a.nb; m0 += step)
    hipLaunchKernelGGL(row_pairs_kernel, grid, dim3(PRUNE_THREADS), 0, st, a, m0, std::min(m0 + step, a.nb));
  return hipGetLastError();
}

}  // namespace skm
