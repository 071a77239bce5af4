// HBM-bound kernels around the two phases: initial threshold, centroid preparation (norms and the
// block-major copy of the trailing dimensions), unpacking of the argmin, and the centroid update as
// a segmented reduction (Section 3.2 "In between iterations", Section 3.4 "Initial threshold").
#include "skm_internal.h"

namespace skm {

// Sum over the 32 lanes of either half of a wavefront, in every lane: partners 1, 2, 4, 8 and 16 lanes away in turn, on the
// vector unit's lane moves (once pairs, quads and half rows agree, a mirror brings the partner's value).
__device__ inline float half_sum(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, false));   // row_half_mirror
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, false));   // row_mirror
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned int, v), __builtin_bit_cast(unsigned int, v), false, false);
  return __builtin_bit_cast(float, (unsigned int)r[0]) + __builtin_bit_cast(float, (unsigned int)r[1]);
}
__device__ inline float wave_sum(float v) {
  v = half_sum(v);
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned int, v), __builtin_bit_cast(unsigned int, v), false, false);
  return __builtin_bit_cast(float, (unsigned int)r[0]) + __builtin_bit_cast(float, (unsigned int)r[1]);
}
__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m, 64);
  return v;
}

int num_cus() {
  static const int cus = []() {   // (initialised once, synchronised between threads)
    int dev = 0, v = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    return v;
  }();
  return cus;
}

// ------------------------------------------------------------------ initial threshold
// One wavefront per point: the rotated row and the row of its incumbent centroid are read as
// float4 per lane (1 KiB per wavefront load); squared differences over all dims give tau_i.
// NV = float4 loads per lane and operand (rows of up to 256 * NV floats): all loads of a row pair are
// issued before the first use, so that a wavefront keeps 2 * NV KiB in flight.
//
// The same pass can emit the prefix norms of the point that the progressive kernel tests against: every
// checkpoint t = d' + 64 m is a multiple of 16, so the table xnp[p][i] = ||x_i[0 : 16 (p + 1))||^2 serves any d',
// and the points do not change during a fit, so it is written once (PrefixOut), by the first pass that has the rows
// in registers anyway.  Lane l holds dims 4 l + 256 u .. + 3; a quad of lanes holds a 16-dim piece, and an
// inclusive scan over the 16 quads of the wavefront (then over u) gives every quad the norm of the row up to the
// end of its piece.
// With `xs` the pass also writes the split-fp16 copy of the row that the progressive kernel multiplies (the layout
// of launch_split_rows).
struct PrefixOut {
  float *xnp;        // [ds / 16][n] or NULL
  int64_t n;
  int32_t ds;
  uint32_t *xs;      // the split copy or NULL
  uint32_t *xh;      // or NULL (with xs): the hi halves as a plane of their own
  const unsigned int *absmax;   // bound of |X| (bit pattern) that fixes the scale of xs
  float scale;       // split_scale(*absmax), set by the kernel
  // Regrouping (all three or none): output slot p takes point order[p]; its row is copied to xr_out (row stride ds)
  // and its label to label_out[p], so that every per-point array continues in the new order.
  const int32_t *order;
  float *xr_out;
  int32_t *label_out;
  unsigned int *unset = nullptr;   // labels taken from packed keys: bit 1 is set if a point has none
  int span = 64;                   // BATCH: points a workgroup takes at a time (64, or 16 when there are few)
  stamp_t *stamp = nullptr;
  int hi_dims = 1 << 30;           // xh is zero from this dimension on
  uint32_t *xd = nullptr;          // or NULL (with xs): the hi halves from dimension xd_from on (CentroidPrep::Yd)
  int xd_from = 0;
};

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
struct SplitHalves {
  uint2 hi, lo;
};
__device__ inline SplitHalves split_halves(const float4 &v, float scale) {
  const f32x2_t p0 = {v.x * scale, v.y * scale}, p1 = {v.z * scale, v.w * scale};
  const f16x2_t h0 = __builtin_convertvector(p0, f16x2_t), h1 = __builtin_convertvector(p1, f16x2_t);
  const f16x2_t l0 = __builtin_convertvector(p0 - __builtin_convertvector(h0, f32x2_t), f16x2_t);
  const f16x2_t l1 = __builtin_convertvector(p1 - __builtin_convertvector(h1, f32x2_t), f16x2_t);
  return {make_uint2(__builtin_bit_cast(unsigned int, h0), __builtin_bit_cast(unsigned int, h1)),
          make_uint2(__builtin_bit_cast(unsigned int, l0), __builtin_bit_cast(unsigned int, l1))};
}
// a quad of lanes holds a granule; its lanes 0, 1 receive the 32 bytes of hi halves, lanes 2, 3 the lo halves, 16 bytes each
__device__ inline uint4 granule_piece(const SplitHalves &v, int lane) {
  auto even = [](unsigned int w) { return (unsigned int)__builtin_amdgcn_mov_dpp((int)w, 0x88, 0xF, 0xF, true); };   // quad_perm [0,2,0,2]
  auto odd = [](unsigned int w) { return (unsigned int)__builtin_amdgcn_mov_dpp((int)w, 0xDD, 0xF, 0xF, true); };    // quad_perm [1,3,1,3]
  const uint4 h = make_uint4(even(v.hi.x), even(v.hi.y), odd(v.hi.x), odd(v.hi.y));
  const uint4 l = make_uint4(even(v.lo.x), even(v.lo.y), odd(v.lo.x), odd(v.lo.y));
  return lane & 2 ? l : h;
}
// this lane's float4 at column c (a quarter of granule c / 16; c / 4 = lane modulo 4) -> hi and lo halves in the split copy of
// row i
__device__ inline void emit_split(const PrefixOut &po, int64_t i, int c, const float4 &v) {
  const SplitHalves h = split_halves(v, po.scale);
  const int ld = split_ld(po.ds), q = (c / 4) & 3;
  *reinterpret_cast<uint4 *>(po.xs + split_row(i, ld) + 32 * (c / 16 + 1) + 4 * q) = granule_piece(h, q);
  if (po.xh)
    *reinterpret_cast<uint2 *>(po.xh + split_row(i, ld / 2) + 32 * (c / 32) + (c % 32) / 2) = c < po.hi_dims ? h.hi : make_uint2(0u, 0u);
  if (po.xd && c >= po.xd_from) {
    const int e = c - po.xd_from;
    *reinterpret_cast<uint2 *>(po.xd + split_row(i, ld) + 32 * (po.xd_from / 32 + e / 32) + (e % 32) / 2) = h.hi;
  }
}
// The same of rows i and i + 1, i even (tables of points), 256 columns from c0 on, through 2 KB of LDS of this wavefront's own:
// there the two rows' granules lie as they do in memory, 128 bytes each (the 16-byte pieces rotated by the granule's number),
// and every store takes whole lines.  (Half lines a store, a row a wavefront: the pass of 1M x 1536 that writes the tables
// 4.7 instead of 3.3 ms.)  All lanes take part; zeros past the row.
__device__ inline void emit_split_pair(const PrefixOut &po, int64_t i, int lane, int c0, const float4 &v0, const float4 &v1,
                                       uint32_t *ex) {
  const int ld = split_ld(po.ds);
  auto at = [](int g, int piece) { return 32 * g + 4 * (piece ^ (g & 7)); };
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const SplitHalves h = split_halves(r ? v1 : v0, po.scale);
    uint32_t *w = ex + at(lane >> 2, 4 * r + ((lane >> 1) & 1)) + 2 * (lane & 1);
    *reinterpret_cast<uint2 *>(w) = h.hi;
    *reinterpret_cast<uint2 *>(ex + at(lane >> 2, 4 * r + 2 + ((lane >> 1) & 1)) + 2 * (lane & 1)) = h.lo;
  }
  __builtin_amdgcn_wave_barrier();
  uint32_t *dst = po.xs + (i >> 1) * (2 * (int64_t)ld) + 32 * (c0 / 16 + 1) + 4 * lane;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int g = 8 * e + (lane >> 3);
    if (c0 + 16 * g < po.ds) *reinterpret_cast<uint4 *>(dst + 256 * e) = *reinterpret_cast<const uint4 *>(ex + at(g, lane & 7));
  }
  if (po.xh) {   // unit lane / 8 of 32 dimensions, row (lane / 4) & 1, piece lane & 3: a half of one granule's hi halves
    const int g = 2 * (lane >> 3) + ((lane >> 1) & 1);
    if (c0 + 16 * g < po.ds)
      *reinterpret_cast<uint4 *>(po.xh + (i >> 1) * (int64_t)ld + c0 + 4 * lane) =
          *reinterpret_cast<const uint4 *>(ex + at(g, (lane & 4) + (lane & 1)));
  }
  __builtin_amdgcn_wave_barrier();
}
// the zero granules before and after the data of row i (lanes 0..3 and 4..7, 16 bytes each), and the zero half of the hi
// plane's last unit (lanes 8, 9)
__device__ inline void emit_split_pads(const PrefixOut &po, int64_t i, int lane) {
  if (lane < 8) {
    uint32_t *dst = po.xs + split_row(i, split_ld(po.ds)) + (lane < 4 ? 0 : 32 * (po.ds / 16 + 1)) + 4 * (lane & 3);
    *reinterpret_cast<uint4 *>(dst) = make_uint4(0u, 0u, 0u, 0u);
  } else if (lane < 10 && po.xh && po.ds % 32 != 0) {
    uint32_t *dst = po.xh + split_row(i, split_ld(po.ds) / 2) + 32 * (po.ds / 32) + 8 + 4 * (lane - 8);
    *reinterpret_cast<uint4 *>(dst) = make_uint4(0u, 0u, 0u, 0u);
  }
}

// inclusive scan over the 16 quads of a wavefront of a value that is equal within each quad
__device__ inline float quad_scan64(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x114, 0xF, 0xF, false));  // row_shr:4
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x118, 0xF, 0xF, false));  // row_shr:8
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x142, 0xA, 0xF, false));  // row_bcast:15 -> rows 1, 3
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x143, 0xC, 0xF, false));  // row_bcast:31 -> rows 2, 3
  return v;
}
__device__ inline float quad_sum(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  return v;
}
// q = sum of squares of this lane's float4 at column c0 = 4 lane + 256 u; base = norm of the row before column 256 u.
// Returns the norm of the row up to column 256 (u + 1).
// With `stage` (LDS, [ds / 16][64]) the value goes to column `slot` of it instead of the table: the caller writes the
// table 64 points at a time.
__device__ inline float emit_prefix(const PrefixOut &po, int64_t i, int lane, int u, float q, float base,
                                    float *stage = nullptr, int slot = 0) {
  const float upto = base + quad_scan64(quad_sum(q));   // norm up to the end of this quad's 16-dim piece
  const int t = 256 * u + 16 * (lane >> 2) + 16;          // that end
  if ((lane & 3) == 0 && t <= po.ds) {
    if (stage) stage[((t >> 4) - 1) * 64 + slot] = upto;
    else po.xnp[(int64_t)((t >> 4) - 1) * po.n + i] = upto;
  }
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, upto), 63));
}

// 16-byte load with the non-temporal hint (data read once)
__device__ inline float4 load_stream4(const float *p) {
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  const f32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}

// TABLES (po.xnp and po.xs; po.order too if the points change places).  Up to 2048 dimensions (BATCH) a workgroup takes 64 consecutive
// points at a time and writes their prefix norms through LDS, 256 contiguous bytes per table row, instead of one 4-byte store per
// point and row.  Where 64 points a workgroup would leave most of the chip without one (a wavefront then walks sixteen rows one
// after the other while other CUs idle), it takes 16.
// A pair of rows is a chain of loads (place, label, centroid) and of sums over the lanes, and registers allow sixteen wavefronts a CU.
// Rows of up to 256 dimensions leave room for the next pair's labels and rows, requested ahead of this one's: 120 001 x 208 56.6 -> 45.5
// us, changing places as well 108.7 -> 94.6 (3.7 TB/s); 20 000 x 128 15.9 -> 14.2. (More wavefronts instead, with registers in
// memory: five to six a SIMD 80 and 151 us, 2.5M x 384 2.92 -> 3.31 ms, 1M x 768 2.23 -> 2.31.)
// Without TABLES their code is left out: it costs registers (NV = 6: 68 without it, 137 with it; labels and distances of 11 800 x 1152 in 13.1
// and 16.9 us).
constexpr int kPrefixStageRows = 128;   // ds <= 2048 in the batched form
template <int NV, bool TABLES>
__global__ void __launch_bounds__(256) tau_init_kernel(const float *Xr, int64_t ldx, int64_t n, int32_t ds,
                                                       const float *Y, int64_t ldy, const int32_t *assign, float *tau,
                                                       unsigned long long *best, PrefixOut po) {
  constexpr bool BATCH = TABLES && NV > 0, AHEAD = NV == 1;
  __shared__ float s_np[BATCH ? kPrefixStageRows * 64 : 1];
  __shared__ __align__(16) uint32_t s_pair[BATCH ? 4 * 512 : 4];
  put_stamp(po.stamp);
  if (TABLES) po.scale = split_scale(*po.absmax);
  const int lane = threadIdx.x & 63;
  auto point = [&](int64_t p) {   // output slot p <- point i
    const int64_t i = TABLES && po.order ? (int64_t)po.order[p] : p;
    int a;
    if (assign) {
      a = assign[i];
    } else {   // the labels are still packed keys (an argmin that has just run)
      const unsigned long long key = best[i];
      a = (int)(key & 0xffffffffull);
      if (key == ~0ull) {   // no kernel offered this point a centroid: reported, kept in range
        a = 0;
        if (lane == 0 && po.unset) atomicOr(po.unset, 2u);
      }
    }
    const float *x = Xr + i * ldx;
    const float *y = Y + (int64_t)a * ldy;
    float s = 0.f;
    if (NV > 0) {
      float4 xv[NV > 0 ? NV : 1], yv[NV > 0 ? NV : 1];
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const int c = lane * 4 + 256 * u;
        // the points stream through once per step: keep them from displacing the centroids in the L2
        xv[u] = c < ds ? load_stream4(x + c) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const int c = lane * 4 + 256 * u;
        yv[u] = c < ds ? *reinterpret_cast<const float4 *>(y + c) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const float dx = xv[u].x - yv[u].x, dy = xv[u].y - yv[u].y, dz = xv[u].z - yv[u].z, dw = xv[u].w - yv[u].w;
        s = fmaf(dx, dx, s);
        s = fmaf(dy, dy, s);
        s = fmaf(dz, dz, s);
        s = fmaf(dw, dw, s);
      }
    } else {
      float base = 0.f;
      for (int c0 = 0; c0 < ds; c0 += 256) {
        const int c = c0 + lane * 4;
        float4 xv = make_float4(0.f, 0.f, 0.f, 0.f), yv = xv;
        if (c < ds) {
          xv = *reinterpret_cast<const float4 *>(x + c);
          yv = *reinterpret_cast<const float4 *>(y + c);
        }
        const float dx = xv.x - yv.x, dy = xv.y - yv.y, dz = xv.z - yv.z, dw = xv.w - yv.w;
        s = fmaf(dx, dx, s);
        s = fmaf(dy, dy, s);
        s = fmaf(dz, dz, s);
        s = fmaf(dw, dw, s);
        if (TABLES) {
          const float q = fmaf(xv.x, xv.x, fmaf(xv.y, xv.y, fmaf(xv.z, xv.z, xv.w * xv.w)));
          base = emit_prefix(po, p, lane, c0 >> 8, q, base);
          if (c0 == 0) emit_split_pads(po, p, lane);
          if (c < ds) {
            emit_split(po, p, c, xv);
            if (po.xr_out) *reinterpret_cast<float4 *>(po.xr_out + p * (int64_t)ds + c) = xv;
          }
        }
      }
    }
    s = wave_sum(s);
    if (lane == 0) {
      if (tau) tau[p] = s;
      if (best) best[p] = pack_key(s, a);
      if (po.label_out) po.label_out[p] = a;
    }
  };
  // rows p and p + 1 (p even), for the tables; past the end row p stands for row p + 1 and only fills the odd row of its pair
  constexpr int NX = NV > 0 ? NV : 1;
  auto take_two = [&](int64_t p, int (&a)[2], float4 (&xv)[2][NX]) {   // their labels and rows
    const bool both = p + 1 < n;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int64_t o = both ? p + r : p, i = po.order ? (int64_t)po.order[o] : o;
      if (assign) {
        a[r] = assign[i];
      } else {   // the labels are still packed keys (an argmin that has just run)
        const unsigned long long key = best[i];
        a[r] = (int)(key & 0xffffffffull);
        if (key == ~0ull) {   // no kernel offered this point a centroid: reported, kept in range
          a[r] = 0;
          if (lane == 0 && po.unset) atomicOr(po.unset, 2u);
        }
      }
#pragma unroll
      for (int u = 0; u < NX; ++u) {
        const int c = lane * 4 + 256 * u;
        xv[r][u] = c < ds ? load_stream4(Xr + i * ldx + c) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  };
  auto two_points = [&](int64_t p, int slot, const int (&a)[2], const float4 (&xv)[2][NX]) {
    const bool both = p + 1 < n;
    float s[2] = {0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      __builtin_amdgcn_sched_barrier(0);   // (one centroid row at a time in registers)
      const float *y = Y + (int64_t)a[r] * ldy;
      float4 yv[NX];
#pragma unroll
      for (int u = 0; u < NX; ++u) {
        const int c = lane * 4 + 256 * u;
        yv[u] = c < ds ? *reinterpret_cast<const float4 *>(y + c) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      float base = 0.f;
#pragma unroll
      for (int u = 0; u < NX; ++u) {
        const float4 &x = xv[r][u];
        const float dx = x.x - yv[u].x, dy = x.y - yv[u].y, dz = x.z - yv[u].z, dw = x.w - yv[u].w;
        s[r] = fmaf(dx, dx, s[r]);
        s[r] = fmaf(dy, dy, s[r]);
        s[r] = fmaf(dz, dz, s[r]);
        s[r] = fmaf(dw, dw, s[r]);
      }
#pragma unroll
      for (int u = 0; u < NX; ++u) {
        if (256 * u >= ds) break;
        const float4 &x = xv[r][u];
        const float q = fmaf(x.x, x.x, fmaf(x.y, x.y, fmaf(x.z, x.z, x.w * x.w)));
        base = emit_prefix(po, p + r, lane, u, q, base, s_np, slot + r);
      }
    }
    emit_split_pads(po, p, lane);
    emit_split_pads(po, p + 1, lane);
#pragma unroll
    for (int u = 0; u < NX; ++u)
      if (256 * u < ds) emit_split_pair(po, p, lane, 256 * u, xv[0][u], xv[1][u], s_pair + 512 * (threadIdx.x >> 6));
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      if (r == 1 && !both) break;
      if (po.xr_out) {
#pragma unroll
        for (int u = 0; u < NX; ++u)
          if (lane * 4 + 256 * u < ds) *reinterpret_cast<float4 *>(po.xr_out + (p + r) * (int64_t)ds + lane * 4 + 256 * u) = xv[r][u];
      }
      const float sum = wave_sum(s[r]);
      if (lane == 0) {
        if (tau) tau[p + r] = sum;
        if (best) best[p + r] = pack_key(sum, a[r]);
        if (po.label_out) po.label_out[p + r] = a[r];
      }
    }
  };
  if (BATCH) {
    const int wave = threadIdx.x >> 6, rows = ds >> 4;
    const int span = po.span, sh = span == 64 ? 6 : 4;
    for (int64_t b0 = (int64_t)blockIdx.x * span; b0 < n; b0 += (int64_t)gridDim.x * span) {
      int a[2], a_next[2] = {0, 0};
      float4 xv[2][NX], xv_next[2][NX];
      if (AHEAD && b0 + 2 * wave < n) take_two(b0 + 2 * wave, a_next, xv_next);
      for (int slot = 2 * wave; slot < span && b0 + slot < n; slot += 8) {
        if (AHEAD) {
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            a[r] = a_next[r];
            xv[r][0] = xv_next[r][0];
          }
          if (slot + 8 < span && b0 + slot + 8 < n) take_two(b0 + slot + 8, a_next, xv_next);
        } else {
          take_two(b0 + slot, a, xv);
        }
        two_points(b0 + slot, slot, a, xv);
      }
      __syncthreads();
      const int col = threadIdx.x & (span - 1);
      if (b0 + col < n)
        for (int p = threadIdx.x >> sh; p < rows; p += 256 >> sh) po.xnp[(int64_t)p * po.n + b0 + col] = s_np[p * 64 + col];
      __syncthreads();
    }
  } else {
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += nwaves) point(i);
  }
}

// The pass over rows of at most 128 H dimensions (H = 1, 2) that writes no tables: half a wavefront holds a row and takes two
// rows at a time.  With a wavefront a row, lanes idle and one row in flight at a time, 100 003 x 100 took 27 us, 20 000 x
// 128 9.3 and 120 001 x 208 32.7; now 11.4, 4.2 and 18.7.  The sums are those of the form above, bit for bit.
template <int H>
__device__ inline void tau_short(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const float *Y, int64_t ldy, const int32_t *assign,
                                 float *tau, unsigned long long *best, int32_t *label_out, unsigned int *unset, int block, int nblocks) {
  const int lane = threadIdx.x & 31, c = 4 * lane;
  for (int64_t p0 = (int64_t)block * 16 + (threadIdx.x >> 5); p0 < n; p0 += (int64_t)nblocks * 16) {
    int64_t p[2];
    int a[2];
    float4 x[2][H], y[2][H];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      p[u] = min(p0 + 8 * u, n - 1);   // (past the end: the last row once more, not stored)
#pragma unroll
      for (int h = 0; h < H; ++h)
        x[u][h] = c + 128 * h < ds ? load_stream4(Xr + p[u] * ldx + c + 128 * h) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (assign) {
        a[u] = assign[p[u]];
      } else {   // the labels are still packed keys (an argmin that has just run)
        const unsigned long long key = best[p[u]];
        a[u] = (int)(key & 0xffffffffull);
        if (key == ~0ull) {   // no kernel offered this point a centroid: reported, kept in range
          a[u] = 0;
          if (lane == 0 && unset) atomicOr(unset, 2u);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int h = 0; h < H; ++h)
        y[u][h] = c + 128 * h < ds ? *reinterpret_cast<const float4 *>(Y + (int64_t)a[u] * ldy + c + 128 * h)
                                   : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float s = 0.f;
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const float dx = x[u][h].x - y[u][h].x, dy = x[u][h].y - y[u][h].y, dz = x[u][h].z - y[u][h].z, dw = x[u][h].w - y[u][h].w;
        float q = dx * dx;
        q = fmaf(dy, dy, q);
        q = fmaf(dz, dz, q);
        q = fmaf(dw, dw, q);
        q = half_sum(q);
        s = h == 0 ? q : s + q;
      }
      if (lane == 0 && p0 + 8 * u < n) {
        if (tau) tau[p[u]] = s;
        if (best) best[p[u]] = pack_key(s, a[u]);
        if (label_out) label_out[p[u]] = a[u];
      }
    }
  }
}
template <int H>
__global__ void __launch_bounds__(256) tau_short_kernel(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const float *Y,
                                                        int64_t ldy, const int32_t *assign, float *tau,
                                                        unsigned long long *best, int32_t *label_out, unsigned int *unset,
                                                        stamp_t *stamp) {
  put_stamp(stamp);
  tau_short<H>(Xr, ldx, n, ds, Y, ldy, assign, tau, best, label_out, unset, blockIdx.x, gridDim.x);
}
static unsigned tau_short_grid(int64_t n) { return (unsigned)std::min<int64_t>((n + 15) / 16, (int64_t)num_cus() * 32); }

hipError_t launch_tau_init(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const float *Y, int64_t ldy,
                           const int32_t *assign, float *tau, unsigned long long *best, hipStream_t st, float *xnp,
                           uint32_t *xs, const unsigned int *x_absmax, const int32_t *order, float *xr_out,
                           int32_t *label_out, uint32_t *xh, unsigned int *unset, stamp_t *stamp) {
  if (n <= 0) return hipSuccess;
  const int nv = (ds + 255) / 256;
  const bool batch = xnp != nullptr && nv <= 8;   // (then ds / 16 <= kPrefixStageRows)
  // (below five workgroups a CU, 16 points at a time)
  const int span = n >= (int64_t)num_cus() * 5 * 64 ? 64 : 16;
  int64_t blocks = batch ? (n + span - 1) / span : (n + 3) / 4;
  const int64_t cap = (int64_t)num_cus() * 32;
  if (blocks > cap) blocks = cap;
  if (xs && (ds % 16 != 0 || !x_absmax)) return hipErrorInvalidValue;
  if ((xnp != nullptr) != (xs != nullptr) || (order && !xnp)) return hipErrorInvalidValue;   // (all tables or none)
  if ((order != nullptr) != (xr_out != nullptr) || (order && (!label_out || !assign)) || (!assign && !best)) return hipErrorInvalidValue;
  if (xr_out && (reinterpret_cast<uintptr_t>(xr_out) & 15u)) return hipErrorInvalidValue;
  if (xh && (!xs || (reinterpret_cast<uintptr_t>(xh) & 15u))) return hipErrorInvalidValue;
  if (ds <= 256 && !xnp && !xs && !order) {
    hipLaunchKernelGGL(ds <= 128 ? tau_short_kernel<1> : tau_short_kernel<2>, dim3(tau_short_grid(n)), dim3(256), 0, st, Xr, ldx, n, ds, Y, ldy,
                       assign, tau, best, label_out, unset, stamp);
    return hipGetLastError();
  }
  const PrefixOut po{xnp, n, ds, xs, xh, x_absmax, 0.f, order, xr_out, label_out, unset, span, stamp};
  // Long rows that stream from memory do so faster four workgroups a CU (room in LDS that is not used) than seven: 1M x 1536 1218 -> 1189
  // us (in a fit, points grouped, 1132 -> 1118), 400 000 x 2048 586 -> 582, 100 000 x 1536 98.5 -> 97.7; but 11 800 x 1152 11.4 -> 12.8, and
  // rows of up to 1024 dimensions, 1M x 768 632 -> 635, 60 000 x 1024 37.4 -> 40.4, 1M x 384 311 -> 409.  (The line: the rows outgrow the
  // Infinity Cache of 256 MB.)
  const unsigned room = !xnp && nv > 4 && nv <= 8 && n * ds >= (int64_t)1 << 26 ? 32 * 1024 : 0;
#define SKM_TAU_LAUNCH(NV)                                                                                          \
  hipLaunchKernelGGL((xnp ? tau_init_kernel<NV, true> : tau_init_kernel<NV, false>), dim3((unsigned)blocks), dim3(256), room, st, \
                     Xr, ldx, n, ds, Y, ldy, assign, tau, best, po)
  if (nv <= 1) SKM_TAU_LAUNCH(1);
  else if (nv <= 2) SKM_TAU_LAUNCH(2);
  else if (nv <= 3) SKM_TAU_LAUNCH(3);
  else if (nv <= 4) SKM_TAU_LAUNCH(4);
  else if (nv <= 6) SKM_TAU_LAUNCH(6);
  else if (nv <= 8) SKM_TAU_LAUNCH(8);
  else SKM_TAU_LAUNCH(0);
#undef SKM_TAU_LAUNCH
  return hipGetLastError();
}

// Thresholds of a step before which few clusters were touched: a point whose cluster neither gained nor lost a point has the
// centroid, the label and with them the threshold of the step before, which is still in tau[]; only the others are taken again
// (a wavefront's points one after the other, two rows in flight).  touched: a word per cluster, or NULL where none was.  The
// sums are those of tau_init_kernel.  1M x 1536 1112 us -> 8 with no cluster touched, 103 with a tenth of them.
template <int NV>
__global__ void __launch_bounds__(256) tau_kept_kernel(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const float *Y,
                                                       int64_t ldy, const int32_t *assign, const uint32_t *touched, float *tau,
                                                       unsigned long long *best, stamp_t *stamp) {
  put_stamp(stamp);
  const int lane = threadIdx.x & 63;
  for (int64_t base = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64; base < n; base += (int64_t)gridDim.x * 256) {
    const int64_t p = min(base + lane, n - 1);
    const bool in = base + lane < n;
    const int a = assign[p];
    const bool again = in && touched && touched[a] != 0u;
    if (in && !again) best[p] = pack_key(tau[p], a);
    unsigned long long left = __ballot(again);
    while (left) {
      int64_t i[2];
      int c[2];
      float4 x[2][NV], y[2][NV];
      const int first = __builtin_ctzll(left);
      left &= left - 1ull;
      const bool two = left != 0ull;
      const int second = two ? __builtin_ctzll(left) : first;
      left &= left - (two ? 1ull : 0ull);
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int b = r ? second : first;
        i[r] = base + b;
        c[r] = __builtin_amdgcn_readlane(a, b);
#pragma unroll
        for (int u = 0; u < NV; ++u) {
          const int col = lane * 4 + 256 * u;
          x[r][u] = col < ds ? load_stream4(Xr + i[r] * ldx + col) : make_float4(0.f, 0.f, 0.f, 0.f);
          y[r][u] = col < ds ? *reinterpret_cast<const float4 *>(Y + (int64_t)c[r] * ldy + col) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
          const float dx = x[r][u].x - y[r][u].x, dy = x[r][u].y - y[r][u].y, dz = x[r][u].z - y[r][u].z, dw = x[r][u].w - y[r][u].w;
          s = fmaf(dx, dx, s);
          s = fmaf(dy, dy, s);
          s = fmaf(dz, dz, s);
          s = fmaf(dw, dw, s);
        }
        s = wave_sum(s);
        if (lane == 0) {
          tau[i[r]] = s;
          best[i[r]] = pack_key(s, c[r]);
        }
      }
    }
  }
}
hipError_t launch_tau_kept(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const float *Y, int64_t ldy, const int32_t *assign,
                           const uint32_t *touched, float *tau, unsigned long long *best, hipStream_t st, stamp_t *stamp) {
  if (n <= 0) return hipSuccess;
  if (ds > kTauKeptMaxDims) return hipErrorInvalidValue;
  const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, (int64_t)num_cus() * 32);
  const int nv = (ds + 255) / 256;
#define SKM_TAU_KEPT(NV) hipLaunchKernelGGL(tau_kept_kernel<NV>, dim3(blocks), dim3(256), 0, st, Xr, ldx, n, ds, Y, ldy, assign, touched, tau, best, stamp)
  if (nv <= 1) SKM_TAU_KEPT(1);
  else if (nv <= 2) SKM_TAU_KEPT(2);
  else if (nv <= 3) SKM_TAU_KEPT(3);
  else if (nv <= 4) SKM_TAU_KEPT(4);
  else if (nv <= 6) SKM_TAU_KEPT(6);
  else SKM_TAU_KEPT(8);
#undef SKM_TAU_KEPT
  return hipGetLastError();
}

// touched[c] = 1 for the clusters that the m labels name, 0 for the others (one workgroup: the two passes are ordered)
__global__ void __launch_bounds__(1024) mark_touched_kernel(const int32_t *labels, int m, int32_t k, uint32_t *touched) {
  for (int c = threadIdx.x; c < k; c += 1024) touched[c] = 0u;
  __syncthreads();
  for (int e = threadIdx.x; e < m; e += 1024) touched[labels[e]] = 1u;
}
hipError_t launch_mark_touched(const int32_t *labels, int32_t m, int32_t k, uint32_t *touched, hipStream_t st) {
  hipLaunchKernelGGL(mark_touched_kernel, dim3(1), dim3(1024), 0, st, labels, m, k, touched);
  return hipGetLastError();
}

// dst[idx[p]] = src[p] (4-byte items): per-point results back from a regrouped order to the caller's
__global__ void scatter_by_index_kernel(const uint32_t *src, const int32_t *idx, int64_t n, uint32_t *dst) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) dst[idx[p]] = src[p];
}
hipError_t launch_scatter_by_index(const void *src, const int32_t *idx, int64_t n, void *dst, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, (int64_t)num_cus() * 16);
  hipLaunchKernelGGL(scatter_by_index_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const uint32_t *)src, idx, n,
                     (uint32_t *)dst);
  return hipGetLastError();
}

// Sub-order of the points inside a cluster for the regrouping.  key[i] = the signs of the first four (rotated)
// dimensions of point i: four random hyperplanes through the origin cut every cluster into up to 16 pieces that are
// compact in space, and points of one piece share their challengers more than points of the whole cluster do.
__global__ void sign_key_kernel(const float *Xr, int64_t ldx, int64_t n, unsigned char *key) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float4 v = *reinterpret_cast<const float4 *>(Xr + i * ldx);
    key[i] = (unsigned char)((v.x > 0.f) | ((v.y > 0.f) << 1) | ((v.z > 0.f) << 2) | ((v.w > 0.f) << 3));
  }
}
// order_out = order_in with every cluster's segment [off[c], off[c+1]) stably sorted by key (16 values): one
// workgroup per cluster, thread t takes the t-th contiguous part of the segment, so that the order inside a key is kept.
__global__ void __launch_bounds__(256) suborder_kernel(const int32_t *off, const int32_t *order_in, const unsigned char *key,
                                                       int32_t *order_out) {
  __shared__ int s_cnt[16][256];   // [key][thread]: count, then first output slot
  __shared__ int s_tot[16];
  const int c = blockIdx.x, t = threadIdx.x;
  const int lo = off[c], len = off[c + 1] - lo;
  const int part = (len + 255) / 256;
  const int p0 = min(t * part, len), p1 = min(p0 + part, len);
  for (int b = 0; b < 16; ++b) s_cnt[b][t] = 0;
  for (int p = p0; p < p1; ++p) s_cnt[key[order_in[lo + p]]][t] += 1;
  __syncthreads();
  if (t < 16) {   // exclusive scan of this key's counts over the threads
    int run = 0;
    for (int u = 0; u < 256; ++u) {
      const int v = s_cnt[t][u];
      s_cnt[t][u] = run;
      run += v;
    }
    s_tot[t] = run;
  }
  __syncthreads();
  if (t == 0) {   // first slot of every key
    int run = 0;
    for (int b = 0; b < 16; ++b) {
      const int v = s_tot[b];
      s_tot[b] = run;
      run += v;
    }
  }
  __syncthreads();
  for (int p = p0; p < p1; ++p) {
    const int id = order_in[lo + p];
    const int b = key[id];
    order_out[lo + s_tot[b] + s_cnt[b][t]] = id;
    s_cnt[b][t] += 1;
  }
}
hipError_t launch_suborder(const float *Xr, int64_t ldx, int64_t n, int32_t k, const int32_t *off, const int32_t *order_in,
                           unsigned char *key_scratch, int32_t *order_out, hipStream_t st) {
  if (n <= 0 || k <= 0) return hipSuccess;
  if ((reinterpret_cast<uintptr_t>(Xr) & 15u) || ldx % 4 != 0) return hipErrorInvalidValue;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, (int64_t)num_cus() * 16);
  hipLaunchKernelGGL(sign_key_kernel, dim3((unsigned)blocks), dim3(256), 0, st, Xr, ldx, n, key_scratch);
  hipLaunchKernelGGL(suborder_kernel, dim3((unsigned)k), dim3(256), 0, st, off, order_in, (const unsigned char *)key_scratch,
                     order_out);
  return hipGetLastError();
}

// out[p] = a[b[p]]
__global__ void compose_kernel(const int32_t *a, const int32_t *b, int64_t n, int32_t *out) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) out[p] = a[b[p]];
}
hipError_t launch_compose(const int32_t *a, const int32_t *b, int64_t n, int32_t *out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, (int64_t)num_cus() * 16);
  hipLaunchKernelGGL(compose_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a, b, n, out);
  return hipGetLastError();
}

// inv[perm[p]] = p, then the point id in the low half of every key replaced by its position (keys of ~0 stay)
__global__ void invert_permutation_kernel(const int32_t *perm, int64_t n, int32_t *inv) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) inv[perm[p]] = (int32_t)p;
}
__global__ void remap_key_ids_kernel(unsigned long long *keys, int64_t m, const int32_t *inv, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
    const unsigned long long key = keys[e];
    const unsigned long long id = key & 0xffffffffull;
    if (key != ~0ull && (int64_t)id < n) keys[e] = (key & ~0xffffffffull) | (unsigned long long)(unsigned int)inv[id];
  }
}
hipError_t launch_remap_key_ids(unsigned long long *keys, int64_t m, const int32_t *perm, int64_t n, int32_t *inv_scratch,
                                hipStream_t st) {
  if (n <= 0 || m <= 0) return hipSuccess;
  const int64_t b1 = std::min<int64_t>((n + 255) / 256, (int64_t)num_cus() * 16);
  hipLaunchKernelGGL(invert_permutation_kernel, dim3((unsigned)b1), dim3(256), 0, st, perm, n, inv_scratch);
  const int64_t b2 = std::min<int64_t>((m + 255) / 256, (int64_t)num_cus() * 16);
  hipLaunchKernelGGL(remap_key_ids_kernel, dim3((unsigned)b2), dim3(256), 0, st, keys, m, (const int32_t *)inv_scratch, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------ centroid preparation
// Everything a step needs from the centroids in one pass over them, one workgroup per centroid, a float4 per thread:
// prefix norms at the checkpoints (ynp) or over dims [0, dn) (ynorm), the trailing dims from dprime on copied to
// Ypdx[m][c][0..63] (block m = dims dprime + 64 m .., zero filled past the row), and the split-fp16 copy of the row with
// its plane of hi halves (layouts of launch_split_rows).  The same launch carries the step's two small host-side jobs:
// it clears the words that the step counts into and writes the theta ratios, which arrive as kernel arguments.  A small
// step is a chain of launches of a few microseconds each, and a memset or a copy from the host costs three launches:
// with all five in one, a pruned step of 20 000 x 128 points against 100 centroids issues four commands fewer.
// The order in which a norm's squares are added is part of the results (see unit_three in progressive.hip): for ynp the
// dimensions of a piece of 16 and then the pieces, one after the other; for ynorm thread t adds the dimensions t, t + 256, ..
// and the threads' sums are added pairwise.
__device__ inline void prep_centroid(const CentroidPrep &a, const ThetaRatios &ratios, int c) {
  __shared__ float s_piece[1024];   // ||y[16 p : 16 p + 16)||^2 at p (ds <= 16384)
  __shared__ float s_red[4];
  const int tid = threadIdx.x;
  for (int64_t w = (int64_t)c * 256 + tid; w < a.clear_words; w += (int64_t)a.k * 256) a.clear[w] = 0u;
  if (c == 0 && a.ratio_out)
    for (int m = tid; m < ratios.n; m += 256) a.ratio_out[m] = ratios.v[m];
  const float *y = a.Y + (int64_t)c * a.ldy;
  PrefixOut po{nullptr, a.k, a.ds, a.Ys, a.Yh, nullptr, 0.f, nullptr, nullptr, nullptr};
  if (a.Ys) {
    po.scale = split_scale(*a.y_absmax);
    po.hi_dims = a.hi_dims;
    po.xd = a.Yd;
    po.xd_from = a.dprime;
    if (tid < 64) emit_split_pads(po, c, tid);
  }
  const int pdx_end = a.Ypdx ? a.dprime + a.nb * kBlockDims : 0;   // columns up to here have a place in Ypdx
  const int cend = a.ds > pdx_end ? a.ds : pdx_end;
  for (int c0 = 0; c0 < cend; c0 += 1024) {
    const int col = c0 + 4 * tid;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (col < a.ds) v = *reinterpret_cast<const float4 *>(y + col);
    if (a.ynp) {
      // the 16 squares of a piece one after the other, handed from lane to lane of its quad: lane 3 ends with all of them
      float q = 0.f;
#pragma unroll
      for (int l = 0; l < 4; ++l) {
        if (l > 0) q = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, q), 0x90, 0xF, 0xF, true));   // quad_perm [0,0,1,2]
        q = fmaf(v.w, v.w, fmaf(v.z, v.z, fmaf(v.y, v.y, fmaf(v.x, v.x, q))));
      }
      if ((tid & 3) == 3 && col < a.ds) s_piece[col >> 4] = q;
    }
    if (col < a.ds && a.Ys) emit_split(po, c, col, v);
    if (col >= a.dprime && col < pdx_end) {
      const int t = col - a.dprime;
      if (col >= a.pdx_cols) v = make_float4(0.f, 0.f, 0.f, 0.f);
      *reinterpret_cast<float4 *>(a.Ypdx + ((int64_t)(t / kBlockDims) * a.k + c) * kBlockDims + t % kBlockDims) = v;
    }
  }
  if (a.ynorm) {
    float s = 0.f;
    for (int j = tid; j < a.dn; j += 256) s = fmaf(y[j], y[j], s);
    s = wave_sum(s);
    if ((tid & 63) == 0) s_red[tid >> 6] = s;
  }
  __syncthreads();
  if (a.ynorm && tid == 0) a.ynorm[c] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
  if (a.ynp)
    for (int m = tid; m <= a.nb; m += 256) {
      const int np = (m == a.nb ? a.ds : min(a.ds, a.dprime + kBlockDims * m)) >> 4;
      float acc = 0.f;
#pragma unroll 8
      for (int p = 0; p < np; ++p) acc += s_piece[p];   // (in order, whatever d' is)
      a.ynp[(int64_t)m * a.k + c] = acc;
    }
}

__global__ void __launch_bounds__(256) prep_centroids_kernel(CentroidPrep a, ThetaRatios ratios) {
  put_stamp(a.stamp);
  prep_centroid(a, ratios, blockIdx.x);
}
// The same with the thresholds of short rows beside it: both wait for the centroids only.  A launch less in every step: a fit of
// 20 000 x 128 into 100 clusters, eleven steps, 856 -> 834 us, of 120 001 x 200 2212 -> 2206.
template <int H>
__global__ void __launch_bounds__(256) prep_thresholds_kernel(CentroidPrep a, ThetaRatios ratios, ShortThresholds t) {
  put_stamp(a.stamp);
  if ((int)blockIdx.x < a.k) prep_centroid(a, ratios, blockIdx.x);
  else tau_short<H>(t.Xr, t.ldx, t.n, a.ds, a.Y, a.ldy, t.labels, t.tau, t.best, nullptr, nullptr, blockIdx.x - a.k, gridDim.x - a.k);
}

hipError_t launch_prep_centroids(const CentroidPrep &a, hipStream_t st, const float *ratio, int nratio, const ShortThresholds *t) {
  if (a.k <= 0) return hipSuccess;
  if (a.ds % 16 != 0 || a.ds > 16384 || a.ldy % 4 != 0 || (reinterpret_cast<uintptr_t>(a.Y) & 15u) || a.dn % 16 != 0 ||
      a.dn > a.ds || a.dprime % 16 != 0 || (a.Ys && !a.y_absmax) || (a.Yh && !a.Ys) || (a.Yd && !a.Ys) || (a.Yh && a.hi_dims <= 0) || nratio > kMaxBlocks + 1 ||
      (a.ratio_out != nullptr) != (nratio > 0))
    return hipErrorInvalidValue;
  ThetaRatios r;
  r.n = nratio;
  for (int m = 0; m < nratio; ++m) r.v[m] = ratio[m];
  if (t) {
    if (a.ds > 256 || !t->labels || t->n <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(a.ds <= 128 ? prep_thresholds_kernel<1> : prep_thresholds_kernel<2>, dim3((unsigned)a.k + tau_short_grid(t->n)), dim3(256), 0, st,
                       a, r, *t);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(prep_centroids_kernel, dim3(a.k), dim3(256), 0, st, a, r);
  return hipGetLastError();
}

// ------------------------------------------------------------------ fills
template <typename T>
__global__ void fill_kernel(T *p, int64_t n, T v, stamp_t *stamp) {
  put_stamp(stamp);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}
template <typename T>
static hipError_t launch_fill(T *p, int64_t n, T v, hipStream_t st, stamp_t *stamp = nullptr) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(fill_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v, stamp);
  return hipGetLastError();
}
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t st) {
  return launch_fill<unsigned long long>(p, n, v, st);
}
hipError_t launch_fill_u32(unsigned int *p, int64_t n, unsigned int v, hipStream_t st, stamp_t *stamp) {
  return launch_fill<unsigned int>(p, n, v, st, stamp);
}
__global__ void stamp_kernel(stamp_t *stamp) { put_stamp(stamp); }
hipError_t launch_stamp(stamp_t *stamp, hipStream_t st) {
  if (!stamp) return hipSuccess;
  hipLaunchKernelGGL(stamp_kernel, dim3(1), dim3(64), 0, st, stamp);
  return hipGetLastError();
}

// ------------------------------------------------------------------ largest magnitude of a matrix
// Non-negative floats order like their bit patterns, so the maximum is kept with an unsigned atomicMax.
// max |v| over a workgroup of 256 threads into *out (bit pattern, unsigned order): one atomic per workgroup, and
// only if it would raise the word that thousands of workgroups share
__device__ inline void block_absmax(float v, unsigned int *out) {
  __shared__ unsigned int s_m[4];
  float m = fabsf(v);
#pragma unroll
  for (int w = 1; w < 64; w <<= 1) m = fmaxf(m, __shfl_xor(m, w, 64));
  if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = __builtin_bit_cast(unsigned int, m);
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned int mb = max(max(s_m[0], s_m[1]), max(s_m[2], s_m[3]));
    if (mb > __atomic_load_n(out, __ATOMIC_RELAXED)) atomicMax(out, mb);
  }
}

// Rows without gaps (lda == cols) are read as one array of at least four values, 16 bytes a load whatever its alignment (global loads
// need 4 bytes; 46 467 x 495 a value at a time: 70 us, now 16), four loads in flight.  A kernel by itself: behind the code for rows
// with gaps a small array took 6.4 us instead of 4.5, most of it for the instructions.
template <int LOADS>   // in flight
__device__ inline void absmax_flat(const float *A, int64_t count, unsigned int *out, int block, int nblocks) {
  const int64_t last = count - 4, stride = (int64_t)nblocks * 256 * LOADS;
  float m = 0.f;
  for (int64_t e = (int64_t)block * 256 * LOADS + threadIdx.x; 4 * e < count; e += stride) {
    f32x4_u v[LOADS];
#pragma unroll
    for (int u = 0; u < LOADS; ++u) v[u] = *reinterpret_cast<const f32x4_u *>(A + min(4 * (e + 256 * u), last));   // (past the end: the last four again)
#pragma unroll
    for (int u = 0; u < LOADS; ++u) m = fmaxf(m, fmaxf(fmaxf(fabsf(v[u].x), fabsf(v[u].y)), fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
  }
  block_absmax(m, out);
}
__global__ void __launch_bounds__(256) absmax_flat_kernel(const float *A, int64_t count, unsigned int *out) {
  absmax_flat<4>(A, count, out, blockIdx.x, gridDim.x);
}
// Rows with gaps: an element index is split into row and column.
template <bool VEC4>
__global__ void __launch_bounds__(256) absmax_kernel(const float *A, int64_t lda, int64_t rows, int32_t cols,
                                                     unsigned int *out) {
  const int64_t per_row = VEC4 ? cols / 4 : cols;
  const int64_t total = rows * per_row;
  float m = 0.f;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e / per_row;
    const float *at = A + r * lda + (e - r * per_row) * (VEC4 ? 4 : 1);
    if (VEC4) {
      const float4 v = *reinterpret_cast<const float4 *>(at);
      m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    } else {
      m = fmaxf(m, fabsf(*at));
    }
  }
  block_absmax(m, out);
}

hipError_t launch_absmax(const float *A, int64_t lda, int64_t rows, int32_t cols, unsigned int *out, hipStream_t st,
                         int max_blocks) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  const bool vec = (reinterpret_cast<uintptr_t>(A) & 15u) == 0 && lda % 4 == 0 && cols % 4 == 0;
  const bool flat = lda == cols && rows * (int64_t)cols >= 4;
  const int64_t work = vec || flat ? (rows * (int64_t)cols + 3) / 4 : rows * (int64_t)cols;
  // At least four elements per thread where there are that many, and two workgroups per CU at most: that keeps enough
  // loads in flight, and the atomics at the one result word, 10 ns each, stay few (4096 workgroups: 40 us for 20 000 x 1536).
  const unsigned blocks = (unsigned)std::min<int64_t>((work + 1023) / 1024, max_blocks > 0 ? max_blocks : 2 * num_cus());
  if (flat) hipLaunchKernelGGL(absmax_flat_kernel, dim3(blocks), dim3(256), 0, st, A, rows * (int64_t)cols, out);
  else if (vec) hipLaunchKernelGGL(absmax_kernel<true>, dim3(blocks), dim3(256), 0, st, A, lda, rows, cols, out);
  else hipLaunchKernelGGL(absmax_kernel<false>, dim3(blocks), dim3(256), 0, st, A, lda, rows, cols, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ unit-length rows (angular metric)
// One wavefront per row: sum of squares in fp32 over float4 loads, then the row is scaled in place.
// Rows of zeros are left alone.  absmax (optional): the largest magnitude of the scaled rows.
__global__ void __launch_bounds__(256) normalize_rows_kernel(float *A, int64_t lda, int64_t rows, int32_t cols,
                                                             unsigned int *absmax) {
  const int lane = threadIdx.x & 63;
  float m = 0.f;
  for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += (int64_t)gridDim.x * 4) {
    float *row = A + r * lda;
    float s = 0.f;
    for (int c = 4 * lane; c < cols; c += 256) {
      const float4 v = *reinterpret_cast<const float4 *>(row + c);
      s = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, fmaf(v.w, v.w, s))));
    }
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) s += __shfl_xor(s, w, 64);
    if (!(s > 0.f)) continue;
    const float inv = 1.0f / sqrtf(s);
    for (int c = 4 * lane; c < cols; c += 256) {
      float4 v = *reinterpret_cast<const float4 *>(row + c);
      v.x *= inv; v.y *= inv; v.z *= inv; v.w *= inv;
      m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
      *reinterpret_cast<float4 *>(row + c) = v;
    }
  }
  if (absmax) block_absmax(m, absmax);
}

// cols and lda multiples of 4, A 16-byte aligned (the padded buffers of the library)
hipError_t launch_normalize_rows(float *A, int64_t lda, int64_t rows, int32_t cols, hipStream_t st, unsigned int *absmax) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if ((reinterpret_cast<uintptr_t>(A) & 15u) || lda % 4 || cols % 4) return hipErrorInvalidValue;
  const int64_t blocks = std::min<int64_t>((rows + 3) / 4, (int64_t)num_cus() * 32);
  hipLaunchKernelGGL(normalize_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st, A, lda, rows, cols, absmax);
  return hipGetLastError();
}

// ------------------------------------------------------------------ argmin unpack
// A workgroup takes 8192 consecutive points.  The cluster sizes are counted in LDS first when the k counters fit
// (k <= FIN_LDS_BINS) and flushed once per workgroup: a million atomic increments on the 64 cache lines that hold 1024
// counters took 0.2 ms per step; larger k spreads them over more lines and goes to memory directly.
// (1024 threads share them: with 256 the loads of a workgroup were one long chain, 46 us a million points, 24 us.)
// Small inputs (one small fit of many, as in the hierarchical fit) take 1024 points per workgroup instead: the
// launch is then a few workgroups side by side rather than one long loop.  They count in LDS as well where a cluster
// holds more than a handful of the points (direct increments of 20 000 points on 100 counters: 54 us, in LDS: 5 us).
// Where *flag is set before the launch, labels and distances are left as they are (the caller's arrays of a refused call).
// The last workgroup to finish closes the step: it adds the objective's partials and the counter replicas in a fixed
// order, takes the number of empty clusters and the largest size, turns the per-workgroup counts of changed points into
// starts (for the incremental update), and writes the step's report straight into page-locked host memory.
// It is bound by latency, a chain of reads from memory: 20 000 points 10.0 -> 6.6 us, 120 000 12.0 -> 8.2, a million 21.9 ->
// 18.8 since every thread asks for all it needs at once, both of its points and of the closing.
constexpr int FIN_LDS_BINS = 8192;
static int finalize_per_block(int64_t n) { return n >= (int64_t)1 << 18 ? 8192 : 1024; }
int64_t finalize_blocks(int64_t n) { return (n + finalize_per_block(n) - 1) / finalize_per_block(n); }

template <typename T>
__device__ inline T load_agent(const T *p) {   // a value that other workgroups of this launch have written
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline void store_system(T *p, T v) {   // a value for the host: written through
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int FIN_THREADS, int PER>
__global__ void __launch_bounds__(FIN_THREADS) finalize_assign_kernel(FinalizeArgs a, int in_lds) {
  __shared__ double red[FIN_THREADS];
  constexpr int NW = FIN_THREADS / 64;
  __shared__ unsigned int redc[NW];
  __shared__ int s_hist[FIN_LDS_BINS];
  __shared__ int s_last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  put_stamp(a.stamp);
  // All of a thread's points are asked for before the first is looked at (with the loads in the loop below, behind its
  // atomics and stores, each turn waited for memory by itself).
  const int64_t base = (int64_t)blockIdx.x * (FIN_THREADS * PER);
  const int mine = (int)min((int64_t)(FIN_THREADS * PER), a.n - base);
  unsigned long long keys[PER];
  int32_t before[PER];
  // (flags of the kernels before this one: a label out of range, a list that ran over)
  const unsigned int flag_in = a.flag ? load_agent(a.flag) : 0u;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t i = base + min(u * FIN_THREADS + tid, mine - 1);
    keys[u] = a.best[i];
    before[u] = a.prev ? a.prev[i] : 0;
  }
  if (in_lds) {
    for (int b = tid; b < a.k; b += FIN_THREADS) s_hist[b] = 0;
    __syncthreads();
  }
  const bool refused = flag_in != 0u;
  double s = 0.0;
  unsigned int ch = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int t = u * FIN_THREADS + tid;
    if (t < mine) {
      const int64_t i = base + t;
      const unsigned long long key = keys[u];
      int32_t l = (int32_t)(key & 0xffffffffull);
      float dv = ord2f((uint32_t)(key >> 32));
      if (key == ~0ull) {   // a point no kernel offered a centroid for: reported through `flag`, kept in range
        l = 0;
        dv = 0.f;
        if (a.flag) atomicOr(a.flag, 2u);   // bit 1: unset point (bit 0 is the hand-over list's overflow)
      }
      if (!refused) {
        a.assign[i] = l;
        if (a.dist) a.dist[i] = dv;
      }
      if (in_lds) atomicAdd(&s_hist[l], 1);
      else if (a.cnt) atomicAdd(a.cnt + l, 1);
      if (a.prev) ch += (before[u] != l);
      s += (double)dv;
    }
  }
  s = wave_sum(s);
  for (int m = 1; m < 64; m <<= 1) ch += __shfl_xor(ch, m, 64);
  if (lane == 0) {
    red[wave] = s;
    redc[wave] = ch;
  }
  __syncthreads();
  if (in_lds) {   // (the barrier above has ordered the LDS increments before these reads)
    for (int b = tid; b < a.k; b += FIN_THREADS) {
      const int v = s_hist[b];
      if (v) atomicAdd(a.cnt + b, v);
    }
  }
  if (!a.done) return;
  if (tid == 0) {
    double t = 0.0;
    unsigned int c = 0;
    for (int u = 0; u < NW; u += 4) {
      t += (red[u] + red[u + 1]) + (red[u + 2] + red[u + 3]);
      c += (redc[u] + redc[u + 1]) + (redc[u + 2] + redc[u + 3]);
    }
    __hip_atomic_store(a.obj_partial + blockIdx.x, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.change_start + blockIdx.x, (int)c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // ---- the last workgroup closes the step.  What it reads of the others are agent-scope atomics (sizes, flag, partials,
  // counters): they have been performed once they are no longer outstanding, so a wait orders them before the ticket.  (A
  // release fence would write the caches' dirty lines back first, the eight megabytes of labels and distances among
  // them: 50 us a million points, 28 us.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) s_last = __hip_atomic_fetch_add(a.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  __syncthreads();
  if (!s_last) return;
  // The closing is one chain of dependent reads, so everything it reads is asked for together: the partials, the first
  // sizes, and the counters, whose replicas eight lanes share.  (Read where each is used, with tree and scan over
  // barriers, the closing alone was some 5 us.)
  const int nblk = gridDim.x;
  constexpr int CNT_AHEAD = 4, QL = 8, QR = kStatReplicas / QL;
  const int per = (nblk + FIN_THREADS - 1) / FIN_THREADS;
  const int lo = min(tid * per, nblk), hi = min(lo + per, nblk);
  const int lo_c = min(lo, nblk - 1);
  const unsigned int flag_out = load_agent(a.flag);
  const double first_part = load_agent(a.obj_partial + lo_c);
  const int first_changed = load_agent(a.change_start + lo_c);
  unsigned long long sc[QR];
  {
    const int q = min(tid / QL, a.nscal - 1);
#pragma unroll
    for (int j = 0; j < QR; ++j) sc[j] = load_agent(a.scal + (size_t)((tid & (QL - 1)) + QL * j) * SC_COUNT + q);
  }
  int size[CNT_AHEAD];
  if (a.cnt) {
#pragma unroll
    for (int u = 0; u < CNT_AHEAD; ++u) size[u] = load_agent(a.cnt + min(u * FIN_THREADS + tid, a.k - 1));
  }
  // objective: thread t adds the t-th contiguous part, the parts are added pairwise (stride halved each time); changed
  // points: the same parts scanned, every workgroup's count becomes the number of changed points before it
  {
    double t = 0.0;
    int part = 0;
    if (lo < hi) {
      t += first_part;
      part += first_changed;
    }
    for (int i = lo + 1; i < hi; ++i) {
      t += load_agent(a.obj_partial + i);
      part += load_agent(a.change_start + i);
    }
    red[tid] = t;
    int run = part;   // inclusive scan of the wavefront
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(run, o, 64);
      if (lane >= o) run += v;
    }
    if (lane == 63) redc[wave] = (unsigned int)run;
    __syncthreads();
    run -= part;
    for (int w = 0; w < NW; ++w)
      if (w < wave) run += (int)redc[w];
    for (int i = lo; i < hi; ++i) {
      const int v = i == lo ? first_changed : load_agent(a.change_start + i);
      a.change_start[i] = run;
      run += v;
    }
  }
  StepReport *r = a.report;
  for (int q0 = 0; q0 < a.nscal; q0 += FIN_THREADS / QL) {   // (one turn up to 32 scalars, 128 where PER is 8)
    const int q = q0 + tid / QL;
    if (q0) {
      const int qc = min(q, a.nscal - 1);
#pragma unroll
      for (int j = 0; j < QR; ++j) sc[j] = load_agent(a.scal + (size_t)((tid & (QL - 1)) + QL * j) * SC_COUNT + qc);
    }
    unsigned long long v = 0;
#pragma unroll
    for (int j = 0; j < QR; ++j) v += sc[j];
#pragma unroll
    for (int m = 1; m < QL; m <<= 1) v += __shfl_xor(v, m, 64);
    if ((tid & (QL - 1)) == 0 && q < a.nscal && q != SC_CHANGED) store_system(&r->scal[q], v);
  }
  int empty = 0, largest = 0;
  if (a.cnt) {
#pragma unroll
    for (int u = 0; u < CNT_AHEAD; ++u)
      if (u * FIN_THREADS + tid < a.k) {
        empty += size[u] == 0;
        largest = max(largest, size[u]);
      }
    for (int b = CNT_AHEAD * FIN_THREADS + tid; b < a.k; b += FIN_THREADS) {
      const int v = load_agent(a.cnt + b);
      empty += v == 0;
      largest = max(largest, v);
    }
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    empty += __shfl_xor(empty, m, 64);
    largest = max(largest, __shfl_xor(largest, m, 64));
  }
  if (lane == 0) {   // (nothing reads s_hist any more: the last read was before the ticket)
    s_hist[wave] = empty;
    s_hist[NW + wave] = largest;
  }
  double parts[NW];   // the tree over `red`: wavefront 0 holds NW values a lane (its barrier was the scan's)
#pragma unroll
  for (int u = 0; u < NW; ++u) parts[u] = red[u * 64 + lane];
#pragma unroll
  for (int w = NW / 2; w > 0; w >>= 1)
#pragma unroll
    for (int u = 0; u < w; ++u) parts[u] += parts[u + w];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) parts[0] += __shfl_down(parts[0], o, 64);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the counters have arrived: the host may take seq for all of the report)
  __syncthreads();
  if (tid == 0) {
    store_system(&r->objective, parts[0]);
    store_system(&r->flag, flag_out);
    int e = 0, l = 0;
    unsigned int changed = 0;
    for (int u = 0; u < NW; ++u) {
      e += s_hist[u];
      l = max(l, s_hist[NW + u]);
      changed += redc[u];
    }
    store_system(&r->nempty, e);
    store_system(&r->largest, l);
    if (a.nscal > SC_CHANGED) store_system(&r->scal[SC_CHANGED], (unsigned long long)changed);
    a.scal[SC_CHANGED] = (unsigned long long)changed;   // (no other kernel of the step writes it)
    if (a.stamp_end) *a.stamp_end = wall_clock64();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    store_system(&r->seq, a.seq);
  }
}

hipError_t launch_finalize_assign(const FinalizeArgs &a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  if (a.done && (!a.obj_partial || !a.change_start || !a.scal || !a.report || !a.flag)) return hipErrorInvalidValue;
  const int per_block = finalize_per_block(a.n);
  const int in_lds = a.cnt && a.k <= FIN_LDS_BINS && (per_block > 1024 || a.n >= 8 * (int64_t)a.k);
  if (per_block > 1024)
    hipLaunchKernelGGL((finalize_assign_kernel<1024, 8>), dim3((unsigned)finalize_blocks(a.n)), dim3(1024), 0, st, a, in_lds);
  else
    hipLaunchKernelGGL((finalize_assign_kernel<256, 4>), dim3((unsigned)finalize_blocks(a.n)), dim3(256), 0, st, a, in_lds);
  return hipGetLastError();
}

// Counting by label.  Where a label holds several of the points, a workgroup counts its points in LDS first: a million
// returning atomics on the few cache lines that hold 1024 counters took 0.2 ms, with one atomic per (workgroup, label)
// 0.02 ms.  Labels outside [0, k) are left out and set bit 2 of *flag (if given).
constexpr int CNT_THREADS = 512;
constexpr int CNT_LDS_BINS = 8192;
static int count_per_block(int64_t n) { return n >= (int64_t)1 << 18 ? 8192 : 1024; }
static bool count_in_lds(int64_t n, int32_t k) { return k <= CNT_LDS_BINS && n >= 8 * (int64_t)k; }

__global__ void __launch_bounds__(CNT_THREADS) histogram_kernel(const int32_t *assign, int64_t n, int32_t k, int32_t *cnt,
                                                                unsigned int *flag, int per_block, int in_lds) {
  extern __shared__ int s_bins[];
  if (in_lds) {
    for (int b = threadIdx.x; b < k; b += CNT_THREADS) s_bins[b] = 0;
    __syncthreads();
  }
  const int64_t base = (int64_t)blockIdx.x * per_block;
  for (int t = threadIdx.x; t < per_block; t += CNT_THREADS) {
    const int64_t i = base + t;
    if (i >= n) break;
    const int a = assign[i];
    if ((unsigned int)a >= (unsigned int)k) {
      if (flag) atomicOr(flag, 4u);
    } else {
      atomicAdd(in_lds ? s_bins + a : cnt + a, 1);
    }
  }
  if (!in_lds) return;
  __syncthreads();
  for (int b = threadIdx.x; b < k; b += CNT_THREADS) {
    const int v = s_bins[b];
    if (v) atomicAdd(cnt + b, v);
  }
}
hipError_t launch_histogram(const int32_t *assign, int64_t n, int32_t k, int32_t *cnt, unsigned int *flag, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int per = count_per_block(n);
  const int in_lds = count_in_lds(n, k);
  hipLaunchKernelGGL(histogram_kernel, dim3((unsigned)((n + per - 1) / per)), dim3(CNT_THREADS),
                     in_lds ? (size_t)k * sizeof(int) : 0, st, assign, n, k, cnt, flag, per, in_lds);
  return hipGetLastError();
}

// out[i] = a[i] where that is a label in [0, k); any other becomes 0 and sets bit 2 of *flag (the caller's labels are
// checked and copied in one pass: nothing behind it indexes with an unchecked label)
__global__ void copy_labels_kernel(const int32_t *a, int64_t n, int32_t k, int32_t *out, unsigned int *flag) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int32_t v = a[i];
    if (v < 0 || v >= k) {
      v = 0;
      atomicOr(flag, 4u);
    }
    out[i] = v;
  }
}
hipError_t launch_copy_labels(const int32_t *a, int64_t n, int32_t k, int32_t *out, unsigned int *flag, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(copy_labels_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a, n, k, out, flag);
  return hipGetLastError();
}

// ------------------------------------------------------------------ centroid update
int64_t update_max_segments(int64_t n, int32_t k) { return (int64_t)k + n / kSegPoints + 1; }

// single workgroup: exclusive scans of the cluster sizes and of the segment counts.  Thread t takes the t-th contiguous
// part; one scan over the parts (k = 32 768: 122 us with a scan per 1024 sizes, 14 us).  Also clears the word that the
// means' largest magnitude is folded into later (zero, optional).
__global__ void __launch_bounds__(1024) scan_counts_kernel(const int32_t *cnt, int32_t k, int32_t *off, int32_t *cursor,
                                                           int32_t *segoff, unsigned int *zero) {
  __shared__ int s_a[16], s_b[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (zero && tid == 0) *zero = 0u;
  const int per = (k + 1023) / 1024;
  const int lo = min(tid * per, k), hi = min(lo + per, k);
  int va = 0, vb = 0;
  for (int c = lo; c < hi; ++c) {
    const int v = cnt[c];
    va += v;
    vb += (v + kSegPoints - 1) / kSegPoints;
  }
  int ia = va, ib = vb;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int ta = __shfl_up(ia, o, 64), tb = __shfl_up(ib, o, 64);
    if (lane >= o) { ia += ta; ib += tb; }
  }
  if (lane == 63) { s_a[wave] = ia; s_b[wave] = ib; }
  __syncthreads();
  int ra = ia - va, rb = ib - vb;
  for (int w = 0; w < wave; ++w) { ra += s_a[w]; rb += s_b[w]; }
  for (int c = lo; c < hi; ++c) {
    const int v = cnt[c];
    off[c] = ra;
    segoff[c] = rb;
    cursor[c] = 0;
    ra += v;
    rb += (v + kSegPoints - 1) / kSegPoints;
  }
  if (tid == 1023) { off[k] = ra; segoff[k] = rb; }
}

// order[...] = i (or ids[i] when the labelled items are a list of ids), grouped by label.  With the counters in LDS a
// workgroup takes the rank of each of its items among its own, reserves one range per label it holds, and writes (80 to
// 217 us for a million points with a returning atomic per point, 20 us).  Items with a label outside [0, k) are skipped.
constexpr int CNT_ITEMS = 8192 / CNT_THREADS;
__global__ void __launch_bounds__(CNT_THREADS) scatter_order_kernel(const int32_t *assign, int64_t n, int32_t k,
                                                                    const int32_t *off, int32_t *cursor, int32_t *order,
                                                                    const int32_t *ids, int per_block, int in_lds) {
  extern __shared__ int s_bins[];
  const int64_t base = (int64_t)blockIdx.x * per_block;
  if (!in_lds) {
    for (int t = threadIdx.x; t < per_block; t += CNT_THREADS) {
      const int64_t i = base + t;
      if (i >= n) break;
      const int a = assign[i];
      if ((unsigned int)a >= (unsigned int)k) continue;
      order[off[a] + atomicAdd(cursor + a, 1)] = ids ? ids[i] : (int32_t)i;
    }
    return;
  }
  for (int b = threadIdx.x; b < k; b += CNT_THREADS) s_bins[b] = 0;
  __syncthreads();
  int lab[CNT_ITEMS], rank[CNT_ITEMS];
#pragma unroll
  for (int j = 0; j < CNT_ITEMS; ++j) {
    const int t = j * CNT_THREADS + threadIdx.x;
    const int64_t i = base + t;
    lab[j] = -1;
    rank[j] = 0;
    if (t < per_block && i < n) {
      const int a = assign[i];
      if ((unsigned int)a < (unsigned int)k) {
        lab[j] = a;
        rank[j] = atomicAdd(s_bins + a, 1);
      }
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < k; b += CNT_THREADS) {
    const int v = s_bins[b];
    if (v) s_bins[b] = off[b] + atomicAdd(cursor + b, v);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < CNT_ITEMS; ++j)
    if (lab[j] >= 0) {
      const int64_t i = base + j * CNT_THREADS + threadIdx.x;
      order[s_bins[lab[j]] + rank[j]] = ids ? ids[i] : (int32_t)i;
    }
}
static void launch_scatter_order(const int32_t *assign, int64_t n, int32_t k, const int32_t *off, int32_t *cursor,
                                 int32_t *order, const int32_t *ids, hipStream_t st) {
  const int per = count_per_block(n);
  const int in_lds = count_in_lds(n, k);
  hipLaunchKernelGGL(scatter_order_kernel, dim3((unsigned)((n + per - 1) / per)), dim3(CNT_THREADS),
                     in_lds ? (size_t)k * sizeof(int) : 0, st, assign, n, k, off, cursor, order, ids, per, in_lds);
}

// The same grouping with the members of every label in ascending order, without atomics and without a sort: the
// workgroups' label counts become starts (rank_base_kernel: for every label, over the workgroups in order), and a
// workgroup places its points stably.  Its wavefronts own contiguous eighths of its range and count them first, so each
// knows where its own members of a label start; it then walks its points 64 at a time, the lanes of one label finding
// each other by one ballot per label bit.  Grouping a million points by 4096 labels: 17 (scatter) + 84 (ordering the
// groups) us before, 40 us in all; by 1024 labels 11 + 200 us, 38 us.  For up to kStableLabels labels (the wavefronts'
// counters fill the LDS) and not for a label range larger than the point set, where the count matrix would be the work.
constexpr int STB_THREADS = 512, STB_WAVES = STB_THREADS / 64;
constexpr int32_t kStableLabels = 8192;
static int stable_per_block(int64_t n) { return n >= (int64_t)1 << 18 ? 8192 : 1024; }
bool stable_order_applies(int64_t n, int32_t k) { return k <= kStableLabels && n >= 8 * (int64_t)k; }
static int64_t stable_order_blocks(int64_t n) { return (n + stable_per_block(n) - 1) / stable_per_block(n); }
int64_t stable_order_words(int64_t n, int32_t k) {   // for this many points or fewer
  return std::max<int64_t>(stable_order_blocks(n), std::min<int64_t>((n + 1023) / 1024, 256)) * k;
}

// base[blk][c] = number of points of workgroup blk with label c; labels outside [0, k) set bit 2 of *flag (optional)
__global__ void __launch_bounds__(STB_THREADS) block_counts_kernel(const int32_t *lab, int64_t n, int32_t k, int32_t *base,
                                                                   int per_block, unsigned int *flag) {
  extern __shared__ int s_bins[];
  for (int b = threadIdx.x; b < k; b += STB_THREADS) s_bins[b] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * per_block;
  for (int t = threadIdx.x; t < per_block; t += STB_THREADS) {
    if (i0 + t >= n) break;
    const int a = lab[i0 + t];
    if ((unsigned int)a < (unsigned int)k) atomicAdd(s_bins + a, 1);
    else if (flag) atomicOr(flag, 4u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < k; b += STB_THREADS) base[(int64_t)blockIdx.x * k + b] = s_bins[b];
}
// counts -> starts inside the label: base[blk][c] = points of label c in the workgroups before blk; their total to
// cnt[c] (optional)
__global__ void __launch_bounds__(64) rank_base_kernel(int32_t *base, int32_t nblk, int32_t k, int32_t *cnt) {
  const int c = blockIdx.x * 64 + threadIdx.x;
  if (c >= k) return;
  int run = 0;
  int b = 0;
  for (; b + 16 <= nblk; b += 16) {
    int v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = base[(int64_t)(b + u) * k + c];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      base[(int64_t)(b + u) * k + c] = run;
      run += v[u];
    }
  }
  for (; b < nblk; ++b) {
    const int v = base[(int64_t)b * k + c];
    base[(int64_t)b * k + c] = run;
    run += v;
  }
  if (cnt) cnt[c] = run;
}
__global__ void __launch_bounds__(STB_THREADS) stable_scatter_kernel(const int32_t *lab, int64_t n, int32_t k, int bits,
                                                                     const int32_t *off, const int32_t *base,
                                                                     const int32_t *ids, int32_t *order, int per_block) {
  extern __shared__ unsigned short s_cnt[];   // [STB_WAVES][k]: members before this wavefront's next one, in the workgroup
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int per_wave = per_block / STB_WAVES;   // a multiple of 64
  const int64_t i0 = (int64_t)blockIdx.x * per_block + (int64_t)w * per_wave;
  unsigned short *mine = s_cnt + (size_t)w * k;
  for (int b = threadIdx.x; b < STB_WAVES * k / 2; b += STB_THREADS) reinterpret_cast<unsigned int *>(s_cnt)[b] = 0u;
  if ((STB_WAVES * k) & 1) s_cnt[STB_WAVES * k - 1] = 0;
  __syncthreads();
  // lanes of this round with the same label as this lane (all lanes take part; a lane without a point has label k)
  auto peers = [&](int a) {
    unsigned long long m = ~0ull;
    for (int b = 0; b < bits; ++b) {
      const unsigned long long on = __ballot((a >> b) & 1);
      m &= ((a >> b) & 1) ? on : ~on;
    }
    return m;
  };
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int t = 0; t < per_wave; t += 64) {
    const int64_t i = i0 + t + lane;
    int a = i < n ? lab[i] : k;
    if ((unsigned int)a > (unsigned int)k) a = k;
    const unsigned long long m = peers(a);
    if (a < k && (m & below) == 0) mine[a] = (unsigned short)(mine[a] + __popcll(m));
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  for (int c = threadIdx.x; c < k; c += STB_THREADS) {   // counts of the wavefronts -> members before each of them
    unsigned short run = 0;
#pragma unroll
    for (int u = 0; u < STB_WAVES; ++u) {
      const unsigned short v = s_cnt[(size_t)u * k + c];
      s_cnt[(size_t)u * k + c] = run;
      run = (unsigned short)(run + v);
    }
  }
  __syncthreads();
  for (int t = 0; t < per_wave; t += 64) {
    const int64_t i = i0 + t + lane;
    int a = i < n ? lab[i] : k;
    if ((unsigned int)a > (unsigned int)k) a = k;
    const unsigned long long m = peers(a);
    int rank = 0;
    if (a < k) rank = mine[a] + __popcll(m & below);
    __builtin_amdgcn_wave_barrier();   // every lane has read the counter
    if (a < k) {
      if ((m & below) == 0) mine[a] = (unsigned short)(mine[a] + __popcll(m));
      order[off[a] + base[(int64_t)blockIdx.x * k + a] + rank] = ids ? ids[i] : (int32_t)i;
    }
    __builtin_amdgcn_wave_barrier();
  }
}
// the counting half (cnt, if given, receives the label counts, flag as in block_counts_kernel) ...
static void launch_stable_counts(const int32_t *lab, int64_t n, int32_t k, int32_t *base, int32_t *cnt, unsigned int *flag,
                                 hipStream_t st) {
  const unsigned nblk = (unsigned)stable_order_blocks(n);
  hipLaunchKernelGGL(block_counts_kernel, dim3(nblk), dim3(STB_THREADS), (size_t)k * sizeof(int), st, lab, n, k, base,
                     stable_per_block(n), flag);
  hipLaunchKernelGGL(rank_base_kernel, dim3((unsigned)((k + 63) / 64)), dim3(64), 0, st, base, (int32_t)nblk, k, cnt);
}
// ... and the placing half, with the labels' starts known
static hipError_t launch_stable_scatter(const int32_t *lab, int64_t n, int32_t k, const int32_t *off, const int32_t *base,
                                        int32_t *order, const int32_t *ids, hipStream_t st) {
  static const hipError_t attr_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(stable_scatter_kernel),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize,
                                                        STB_WAVES * kStableLabels * (int)sizeof(unsigned short) + 4);
  if (attr_rc != hipSuccess) return attr_rc;
  int bits = 1;
  while ((1 << bits) <= k) ++bits;   // labels 0 .. k
  hipLaunchKernelGGL(stable_scatter_kernel, dim3((unsigned)stable_order_blocks(n)), dim3(STB_THREADS),
                     (size_t)STB_WAVES * k * sizeof(unsigned short) + 4, st, lab, n, k, bits, off, base, ids, order,
                     stable_per_block(n));
  return hipGetLastError();
}

// The cursor order above depends on scheduling; sorting every segment of `order` makes the summation order, and with it
// every bit of the result, independent of it.  One workgroup per cluster.  Up to RANK_CAP ids every thread counts the
// smaller ids of its own (they are distinct, so the count is the position; 244 ids: 0.3 us of compares and two barriers
// where a bitonic network crosses 36: 82 -> 20 us for 4096 clusters of a million points); above, up to SORT_CAP,
// odd-even merge in LDS; larger clusters are summed in fp64 in whatever order they were scattered (the fp64 sum of fp32
// values then differs from the sorted-order sum by at most a few ulps of fp64, far below the fp32 rounding of the mean).
constexpr int SORT_CAP = 8192, RANK_CAP = 2048;
int32_t update_sort_cap() { return SORT_CAP; }
__global__ void __launch_bounds__(256) rank_segments_kernel(const int32_t *off, int32_t *order) {
  __shared__ __align__(16) int32_t s[RANK_CAP];
  const int c = blockIdx.x;
  const int lo = off[c], len = off[c + 1] - lo;
  if (len < 2 || len > RANK_CAP) return;
  const int len4 = (len + 3) & ~3;
  for (int t = threadIdx.x; t < len4; t += 256) s[t] = t < len ? order[lo + t] : 0x7fffffff;
  __syncthreads();
  for (int t0 = 0; t0 < len; t0 += 1024) {   // four ids of its own per thread and pass over the list
    int mine[4], rank[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + 256 * u + threadIdx.x;
      mine[u] = t < len ? s[t] : -0x7fffffff - 1;
      rank[u] = 0;
    }
    const bool one = t0 + 256 >= len;   // only the first of the four is in use
    for (int q = 0; q < len4; q += 4) {
      const int4 o = *reinterpret_cast<const int4 *>(s + q);
      rank[0] += (o.x < mine[0]) + (o.y < mine[0]) + (o.z < mine[0]) + (o.w < mine[0]);
      if (!one)
#pragma unroll
        for (int u = 1; u < 4; ++u) rank[u] += (o.x < mine[u]) + (o.y < mine[u]) + (o.z < mine[u]) + (o.w < mine[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + 256 * u + threadIdx.x;
      if (t < len) order[lo + rank[u]] = mine[u];
    }
  }
}
__global__ void __launch_bounds__(256) sort_segments_kernel(const int32_t *off, int32_t *order) {
  __shared__ int32_t s[SORT_CAP];
  const int c = blockIdx.x;
  const int lo = off[c], len = off[c + 1] - lo;
  if (len <= RANK_CAP || len > SORT_CAP) return;
  int np2 = 1;
  while (np2 < len) np2 <<= 1;
  for (int t = threadIdx.x; t < np2; t += 256) s[t] = t < len ? order[lo + t] : 0x7fffffff;
  __syncthreads();
  for (int kk = 2; kk <= np2; kk <<= 1)
    for (int jj = kk >> 1; jj > 0; jj >>= 1) {
      for (int t = threadIdx.x; t < np2; t += 256) {
        const int p = t ^ jj;
        if (p > t) {
          const int32_t a = s[t], b = s[p];
          const bool up = (t & kk) == 0;
          if ((a > b) == up) { s[t] = b; s[p] = a; }
        }
      }
      __syncthreads();
    }
  for (int t = threadIdx.x; t < len; t += 256) order[lo + t] = s[t];
}
// largest: size of the largest segment where the host knows it, -1 where it does not
static void launch_sort_segments(const int32_t *off, int32_t *order, int32_t k, int64_t n, int32_t largest, hipStream_t st) {
  const int64_t most = largest >= 0 ? largest : n;
  if (most < 2) return;
  hipLaunchKernelGGL(rank_segments_kernel, dim3(k), dim3(256), 0, st, off, order);
  if (most > RANK_CAP) hipLaunchKernelGGL(sort_segments_kernel, dim3(k), dim3(256), 0, st, off, order);
}

// a lane's four dimensions of a row; ALIGNED: rows are 16-byte aligned and a multiple of 4 long; otherwise one by one
template <bool ALIGNED>
__device__ inline void load_row4(const float *row, int32_t ds, int col, float4 &v) {
  const float *x = row + col;
  if (ALIGNED) {
    v = *reinterpret_cast<const float4 *>(x);
  } else {
    v.x = x[0];
    v.y = col + 1 < ds ? x[1] : 0.f;
    v.z = col + 2 < ds ? x[2] : 0.f;
    v.w = col + 3 < ds ? x[3] : 0.f;
  }
}
// SIGNED: an entry i >= 0 adds row i, an entry ~i < 0 subtracts row i
template <bool SIGNED>
__device__ inline void add_row(const float4 &f, int id, double &a0, double &a1, double &a2, double &a3) {
  if (SIGNED) {
    const double sg = id < 0 ? -1.0 : 1.0;
    a0 += sg * (double)f.x; a1 += sg * (double)f.y; a2 += sg * (double)f.z; a3 += sg * (double)f.w;
  } else {
    a0 += (double)f.x; a1 += (double)f.y; a2 += (double)f.z; a3 += (double)f.w;
  }
}

// Sum of rows in a fixed order, for a lane's four dimensions: entries first, first + STEP, ... of s_ids[0 .. count),
// ROWS of them requested while the ROWS before are added (a row is a round trip to memory: 30 us for a segment of 512 rows
// with four in flight behind the loads of their numbers, 23 with twice eight; the whole update of 1M x 768 680 -> 669).
template <bool SIGNED, bool ALIGNED, int STEP>
__device__ inline void add_rows(const float *Xr, int64_t ldx, int32_t ds, int col, const int *s_ids, int count, int first,
                                double &a0, double &a1, double &a2, double &a3) {
  constexpr int ROWS = 8;
  float4 v[2][ROWS];
  int id[2][ROWS];
  auto fetch = [&](int p, float4 (&to)[ROWS], int (&ids)[ROWS]) {
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int raw = __builtin_amdgcn_readfirstlane(s_ids[min(p + STEP * u, count - 1)]);   // (past the end: the last one again)
      ids[u] = raw;
      load_row4<ALIGNED>(Xr + (int64_t)(SIGNED && raw < 0 ? ~raw : raw) * ldx, ds, col, to[u]);
    }
  };
  auto add = [&](int p, const float4 (&from)[ROWS], const int (&ids)[ROWS]) {
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
      if (p + STEP * u < count) add_row<SIGNED>(from[u], ids[u], a0, a1, a2, a3);
  };
  constexpr int BATCH = STEP * ROWS;
  if (first >= count) return;
  fetch(first, v[0], id[0]);
  for (int p = first; p < count; p += 2 * BATCH) {
    if (p + BATCH < count) fetch(p + BATCH, v[1], id[1]);
    add(p, v[0], id[0]);
    if (p + 2 * BATCH < count) fetch(p + 2 * BATCH, v[0], id[0]);
    add(p + BATCH, v[1], id[1]);
  }
}

// The same for a short list in memory (entries first, first + 4, ... of ids[0 .. count)): a wavefront holds the numbers of 64
// entries and asks for four rows at a time (with eight and their registers fewer segments are under way).
template <bool SIGNED, bool ALIGNED>
__device__ inline void add_few_rows(const float *Xr, int64_t ldx, int32_t ds, int col, const int32_t *ids, int count, int first,
                                    int lane, double &a0, double &a1, double &a2, double &a3) {
  constexpr int ROWS = 4;
  for (int b = 0; b < count; b += 64) {
    const int held = ids[min(b + lane, count - 1)];
    const int end = min(count - b, 64);
    for (int p = first; p < end; p += 4 * ROWS) {
      float4 v[ROWS];
      int id[ROWS];
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        id[u] = __builtin_amdgcn_readlane(held, min(p + 4 * u, end - 1));   // (past the end: the last one again)
        load_row4<ALIGNED>(Xr + (int64_t)(SIGNED && id[u] < 0 ? ~id[u] : id[u]) * ldx, ds, col, v[u]);
      }
#pragma unroll
      for (int u = 0; u < ROWS; ++u)
        if (p + 4 * u < end) add_row<SIGNED>(v[u], id[u], a0, a1, a2, a3);
    }
  }
}

// One workgroup per (segment of <= kSegPoints points of one cluster, slice of 256 dims): rows are gathered through
// `order` (each a contiguous row read), fp64 sums per thread; the four wavefronts' sums are added in a fixed order, so the
// result depends on the segment only.
// SIGNED, ALIGNED: see load_row4 and add_row (an entry ~i: a point that left the cluster).  SHORT: see launch_segment_sums.
template <bool SIGNED, bool ALIGNED, bool SHORT>
__global__ void __launch_bounds__(256) segment_sum_kernel(const float *Xr, int64_t ldx, int32_t ds, int32_t k,
                                                          const int32_t *off, const int32_t *segoff,
                                                          const int32_t *order, double *partial) {
  __shared__ double red[3][64][4];
  __shared__ int s_ids[SHORT ? 1 : kSegPoints];
  const int seg = blockIdx.x;
  if (seg >= segoff[k]) return;
  // cluster of this segment: last c with segoff[c] <= seg
  int lo = 0, hi = k;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (segoff[mid] <= seg) lo = mid; else hi = mid;
  }
  const int c = lo;
  const int s_in = seg - segoff[c];
  const int p0 = off[c] + s_in * kSegPoints;
  const int p1 = min(off[c + 1], p0 + kSegPoints);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = (blockIdx.y * 64 + lane) * 4;
  const bool live = col < ds;
  double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
  if constexpr (SHORT) {   // (lanes past the row's end hold numbers as well, and read its last four values)
    add_few_rows<SIGNED, ALIGNED>(Xr, ldx, ds, live ? col : ALIGNED ? ds - 4 : ds - 1, order + p0, p1 - p0, w, lane, a0, a1, a2, a3);
  } else {
    for (int t = threadIdx.x; t < p1 - p0; t += 256) s_ids[t] = order[p0 + t];
    __syncthreads();
    if (live) add_rows<SIGNED, ALIGNED, 4>(Xr, ldx, ds, col, s_ids, p1 - p0, w, a0, a1, a2, a3);
  }
  if (w > 0) {
    red[w - 1][lane][0] = a0; red[w - 1][lane][1] = a1; red[w - 1][lane][2] = a2; red[w - 1][lane][3] = a3;
  }
  __syncthreads();
  if (w == 0 && live) {
    double *dst = partial + (int64_t)seg * ds + col;
    dst[0] = (a0 + red[0][lane][0]) + (red[1][lane][0] + red[2][lane][0]);
    if (ALIGNED || col + 1 < ds) dst[1] = (a1 + red[0][lane][1]) + (red[1][lane][1] + red[2][lane][1]);
    if (ALIGNED || col + 2 < ds) dst[2] = (a2 + red[0][lane][2]) + (red[1][lane][2] + red[2][lane][2]);
    if (ALIGNED || col + 3 < ds) dst[3] = (a3 + red[0][lane][3]) + (red[1][lane][3] + red[2][lane][3]);
  }
}

// (n entries of k lists.)  Segments of a few rows are many workgroups that wait for their numbers and a round trip or two: there the
// short form, without the stop in LDS and with registers for twice as many of them.  Sixteen rows in flight -> short form, us of this
// kernel with 8 | 16 rows on average: 8000 lists of 64 dimensions 23.2 -> 18.1 | 23.6 -> 20.0, of 256 24.6 -> 19.8 | 28.0 -> 26.1, of 768
// 65.2 -> 50.7 | 91.3 -> 91.1; whole updates with 29 rows a list (201 057 x 64) 87.0 -> 83.3; but with 43 (30 000 x 512) 55.5 -> 58.8, 40
// (40 000 x 256) 51.9 -> 55.0, and 1000 lists of 256 rows of 64 dimensions 16.3 -> 21.9.
template <bool SIGNED>
static void launch_segment_sums(bool aligned, int64_t n, int32_t k, unsigned segs, unsigned slices, const float *Xr, int64_t ldx,
                                int32_t ds, const int32_t *off, const int32_t *segoff, const int32_t *order, double *partial,
                                hipStream_t st) {
  const bool few = n < 32 * (int64_t)k;
  auto kern = few ? segment_sum_kernel<SIGNED, true, true> : segment_sum_kernel<SIGNED, true, false>;
  if constexpr (!SIGNED)   // (the rows of a fit are aligned)
    if (!aligned) kern = few ? segment_sum_kernel<false, false, true> : segment_sum_kernel<false, false, false>;
  hipLaunchKernelGGL(kern, dim3(segs, slices), dim3(256), 0, st, Xr, ldx, ds, k, off, segoff, order, partial);
}

// One workgroup per (cluster, slice): partial sums added in segment order, divided by the size.
// S (optional, [k][ds] fp64) keeps the sum of every cluster between updates: it is overwritten by the total of the
// partials, or, with `accumulate`, the total (a signed change) is added to it.
// y_absmax (optional, zero before the launch) receives the bit pattern of max |Y| over all centroids, the bound
// that the split-fp16 GEMMs of the next step scale the centroids by.
__global__ void __launch_bounds__(256) centroid_mean_kernel(const double *partial, int32_t ds, const int32_t *cnt,
                                                            const int32_t *segoff, float *Y, int64_t ldy, double *S,
                                                            int accumulate, unsigned int *y_absmax,
                                                            const unsigned int *flag, unsigned int *flag_host,
                                                            int32_t *counts_out) {
  const int c = blockIdx.x;
  if (flag) {   // labels that the counting pass found outside [0, k): reported, and Y stays what it was
    const unsigned int f = *flag;
    if (c == 0 && blockIdx.y == 0 && threadIdx.x == 0) *flag_host = f;
    if (f) return;
  }
  const int n_c = cnt[c];
  if (counts_out && blockIdx.y == 0 && threadIdx.x == 0) counts_out[c] = n_c;
  const int col = blockIdx.y * 256 + threadIdx.x;
  float y = 0.f;
  if (col < ds) {
    double s = 0.0;
    for (int seg = segoff[c]; seg < segoff[c + 1]; ++seg) s += partial[(int64_t)seg * ds + col];
    if (S) {
      if (accumulate) s += S[(int64_t)c * ds + col];
      S[(int64_t)c * ds + col] = s;
    }
    if (!Y) {
      // sums only (a batch of a larger update: the means follow once all batches are in)
    } else if (n_c == 0) {   // an empty cluster keeps its centroid until the split
      y = Y[(int64_t)c * ldy + col];
    } else {
      y = (float)(s / (double)n_c);
      Y[(int64_t)c * ldy + col] = y;
    }
  }
  if (y_absmax) block_absmax(y, y_absmax);
}

// Y = S / size for every cluster with points (an empty one keeps its row), max |Y| into *y_absmax (zero before).
__global__ void __launch_bounds__(256) means_from_sums_kernel(const double *S, const int32_t *cnt, int32_t ds, float *Y,
                                                              int64_t ldy, unsigned int *y_absmax) {
  const int c = blockIdx.x;
  const int n_c = cnt[c];
  const int col = blockIdx.y * 256 + threadIdx.x;
  float y = 0.f;
  if (col < ds) {
    if (n_c == 0) {
      y = Y[(int64_t)c * ldy + col];
    } else {
      y = (float)(S[(int64_t)c * ds + col] / (double)n_c);
      Y[(int64_t)c * ldy + col] = y;
    }
  }
  if (y_absmax) block_absmax(y, y_absmax);
}
hipError_t launch_means_from_sums(const double *S, const int32_t *cnt, int32_t k, int32_t ds, float *Y, int64_t ldy,
                                  unsigned int *y_absmax, hipStream_t st) {
  if (y_absmax)
    if (hipError_t rc = launch_fill_u32(y_absmax, 1, 0u, st); rc != hipSuccess) return rc;
  hipLaunchKernelGGL(means_from_sums_kernel, dim3(k, (unsigned)((ds + 255) / 256)), dim3(256), 0, st, S, cnt, ds, Y, ldy,
                     y_absmax);
  return hipGetLastError();
}

// total[c] += cnt[c] (sizes of the batches of a pass)
__global__ void add_counts_kernel(const int32_t *cnt, int32_t k, int32_t *total) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < k) total[c] += cnt[c];
}
hipError_t launch_add_counts(const int32_t *cnt, int32_t k, int32_t *total, hipStream_t st) {
  hipLaunchKernelGGL(add_counts_kernel, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, st, cnt, k, total);
  return hipGetLastError();
}

// Points whose label changed: entry (i, new label) and entry (~i, old label), in ascending order of i.  start[b] is the
// number of changed points before the points of workgroup b (the ranges of the finalize kernel, which took them).  A
// wavefront owns a contiguous quarter of the workgroup's points: one pass counts, one writes, no atomics.  Also clears
// what the kernels behind it add to: `zero` (one word) and zero_cnt[k].
__global__ void __launch_bounds__(256) compact_changes_kernel(const int32_t *assign, const int32_t *prev, int64_t n,
                                                              const int32_t *start, int per_block, int32_t *ent_id,
                                                              int32_t *ent_lab, unsigned int cap, unsigned int *zero,
                                                              int32_t *zero_cnt, int32_t k, UpdateAhead ahead) {
  __shared__ int s_cnt[4];
  if (ahead.changed && ahead.entries() == 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == 0 && tid == 0 && zero) *zero = 0u;
  if (zero_cnt)
    for (int64_t c = (int64_t)blockIdx.x * 256 + tid; c < k; c += (int64_t)gridDim.x * 256) zero_cnt[c] = 0;
  const int quarter = per_block / 4;
  const int64_t base = (int64_t)blockIdx.x * per_block + (int64_t)wave * quarter;
  int mine = 0;
  for (int t = 0; t < quarter; t += 64) {
    const int64_t i = base + t + lane;
    mine += __popcll(__ballot(i < n && assign[i] != prev[i]));
  }
  if (lane == 0) s_cnt[wave] = mine;
  __syncthreads();
  if (mine == 0) return;
  unsigned int run = (unsigned int)start[blockIdx.x];
  for (int w = 0; w < wave; ++w) run += (unsigned int)s_cnt[w];
  for (int t = 0; t < quarter; t += 64) {
    const int64_t i = base + t + lane;
    const int a = i < n ? assign[i] : 0, b = i < n ? prev[i] : 0;
    const unsigned long long bal = __ballot(a != b);
    if (a != b) {
      const unsigned int e = 2u * (run + (unsigned int)__popcll(bal & ((1ull << lane) - 1ull)));
      if (e + 2u <= cap) {
        ent_id[e] = (int32_t)i;
        ent_lab[e] = a;
        ent_id[e + 1] = ~(int32_t)i;
        ent_lab[e + 1] = b;
      }
    }
    run += (unsigned int)__popcll(bal);
  }
}

// The whole of a small incremental update behind the compaction: the workgroup of (cluster, slice of 256 dims) looks
// through all m entries, keeps those of its cluster in their order, adds the rows that joined and subtracts those that
// left, and writes the sum and the mean.  Every workgroup reads the m labels (from L2): worth it while
// m * workgroups stays below kDirectUpdate labels; it replaces the counting, scan, scatter, sort, segment-sum and mean
// kernels, whose launches are all the time of an update in which a few points moved (35 -> 12 us).  (47 000 entries on 70
// clusters: a row at a time behind every chunk of 1024 labels 201 us, eight and more in flight over the chunks 100.)
constexpr int64_t kDirectUpdate = (int64_t)1 << 25;
constexpr int DIRECT_CHUNK = 1024;
__global__ void __launch_bounds__(256) direct_update_kernel(const float *Xr, int64_t ldx, int32_t ds, const int32_t *ent_id,
                                                            const int32_t *ent_lab, int m, const int32_t *cnt, double *S,
                                                            float *Y, int64_t ldy, unsigned int *y_absmax, UpdateAhead ahead) {
  if (ahead.changed) {
    m = ahead.entries();
    if (m == 0) return;
  }
  // The rows of a cluster in a chunk of entries go to the four wavefronts in turn (the order of the sums does not depend on
  // how many chunks are taken together); their lists are worked off when one is nearly full, and at the end.
  constexpr int LIST = 1024;
  __shared__ int s_ids[4][LIST];
  __shared__ int s_n[2][DIRECT_CHUNK / 64];   // (by chunk parity: the chunk before may still be read)
  __shared__ double red[3][64][4];
  const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int col = (blockIdx.y * 64 + lane) * 4;
  const bool live = col < ds;
  double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
  bool any = false;
  // thread t holds entries e0 + 256 j + t of a chunk: matches in order of (j, wavefront, lane).  The next chunk's labels are
  // requested behind this one's, the numbers of the rows reach their lists a chunk later.
  constexpr int PER = DIRECT_CHUNK / 256;
  int lab[PER], id[PER], at[PER], len[4] = {0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < PER; ++j) at[j] = -1;
  auto fetch = [&](int e0) {
#pragma unroll
    for (int j = 0; j < PER; ++j) lab[j] = e0 + 256 * j + tid < m ? ent_lab[e0 + 256 * j + tid] : -1;
  };
  auto write = [&]() {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (at[j] >= 0) (&s_ids[0][0])[at[j]] = id[j];
      at[j] = -1;
    }
  };
  auto work_off = [&]() {
    write();
    __syncthreads();
    const int mine = w == 0 ? len[0] : w == 1 ? len[1] : w == 2 ? len[2] : len[3];
    if (live && mine > 0) add_rows<true, true, 1>(Xr, ldx, ds, col, s_ids[w], mine, 0, a0, a1, a2, a3);
    __syncthreads();
    len[0] = len[1] = len[2] = len[3] = 0;
  };
  fetch(0);
  for (int e0 = 0; e0 < m; e0 += DIRECT_CHUNK) {
    const int par = (e0 / DIRECT_CHUNK) & 1;
    unsigned long long bal[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      bal[j] = __ballot(lab[j] == c);
      if (lane == 0) s_n[par][4 * j + w] = __popcll(bal[j]);
    }
    if (e0 + DIRECT_CHUNK < m) fetch(e0 + DIRECT_CHUNK);
    write();
    __syncthreads();
    int have = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (u == w && ((bal[j] >> lane) & 1ull)) {
          const int p = have + __popcll(bal[j] & ((1ull << lane) - 1ull)), q = p & 3;
          at[j] = q * LIST + (q == 0 ? len[0] : q == 1 ? len[1] : q == 2 ? len[2] : len[3]) + (p >> 2);
          id[j] = ent_id[e0 + 256 * j + tid];
        }
        have += s_n[par][4 * j + u];
      }
    any |= have > 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) len[u] += (have + 3 - u) >> 2;
    if (len[0] > LIST - DIRECT_CHUNK / 4) work_off();   // (the longest list; the same for all threads)
  }
  if (len[0] > 0) work_off();
  if (any) {
    if (w > 0) {
      red[w - 1][lane][0] = a0; red[w - 1][lane][1] = a1; red[w - 1][lane][2] = a2; red[w - 1][lane][3] = a3;
    }
    __syncthreads();
  }
  float vmax = 0.f;
  if (w == 0 && live) {
    double d[4] = {a0, a1, a2, a3};
    const int n_c = cnt[c];
    double *sp = S + (int64_t)c * ds + col;
    float *yp = Y + (int64_t)c * ldy + col;
    float4 y = *reinterpret_cast<const float4 *>(yp);
    float *ye = &y.x;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      double s = sp[u];
      if (any) {
        s += (d[u] + red[0][lane][u]) + (red[1][lane][u] + red[2][lane][u]);
        sp[u] = s;
      }
      if (n_c != 0) ye[u] = (float)(s / (double)n_c);   // an empty cluster keeps its centroid until the split
      vmax = fmaxf(vmax, fabsf(ye[u]));
    }
    *reinterpret_cast<float4 *>(yp) = y;
  }
  if (y_absmax) block_absmax(vmax, y_absmax);
}

// order[] = the items grouped by label (off: the groups' starts), ascending in a group: stably where `base` is given, else
// scattered and then ordered
static hipError_t group_by_label(const int32_t *lab, int64_t n, int32_t k, const int32_t *off, int32_t *cursor, int32_t *base,
                                 int32_t *order, const int32_t *ids, int32_t largest, hipStream_t st) {
  if (base) {
    launch_stable_counts(lab, n, k, base, nullptr, nullptr, st);
    return launch_stable_scatter(lab, n, k, off, base, order, ids, st);
  }
  launch_scatter_order(lab, n, k, off, cursor, order, ids, st);
  launch_sort_segments(off, order, k, n, largest, st);
  return hipSuccess;
}

hipError_t launch_update(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const int32_t *assign, int32_t k,
                         const UpdateWs &w, float *Y, int64_t ldy, hipStream_t st, double *S, unsigned int *y_absmax,
                         int accumulate, int32_t largest, const UnsafeLabels *unsafe) {
  if ((w.base && !stable_order_applies(n, k)) || (accumulate && !S) || (!Y && y_absmax)) return hipErrorInvalidValue;
  if (unsafe) {   // labels nobody has counted or checked
    if (w.base) {
      launch_stable_counts(assign, n, k, w.base, w.cnt, unsafe->flag, st);
    } else {
      hipError_t rc = launch_fill_u32(reinterpret_cast<unsigned int *>(w.cnt), k, 0u, st);
      if (rc == hipSuccess) rc = launch_histogram(assign, n, k, w.cnt, unsafe->flag, st);
      if (rc != hipSuccess) return rc;
    }
  }
  hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(1024), 0, st, w.cnt, k, w.off, w.cursor, w.segoff, y_absmax);
  {
    hipError_t rc = unsafe && w.base ? launch_stable_scatter(assign, n, k, w.off, w.base, w.order, nullptr, st)
                                     : group_by_label(assign, n, k, w.off, w.cursor, w.base, w.order, nullptr, largest, st);
    if (rc != hipSuccess) return rc;
  }
  const unsigned slices = (unsigned)((ds + 255) / 256);   // 64 lanes x 4 dims, or 256 dims, per workgroup
  const bool aligned = (reinterpret_cast<uintptr_t>(Xr) & 15u) == 0 && ldx % 4 == 0 && ds % 4 == 0;
  launch_segment_sums<false>(aligned, n, k, (unsigned)w.max_segments, slices, Xr, ldx, ds, w.off, w.segoff, w.order, w.partial, st);
  hipLaunchKernelGGL(centroid_mean_kernel, dim3(k, slices), dim3(256), 0, st, w.partial, ds, w.cnt, w.segoff, Y, ldy, S,
                     accumulate, y_absmax, unsafe ? (const unsigned int *)unsafe->flag : nullptr,
                     unsafe ? unsafe->flag_host : nullptr, unsafe ? unsafe->counts_out : nullptr);
  return hipGetLastError();
}

// order[] = the point ids grouped by label (members of a cluster of at most SORT_CAP points in ascending order, with `base`
// those of any cluster), off[] the start of every group, cnt[] the group sizes: the first half of launch_update, for callers
// that only want the grouping.
hipError_t launch_group_order(const int32_t *labels, int64_t n, int32_t k, int32_t *cnt, int32_t *off, int32_t *cursor,
                              int32_t *segoff, int32_t *order, int32_t *base, hipStream_t st) {
  if (base) {
    if (!stable_order_applies(n, k)) return hipErrorInvalidValue;
    launch_stable_counts(labels, n, k, base, cnt, nullptr, st);
    hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(1024), 0, st, cnt, k, off, cursor, segoff, (unsigned int *)nullptr);
    return launch_stable_scatter(labels, n, k, off, base, order, nullptr, st);
  }
  hipError_t rc = launch_fill_u32(reinterpret_cast<unsigned int *>(cnt), k, 0u, st);
  if (rc != hipSuccess) return rc;
  rc = launch_histogram(labels, n, k, cnt, nullptr, st);
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(1024), 0, st, cnt, k, off, cursor, segoff, (unsigned int *)nullptr);
  launch_scatter_order(labels, n, k, off, cursor, order, nullptr, st);
  launch_sort_segments(off, order, k, n, -1, st);
  return hipGetLastError();
}

// An order of points partitioned, stably, by the class of their threshold: 0 below THR_TAIL times the median, above that by
// halves of what is left, 2 for the top quarter, 3 for the top eighth, ..., THR_CLASSES - 1 for the top 1/32 (1 is empty: the
// median's own half).  Thresholds that are worth a tile of their own are a long tail (incumbents out of date, points far from
// every centroid: quantiles of 2.5M x 384 against 32 768 centroids 0.22 at 1/2, 0.27 at 0.9, 1.44 at 0.99), and a point of the
// tail keeps nearly every column of its row tile alive.  Grouped by label alone nearly every tile of 128 points holds one.
// Column tiles listed per row tile, and the whole call in ms, by label -> with 4 | 6 | 8 classes of any threshold -> with 6 above
// 1.25 | 1.5 | 2 times the median (these on top of a cheaper finish of poor tiles):
//   2.5M x 384, k = 32 768            209 -> 28.1 | 16.4 | 16.4 -> 16.4 | 14.4 | 14.4    99.4 -> 42.7 | 40.8 | 40.8 -> 42.4 | 40.0 | 39.9
//   1M x 768, k = 16 384              108 -> 14.9 | 8.6 | 8.6 -> 8.2 | 8.1 | 8.1         42.3 -> 25.5 | 22.2 | 22.1 -> 22.1 | 21.8 | 21.9
//   1M x 768, k = 5000                22 -> 5.0 | 3.3 | 3.3 -> 2.9 | 2.9 | 2.9           16.3 -> 13.9 | 13.5 | 13.5 -> 13.2 | 13.3 | 13.2
//   40 000 x 256, k = 4500            34 -> 4.8 | 3.6 | 3.6 -> 3.2 | 2.8 | 2.7           0.60 -> 0.58 | 0.59 | 0.57 -> 0.56 | 0.55 | 0.57
//   600 000 x 1536, k = 10 000, no incumbents given  51 -> 7.8 | 5.3 | 5.3 -> 5.0 | 5.0 | 5.0    69.3 -> ... -> 30.9 | 31.0 | 31.0
// Thresholds that are alike are better left in the order of the labels: 2M x 96 around 16 384 centres, every incumbent right, 10.5
// column tiles a row tile, 14.7 with classes of any threshold, 11.5 | 10.5 | 10.5 with a limit (8.1 ms by label, 9.5, 9.0 | 8.5 |
// 8.6).  Twice the median: the squared distances of a normal cloud in 64 dimensions do not reach it.
// The ranks come from a histogram of the thresholds' upper bits (exponent and 5 bits of the mantissa: a bin is 3 % wide, and
// a bin that crosses a border goes to the lower class), so no sort is needed and the order depends on the thresholds alone.
constexpr int THR_BINS = 8192, THR_CLASSES = 6, THR_SAMPLE = 16;
constexpr float THR_TAIL = 2.f;
__global__ void threshold_bins_kernel(const float *tau, int64_t n, int32_t *bin) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    bin[i] = (int32_t)((__float_as_uint(tau[i]) & 0x7fffffffu) >> 18);
}
// class_of[b] = 0 where the bin starts below THR_TAIL times the median's, else floor(log2(n / number of points in the bins from b
// on)), at most THR_CLASSES - 1.  *above (optional): the points of the other classes.  With `quarters` the quarter that the
// bin starts in.
__global__ void __launch_bounds__(1024) threshold_classes_kernel(const int32_t *cnt, int64_t n, int32_t *class_of,
                                                                 int32_t *above, int quarters) {
  constexpr int PER = THR_BINS / 1024;
  __shared__ int s_sum[16];
  __shared__ int s_median, s_above;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int v[PER], sum = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) sum += v[u] = cnt[tid * PER + u];
  int run = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(run, o, 64);
    if (lane >= o) run += t;
  }
  if (lane == 63) s_sum[wave] = run;
  __syncthreads();
  int64_t first = run - sum;   // points in the bins below this thread's
  for (int w = 0; w < wave; ++w) first += s_sum[w];
  int64_t below = first;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (2 * below <= n && 2 * (below + v[u]) > n) s_median = tid * PER + u;
    below += v[u];
  }
  __syncthreads();
  if (tid == 0) s_above = 0;
  __syncthreads();
  int mine = 0;
  const float tail = THR_TAIL * __uint_as_float((unsigned int)s_median << 18);
  below = first;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int b = tid * PER + u;
    int c = 0;
    while (c < THR_CLASSES - 1 && ((n - below) << (c + 1)) <= n) ++c;
    if (__uint_as_float((unsigned int)b << 18) < tail) c = 0;
    if (quarters > 0) c = (int)min(quarters * below / n, (int64_t)quarters - 1);
    class_of[b] = c;
    if (c > 0) mine += v[u];
    below += v[u];
  }
  if (mine) atomicAdd(&s_above, mine);
  __syncthreads();
  if (above && tid == 0) *above = s_above;
}
__global__ void class_of_points_kernel(const int32_t *order, const int32_t *bin, const int32_t *class_of, int64_t n, int32_t *cls) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x)
    cls[p] = class_of[bin[order[p]]];
}
__global__ void sample_labels_kernel(const int32_t *labels, int64_t m, int32_t *out) {
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < m; j += (int64_t)gridDim.x * blockDim.x)
    out[j] = labels[j * THR_SAMPLE];
}
int64_t threshold_class_words(int64_t n) { return 2 * THR_BINS + 4 * (THR_CLASSES + 1) + stable_order_words(n, THR_CLASSES); }
static unsigned threshold_grid(int64_t n) { return (unsigned)std::min<int64_t>((n + 255) / 256, (int64_t)num_cus() * 16); }
// words: [THR_BINS] counts | [THR_BINS] classes | the classes' sizes and starts | block counts of the partition
static hipError_t classify_thresholds(const float *tau, int64_t n, int32_t *bin, int32_t *words, int32_t *above, int quarters,
                                      hipStream_t st) {
  hipLaunchKernelGGL(threshold_bins_kernel, dim3(threshold_grid(n)), dim3(256), 0, st, tau, n, bin);
  hipError_t rc = launch_fill_u32(reinterpret_cast<unsigned int *>(words), THR_BINS, 0u, st);
  if (rc != hipSuccess) return rc;
  // (in LDS for few points too: thresholds that are alike fall into few bins, and 60 000 atomics on those took 0.2 ms)
  const int per = 8192;
  hipLaunchKernelGGL(histogram_kernel, dim3((unsigned)((n + per - 1) / per)), dim3(CNT_THREADS), THR_BINS * sizeof(int), st,
                     (const int32_t *)bin, n, (int32_t)THR_BINS, words, (unsigned int *)nullptr, per, 1);
  hipLaunchKernelGGL(threshold_classes_kernel, dim3(1), dim3(1024), 0, st, (const int32_t *)words, n, words + THR_BINS, above,
                     quarters);
  return hipGetLastError();
}
// A tail of one point in 2000 is in every 16th row tile.  One point of THR_SAMPLE tells whether there is one: the pass over all
// thresholds and the partition are 3 to 5 % of a step that has none (2M x 96 above 0.4 of 8.1 ms), the sample 0.03 to 0.05 ms.
hipError_t launch_threshold_sample(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const float *Y, int64_t ldy,
                                   const int32_t *labels, float *tau, int32_t *bin, int32_t *words, int32_t *above, hipStream_t st) {
  if (n <= 0) return hipErrorInvalidValue;
  const int64_t m = (n + THR_SAMPLE - 1) / THR_SAMPLE;
  hipLaunchKernelGGL(sample_labels_kernel, dim3(threshold_grid(m)), dim3(256), 0, st, labels, m, bin);
  hipError_t rc = launch_tau_init(Xr, ldx * THR_SAMPLE, m, ds, Y, ldy, bin, tau, nullptr, st);
  if (rc != hipSuccess) return rc;
  return classify_thresholds(tau, m, bin, words, above, 0, st);
}
bool thresholds_have_tail(int64_t n, int32_t above) { return (int64_t)above * 2000 > (n + THR_SAMPLE - 1) / THR_SAMPLE; }
hipError_t launch_threshold_classes(const float *tau, int64_t n, int quarters, const int32_t *order, int32_t *bin, int32_t *cls,
                                    int32_t *words, int32_t *order_out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int32_t *class_of = words + THR_BINS;
  int32_t *cnt = words + 2 * THR_BINS, *off = cnt + THR_CLASSES + 1, *cursor = off + THR_CLASSES + 1, *segoff = cursor + THR_CLASSES + 1;
  int32_t *base = segoff + THR_CLASSES + 1;
  hipError_t rc = classify_thresholds(tau, n, bin, words, nullptr, quarters, st);
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(class_of_points_kernel, dim3(threshold_grid(n)), dim3(256), 0, st, order, (const int32_t *)bin, class_of, n, cls);
  launch_stable_counts(cls, n, THR_CLASSES, base, cnt, nullptr, st);
  hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(1024), 0, st, (const int32_t *)cnt, (int32_t)THR_CLASSES, off, cursor, segoff,
                     (unsigned int *)nullptr);
  return launch_stable_scatter(cls, n, THR_CLASSES, off, base, order_out, order, st);
}

// The same update from the points that changed label only: S (the cluster sums of the previous update) takes the
// rows of the points that joined minus those of the points that left, and every centroid is S / size again.
// w.cnt holds the new cluster sizes; `changed` is the number of points with assign != prev (known to the host from
// the assignment step) and change_start what the finalize kernel left; inc is a workspace for 2 * changed entries.
hipError_t launch_update_incremental(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const int32_t *assign,
                                     const int32_t *prev, int64_t changed, const int32_t *change_start, int32_t k,
                                     const UpdateWs &w, const IncUpdateWs &inc, double *S, float *Y, int64_t ldy,
                                     hipStream_t st, unsigned int *y_absmax) {
  const int64_t m2 = 2 * changed;
  if (m2 <= 0 || m2 > inc.capacity || !S) return hipErrorInvalidValue;
  const unsigned slices = (unsigned)((ds + 255) / 256);   // 64 lanes x 4 dims, or 256 dims, per workgroup
  const bool direct = m2 * (int64_t)k * slices <= kDirectUpdate;
  hipLaunchKernelGGL(compact_changes_kernel, dim3((unsigned)finalize_blocks(n)), dim3(256), 0, st, assign, prev, n,
                     change_start, finalize_per_block(n), inc.ent_id, inc.ent_lab, (unsigned int)inc.capacity, y_absmax,
                     direct ? (int32_t *)nullptr : inc.cnt, k, UpdateAhead());
  if (direct) {
    hipLaunchKernelGGL(direct_update_kernel, dim3(k, slices), dim3(256), 0, st, Xr, ldx, ds, (const int32_t *)inc.ent_id,
                       (const int32_t *)inc.ent_lab, (int)m2, w.cnt, S, Y, ldy, y_absmax, UpdateAhead());
    return hipGetLastError();
  }
  hipError_t rc = launch_histogram(inc.ent_lab, m2, k, inc.cnt, nullptr, st);
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(1024), 0, st, inc.cnt, k, inc.off, inc.cursor, inc.segoff,
                     (unsigned int *)nullptr);
  // (the entries are in ascending order of their points, joined before left: stable grouping keeps that)
  rc = group_by_label(inc.ent_lab, m2, k, inc.off, inc.cursor, stable_order_applies(m2, k) ? inc.base : nullptr, inc.order,
                      inc.ent_id, -1, st);
  if (rc != hipSuccess) return rc;
  const int64_t segs = std::min<int64_t>(inc.max_segments, (int64_t)k + m2 / kSegPoints + 1);
  launch_segment_sums<true>(true, m2, k, (unsigned)segs, slices, Xr, ldx, ds, inc.off, inc.segoff, inc.order, inc.partial, st);
  hipLaunchKernelGGL(centroid_mean_kernel, dim3(k, slices), dim3(256), 0, st, inc.partial, ds, w.cnt, inc.segoff, Y, ldy,
                     S, 1, y_absmax, (const unsigned int *)nullptr, (unsigned int *)nullptr, (int32_t *)nullptr);
  return hipGetLastError();
}

int64_t update_ahead_most(int32_t ds, int32_t k, int64_t capacity) {
  return std::min(capacity - 2, kDirectUpdate / ((int64_t)k * ((ds + 255) / 256))) / 2;
}
hipError_t launch_update_ahead(const float *Xr, int64_t ldx, int64_t n, int32_t ds, const int32_t *assign, const int32_t *prev,
                               const int32_t *change_start, int32_t k, const UpdateWs &w, const IncUpdateWs &inc, double *S,
                               float *Y, int64_t ldy, const UpdateAhead &ahead, hipStream_t st, unsigned int *y_absmax) {
  if (ahead.most <= 0 || ahead.most > update_ahead_most(ds, k, inc.capacity) || !ahead.changed || !ahead.flag || !S) return hipErrorInvalidValue;
  hipLaunchKernelGGL(compact_changes_kernel, dim3((unsigned)finalize_blocks(n)), dim3(256), 0, st, assign, prev, n,
                     change_start, finalize_per_block(n), inc.ent_id, inc.ent_lab, (unsigned int)inc.capacity, y_absmax,
                     (int32_t *)nullptr, k, ahead);
  hipLaunchKernelGGL(direct_update_kernel, dim3(k, (unsigned)((ds + 255) / 256)), dim3(256), 0, st, Xr, ldx, ds, (const int32_t *)inc.ent_id,
                     (const int32_t *)inc.ent_lab, 0, w.cnt, S, Y, ldy, y_absmax, ahead);
  return hipGetLastError();
}

// ------------------------------------------------------------------ split of empty clusters
// pairs = (empty, donor) in the order decided on the host.  A donor may be used twice and a re-seeded cluster may
// itself donate later, so the splits of one chain (splits that share clusters, grouped by the host) are applied one
// after the other by one workgroup; chains touch disjoint rows and run side by side.
__global__ void __launch_bounds__(256) split_kernel(float *Y, int64_t ldy, int32_t d, const int32_t *pairs,
                                                    const int32_t *chain_first, float eps) {
  const int s0 = chain_first[blockIdx.x], s1 = chain_first[blockIdx.x + 1];
  for (int s = s0; s < s1; ++s) {
    const int e = pairs[2 * s], c = pairs[2 * s + 1];
    for (int j = threadIdx.x; j < d; j += 256) {
      const float sg = (j & 1) ? -1.f : 1.f;
      const float y = Y[(int64_t)c * ldy + j];
      Y[(int64_t)e * ldy + j] = y * (1.f + eps * sg);
      Y[(int64_t)c * ldy + j] = y * (1.f - eps * sg);
    }
    __syncthreads();
  }
}
hipError_t launch_split(float *Y, int64_t ldy, int32_t d, const int32_t *pairs_dev, const int32_t *chain_first_dev,
                        int32_t nchains, float eps, hipStream_t st) {
  if (nchains <= 0) return hipSuccess;
  hipLaunchKernelGGL(split_kernel, dim3((unsigned)nchains), dim3(256), 0, st, Y, ldy, d, pairs_dev, chain_first_dev, eps);
  return hipGetLastError();
}

// ------------------------------------------------------------------ small copies
__global__ void __launch_bounds__(256) gather_rows_kernel(const float *src, int64_t lds, int32_t d,
                                                          const int64_t *idx, float *dst, int64_t ldd, int32_t dpad,
                                                          unsigned int *absmax, stamp_t *stamp) {
  const int c = blockIdx.x;
  put_stamp(stamp);
  const float *s = src + idx[c] * lds;
  float m = 0.f;
  for (int j = threadIdx.x; j < dpad; j += 256) {
    const float v = j < d ? s[j] : 0.f;
    dst[(int64_t)c * ldd + j] = v;
    m = fmaxf(m, fabsf(v));
  }
  if (absmax) block_absmax(m, absmax);
}
hipError_t launch_gather_rows(const float *src, int64_t lds, int32_t d, const int64_t *idx, int32_t k, float *dst,
                              int64_t ldd, int32_t dpad, hipStream_t st, unsigned int *absmax, stamp_t *stamp) {
  hipLaunchKernelGGL(gather_rows_kernel, dim3(k), dim3(256), 0, st, src, lds, d, idx, dst, ldd, dpad, absmax, stamp);
  return hipGetLastError();
}

// dst[i][j] = src[i][j] (or src[j][i] when transpose) for j < d, 0 for d <= j < dpad
__device__ inline void pad_copy(const float *src, int64_t lds, int64_t n, int32_t d, float *dst, int64_t ldd, int32_t dpad,
                                int32_t transpose, int block, int nblocks) {
  const int64_t total = n * dpad;
  for (int64_t t = (int64_t)block * 256 + threadIdx.x; t < total; t += (int64_t)nblocks * 256) {
    const int64_t i = t / dpad;
    const int j = (int)(t - i * dpad);
    float v = 0.f;
    if (j < d) v = transpose ? src[(int64_t)j * lds + i] : src[i * lds + j];
    dst[i * ldd + j] = v;
  }
}
__global__ void __launch_bounds__(256) pad_copy_kernel(const float *src, int64_t lds, int64_t n, int32_t d, float *dst,
                                                       int64_t ldd, int32_t dpad, int32_t transpose) {
  pad_copy(src, lds, n, d, dst, ldd, dpad, transpose, blockIdx.x, gridDim.x);
}
hipError_t launch_pad_copy(const float *src, int64_t lds, int64_t n, int32_t d, float *dst, int64_t ldd, int32_t dpad,
                           int32_t transpose, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n * dpad + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(pad_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, st, src, lds, n, d, dst, ldd, dpad,
                     transpose);
  return hipGetLastError();
}

// ------------------------------------------------------------------ what opens a call
// Both padded copies of the rotation matrix, the transposed one through a 32 x 33 tile in LDS, and its largest magnitude
// in one pass (a copy each and a pass for the bound before: with d = 128 three launches of 4 us for 64 KB).
// (four tiles a workgroup: every workgroup may raise the one word of the bound, 10 ns each)
constexpr int kOperandTiles = 4;
__device__ inline void rotation_operands(const float *R, int32_t d, float *Rp, float *Rtp, int32_t ld, unsigned int *absmax, int bx, int by) {
  __shared__ float s_t[kOperandTiles][32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int c0 = bx * 32;
  float m = 0.f;
#pragma unroll
  for (int q = 0; q < kOperandTiles; ++q) {
    const int r0 = (by * kOperandTiles + q) * 32;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = r0 + ty + 8 * u, c = c0 + tx;
      const float v = r < d && c < d ? R[(int64_t)r * d + c] : 0.f;
      s_t[q][ty + 8 * u][tx] = v;
      m = fmaxf(m, fabsf(v));
      if (Rp && r < d && c < ld) Rp[(int64_t)r * ld + c] = v;
    }
  }
  __syncthreads();
  if (Rtp)
#pragma unroll
    for (int q = 0; q < kOperandTiles; ++q) {
      const int r0 = (by * kOperandTiles + q) * 32;
#pragma unroll
      for (int u = 0; u < 4; ++u) {   // row c0 + .. of R^T
        const int r = c0 + ty + 8 * u, c = r0 + tx;
        if (r < d && c < ld) Rtp[(int64_t)r * ld + c] = s_t[q][tx][ty + 8 * u];
      }
    }
  block_absmax(m, absmax);
}
// One workgroup does a part of one job.  The long one comes first: its workgroups are then placed evenly and the short
// ones run beside them (last, on whichever CUs the short ones had left, 460 366 x 817 and 1653 centroids took 499 us instead of 252).  A launch behind another costs
// 3 to 5 us whatever it does: whole calls, with the pair of products of gemm.hip, 64 rows of 128 dimensions 210 -> 188 us, 20 000
// of 1536 888 -> 832, exact assignment of 100 003 of 100 127 -> 118.
// A bound takes one workgroup a CU and eight loads in flight: what it costs beside its bytes is its workgroups, which meet at one
// word.  The launch of 20 000 x 1536 and 1024 centroids 43.9 -> 39.2 us with two and four, 100 003 x 100 11.5 -> 9.2, 2.5M x 384 623 ->
// 618 (two and eight 42.5, 12.3 and 638; four and four 49, 21 and 639; one and sixteen 36.5, 11.9 and 618).
constexpr int kBoundLoads = 8;
struct OpeningGrid {
  int ops_x = 0, ops = 0, bound[2] = {0, 0}, pad = 0, fill = 0;   // workgroups of every job
};
__global__ void __launch_bounds__(256) opening_kernel(OpeningJobs j, OpeningGrid g) {
  int b = blockIdx.x;
  if (b < g.bound[0]) return absmax_flat<kBoundLoads>(j.bound[0].A, j.bound[0].count, j.bound[0].out, b, g.bound[0]);
  b -= g.bound[0];
  if (b < g.ops) return rotation_operands(j.R, j.d, j.Rp, j.Rtp, j.ld, j.r_bound, b % g.ops_x, b / g.ops_x);
  b -= g.ops;
  if (b < g.bound[1]) return absmax_flat<kBoundLoads>(j.bound[1].A, j.bound[1].count, j.bound[1].out, b, g.bound[1]);
  b -= g.bound[1];
  if (b < g.pad) return pad_copy(j.src, j.lds, j.rows, j.cols, j.dst, j.ldd, j.dpad, 0, b, g.pad);
  b -= g.pad;
  for (int64_t i = (int64_t)b * 256 + threadIdx.x; i < j.nfill; i += (int64_t)g.fill * 256) j.fill[i] = ~0ull;
}
hipError_t launch_opening(const OpeningJobs &j, hipStream_t st) {
  OpeningGrid g;
  if (j.R) {
    g.ops_x = (j.ld + 31) / 32;
    g.ops = g.ops_x * ((g.ops_x + kOperandTiles - 1) / kOperandTiles);
  }
  for (int u = 0; u < 2; ++u) {
    if (!j.bound[u].out) continue;
    if (j.bound[u].count < 4) return hipErrorInvalidValue;
    g.bound[u] = (int)std::min<int64_t>((j.bound[u].count + 1024 * kBoundLoads - 1) / (1024 * kBoundLoads), num_cus());
  }
  if (j.dst) g.pad = (int)std::min<int64_t>((j.rows * j.dpad + 255) / 256, (int64_t)num_cus() * 16);
  if (j.fill) g.fill = (int)std::min<int64_t>((j.nfill + 255) / 256, (int64_t)num_cus() * 4);
  const int all = g.ops + g.bound[0] + g.bound[1] + g.pad + g.fill;
  if (all <= 0) return hipSuccess;
  hipLaunchKernelGGL(opening_kernel, dim3((unsigned)all), dim3(256), 0, st, j, g);
  return hipGetLastError();
}

}  // namespace skm
