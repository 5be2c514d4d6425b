// Finishing pass of the split-kv attention kernels: the pieces of a (query tile, head) that share
// boundaries cut are combined into its output rows.
#pragma once
#include <math.h>

#include "mts_internal.hpp"

namespace mts {
namespace merge_detail {

typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 merge_bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float merge_f32x4;

// What is needed to finish one (query tile, head) cut by share boundaries; written by the share
// that holds the pair's first tile.
struct MergeDesc {
  int valid;       // 1: a cut pair
  int w_first;     // first share that holds a piece of it
  int w_last;      // last share that holds a piece of it
  int out_row;     // (token row of the tile's first query) * H + head
  int nq;          // queries in the tile
  int first_slot;  // partial slot of the first share's piece (0 leading, 1 trailing)
  int pad[2];
};

// Above these, a softmax denominator or the absolute sum of a query's accumulators asks for a redo with the
// exact max.  A piece's are lower by the number of pieces that a pair can be cut into, so that the sums
// over pieces of one reference stay within fp32 too.
struct RedoLimits { float den, mag; };
constexpr RedoLimits redo_limits(bool cut) {
  static_assert(kAttnMaxWaves <= 1024 && kPrefillMaxWgs <= 1024, "a share holds at most one piece of a pair");
  return cut ? RedoLimits{1e37f / 1024, 3.0e38f / 1024} : RedoLimits{1e37f, 3.0e38f};
}

// What a row's logits are multiplied with ahead of the exponential.  A weight is 2^(c x - R) by one fma, x a logit and R the
// rounded c m of the reference m, so that the reference's own weight is off 1 by up to half a unit in the last place of R
// in its exponent: 2^16 at |R| = 2^29, and from 2^31 on infinite or 0, the row NaN.  From 2^29 on the factor is a power of two
// with which c m lies in 2^30 .. 2^31: its product with every logit is exact, and what is less than m weighs 2^-128 and less,
// where c gives 2^-32 and less.  (c (x - m) instead, an instruction more a score: 1.00 to 1.04 of the time of staged calls.  A factor a
// row instead of a call, 136 calls: 1.001 in the mean, 0.98 to 1.02.)
__device__ __forceinline__ float row_scale(float m, float c) {
  return fabsf(m) * c < 536870912.f ? c : __uint_as_float((284 - (__float_as_uint(m) >> 23 & 255)) << 23);
}

// A numerically safe weighted sum of a pair's pieces in a fixed order (deterministic).  Share
// w_first holds its piece in slot `first_slot`; every later share holds its piece as the leading
// one (slot 0).  A thread folds the 4 dims `d4` of one query, taking pieces four at a time with all
// their loads issued together.
//
// PG = 1: one descriptor per blockIdx.x, all its pieces folded by one thread per 4 dims.
// PG > 1, for calls of a few long pairs cut into many pieces (one user's 6 K history, 4 pairs of 50
// pieces: 12.6 us folded serially, the whole call 27 us; 18.5 us with 8 groups): the pieces are dealt to PG groups of
// threads in contiguous runs and the groups' sums folded through LDS in group order.
// A block looks at DESCS neighbouring descriptors: one where there is a descriptor per pair (launches of pieces) or
// most of them are filled, else four, of which a call of few long pairs fills few.
// FRAGS: a piece lies in the fragment order of the prefill kernel's accumulators (32 queries x 32 dims: 4 x 64 lanes of 4
// dims), else row by row.
template <int D, bool PW, int PG, bool FRAGS, int DESCS>
__global__ __launch_bounds__(256) void attn_merge_kernel(uint16_t* __restrict__ out, float c, float inv_norm, int q_tile,
                                                         int H, int n_desc, const MergeDesc* __restrict__ ws_desc,
                                                         const float* __restrict__ ws_o,
                                                         const float* __restrict__ ws_ml) {
  constexpr int D4 = D / 4, kCols = 256 / PG, kDescs = DESCS;
  __shared__ merge_f32x4 s_num[PG > 1 ? 256 : 1];
  __shared__ float s_m[PG > 1 ? 256 : 1], s_den[PG > 1 ? 256 : 1];
  const int grp = threadIdx.x / kCols, e = blockIdx.y * kCols + threadIdx.x % kCols;
  const int qi = FRAGS ? e / (256 * (D / 32)) * 32 + (e & 31) : e / D4;
  const int d4 = FRAGS ? (e >> 8) % (D / 32) * 8 + (e >> 6 & 3) * 2 + (e >> 5 & 1) : e % D4;
  for (int k = 0; k < kDescs; ++k) {
    const int wd = blockIdx.x * kDescs + k;
    if (DESCS > 1 && wd >= n_desc) return;
    const MergeDesc d = ws_desc[wd];
    if (!d.valid || (int)blockIdx.y * kCols >= (FRAGS ? (d.nq + 31) / 32 * 32 : d.nq) * D4) continue;      // workgroup-uniform
    const bool mine = qi < d.nq;
    const int per = (d.w_last - d.w_first + PG) / PG;                     // pieces per group, rounded up
    const int wa = d.w_first + grp * per, wz = wa + per - 1 < d.w_last ? wa + per - 1 : d.w_last;
    float M = -INFINITY, den = 0.f;
    merge_f32x4 num = {0.f, 0.f, 0.f, 0.f};
    if (mine) {
      for (int w0 = wa; w0 <= wz; w0 += 4) {
        float pm[4], pl[4];
        merge_f32x4 po[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int ww = (w0 + k <= wz) ? (w0 + k) : wz;                  // past the end: repeat, weight 0
          const int slot = (ww == d.w_first) ? d.first_slot : 0;
          const int64_t piece = ((int64_t)ww * 2 + slot) * q_tile, prow = piece + qi;
          pm[k] = PW ? 0.f : ws_ml[prow * 2];
          pl[k] = PW ? 0.f : ws_ml[prow * 2 + 1];
          po[k] = *reinterpret_cast<const merge_f32x4*>(ws_o + (FRAGS ? piece * D + 4 * e : prow * D + 4 * d4));
        }
        asm volatile("" ::: "memory");                                    // all of them are on their way before the first is waited for
        float Mn = M;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (w0 + k <= wz) Mn = fmaxf(Mn, pm[k]);
        const float mref = (Mn == -INFINITY) ? 0.f : Mn;
        const float rescale = __builtin_amdgcn_exp2f((M - mref) * c);     // 0 while nothing was folded in
        num *= rescale;
        den *= rescale;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (w0 + k <= wz) {
            const float wgt = __builtin_amdgcn_exp2f((pm[k] - mref) * c); // a piece with no visible key has max -inf
            num += po[k] * wgt;
            den = fmaf(wgt, pl[k], den);
          }
        }
        M = Mn;
      }
    }
    if constexpr (PG > 1) {
      s_num[threadIdx.x] = num;
      s_m[threadIdx.x] = M;
      s_den[threadIdx.x] = den;
      __syncthreads();
      if (grp == 0) {
        float Mx = M;
#pragma unroll
        for (int p = 1; p < PG; ++p) Mx = fmaxf(Mx, s_m[threadIdx.x + p * kCols]);
        const float mref = (Mx == -INFINITY) ? 0.f : Mx;
        const float own = PW ? 1.f : __builtin_amdgcn_exp2f((M - mref) * c);
        num *= own;
        den *= own;
#pragma unroll
        for (int p = 1; p < PG; ++p) {
          const int i = threadIdx.x + p * kCols;
          const float wgt = PW ? 1.f : __builtin_amdgcn_exp2f((s_m[i] - mref) * c);
          num += s_num[i] * wgt;
          den = fmaf(wgt, s_den[i], den);
        }
      }
      __syncthreads();                                                    // the next descriptor's sums may be put
    }
    if (mine && grp == 0) {
      // pointwise: every piece has reference 0, so the weights above are all 1 and num is the plain sum
      const float inv = PW ? inv_norm : 1.0f / den;
      merge_bf16x4 ob;
#pragma unroll
      for (int k = 0; k < 4; ++k) ob[k] = (__bf16)(num[k] * inv);
      *reinterpret_cast<merge_bf16x4*>(out + ((int64_t)d.out_row + (int64_t)qi * H) * D + 4 * d4) = ob;
    }
  }
}

// The same of pieces in fragment order, for calls of many pairs: a workgroup folds 32 queries x 64 dims of every piece, two
// vectors a thread, and lays the rows out in LDS, so that they are stored in runs of 128 bytes (8 bytes here and there
// instead: 14.3 us against 11.0 for the 160 cut blocks of one user's 5189 tokens x 4 heads of 128, 40 MB of pieces; four vectors
// a thread 11.2).  Bound: reading the pieces, which lie past the L2 that wrote them.
constexpr int kFragDims = 64;
template <int D, bool PW>
__global__ __launch_bounds__(256) void attn_merge_frags_kernel(uint16_t* __restrict__ out, float c, float inv_norm, int q_tile,
                                                               int H, const MergeDesc* __restrict__ ws_desc,
                                                               const float* __restrict__ ws_o,
                                                               const float* __restrict__ ws_ml) {
  constexpr int V = kFragDims / 32, kDims = kFragDims, kParts = D / kDims;           // 32 queries x kDims dims a workgroup
  constexpr int PITCH = kDims + 8;
  __shared__ __attribute__((aligned(16))) uint16_t rows[32 * PITCH];
  // the XCD that wrote a share's pieces merges them (11.6 -> 11.2 us)
  const int wd = gridDim.x % 8 == 0 ? (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
  const MergeDesc d = ws_desc[wd];
  const int q_base = blockIdx.y / kParts * 32, dim_base = blockIdx.y % kParts * kDims;
  if (!d.valid || q_base >= d.nq) return;                                 // workgroup-uniform
  const int r = threadIdx.x & 31, dim8 = threadIdx.x >> 6, hf = threadIdx.x >> 5 & 1;
  const int qi = q_base + r < d.nq ? q_base + r : q_base;                 // rows past the last were not written
  float M = -INFINITY, den = 0.f;
  merge_f32x4 num[V];
#pragma unroll
  for (int v = 0; v < V; ++v) num[v] = merge_f32x4{0.f, 0.f, 0.f, 0.f};
  for (int w0 = d.w_first; w0 <= d.w_last; w0 += 4) {
    float pm[4], pl[4];
    merge_f32x4 po[4][V];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int ww = (w0 + k <= d.w_last) ? (w0 + k) : d.w_last;          // past the end: repeat, weight 0
      const int64_t piece = ((int64_t)ww * 2 + (ww == d.w_first ? d.first_slot : 0)) * q_tile;
      pm[k] = PW ? 0.f : ws_ml[(piece + qi) * 2];
      pl[k] = PW ? 0.f : ws_ml[(piece + qi) * 2 + 1];
#pragma unroll
      for (int v = 0; v < V; ++v)
        po[k][v] = *reinterpret_cast<const merge_f32x4*>(ws_o + piece * D + ((int64_t)(blockIdx.y * V + v) * 256 + threadIdx.x) * 4);
    }
    asm volatile("" ::: "memory");                                        // all of them are on their way before the first is waited for
    float Mn = M;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (w0 + k <= d.w_last) Mn = fmaxf(Mn, pm[k]);
    const float mref = (Mn == -INFINITY) ? 0.f : Mn;
    const float rescale = __builtin_amdgcn_exp2f((M - mref) * c);         // 0 while nothing was folded in
    den *= rescale;
#pragma unroll
    for (int v = 0; v < V; ++v) num[v] *= rescale;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (w0 + k <= d.w_last) {
        const float wgt = __builtin_amdgcn_exp2f((pm[k] - mref) * c);
#pragma unroll
        for (int v = 0; v < V; ++v) num[v] += po[k][v] * wgt;
        den = fmaf(wgt, pl[k], den);
      }
    }
    M = Mn;
  }
  const float inv = PW ? inv_norm : 1.0f / den;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    merge_bf16x4 ob;
#pragma unroll
    for (int k = 0; k < 4; ++k) ob[k] = (__bf16)(num[v][k] * inv);
    *reinterpret_cast<merge_bf16x4*>(rows + r * PITCH + 32 * v + 8 * dim8 + 4 * hf) = ob;
  }
  __syncthreads();
  typedef __attribute__((__vector_size__(16))) unsigned u32x4;
  for (int e = threadIdx.x; e < 32 * (kDims / 8); e += 256) {
    const int row = e / (kDims / 8), ch = e % (kDims / 8);
    if (q_base + row < d.nq)
      *reinterpret_cast<u32x4*>(out + ((int64_t)d.out_row + (int64_t)(q_base + row) * H) * D + dim_base + 8 * ch) =
          *reinterpret_cast<const u32x4*>(rows + row * PITCH + 8 * ch);
  }
}

// `shares` descriptors of at most `pairs` cut pairs, or (`per_pair`) one of each.  Eight or more shares per pair: the pieces of a
// pair are many and its pairs few, so they are folded by groups.
template <int D, bool PW, bool FRAGS = false>
hipError_t launch_merge(uint16_t* out, float c, float inv_norm, int q_tile, int H, int shares, int64_t pairs,
                        const MergeDesc* ws_desc, const float* ws_o, const float* ws_ml, hipStream_t stream,
                        bool per_pair = false) {
  constexpr int kGroups = 8;
  const int cols = q_tile * (D / 4);
  const int descs = per_pair ? (int)pairs : shares;
  if (shares >= 8 * pairs) {
    constexpr int kGroupCols = 256 / kGroups;
    auto kern = per_pair ? attn_merge_kernel<D, PW, kGroups, FRAGS, 1> : attn_merge_kernel<D, PW, kGroups, FRAGS, 4>;
    hipLaunchKernelGGL(kern, dim3(per_pair ? descs : (descs + 3) / 4, (cols + kGroupCols - 1) / kGroupCols), dim3(256), 0, stream, out, c,
                       inv_norm, q_tile, H, descs, ws_desc, ws_o, ws_ml);
  } else if constexpr (FRAGS) {
    hipLaunchKernelGGL((attn_merge_frags_kernel<D, PW>), dim3(descs, q_tile / 32 * (D / kFragDims)), dim3(256), 0, stream, out, c, inv_norm,
                       q_tile, H, ws_desc, ws_o, ws_ml);
  } else {
    hipLaunchKernelGGL((attn_merge_kernel<D, PW, 1, FRAGS, 1>), dim3(descs, (cols + 255) / 256), dim3(256), 0, stream, out, c,
                       inv_norm, q_tile, H, descs, ws_desc, ws_o, ws_ml);
  }
  return hipGetLastError();
}

}  // namespace merge_detail
}  // namespace mts
