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

// A numerically safe weighted sum of a pair's pieces in a fixed order (deterministic).  Share
// w_first holds its piece in slot `first_slot`; every later share holds its piece as the leading
// one (slot 0).  One descriptor per blockIdx.x; a thread folds the 4 dims `d4` of one query,
// taking pieces four at a time with all their loads issued together.
template <int D, bool PW>
__global__ __launch_bounds__(256) void attn_merge_kernel(uint16_t* __restrict__ out, float c, float inv_norm, int q_tile,
                                                         int H, const MergeDesc* __restrict__ ws_desc,
                                                         const float* __restrict__ ws_o,
                                                         const float* __restrict__ ws_ml) {
  const MergeDesc d = ws_desc[blockIdx.x];
  constexpr int D4 = D / 4;
  const int e = blockIdx.y * 256 + threadIdx.x;
  if (!d.valid || e >= d.nq * D4) return;
  const int qi = e / D4, d4 = e % D4;
  float M = -INFINITY, den = 0.f;
  merge_f32x4 num = {0.f, 0.f, 0.f, 0.f};
  for (int w0 = d.w_first; w0 <= d.w_last; w0 += 4) {
    float pm[4], pl[4];
    merge_f32x4 po[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int ww = (w0 + k <= d.w_last) ? (w0 + k) : d.w_last;      // past the end: repeat, weight 0
      const int slot = (ww == d.w_first) ? d.first_slot : 0;
      const int64_t prow = ((int64_t)ww * 2 + slot) * q_tile + qi;
      pm[k] = PW ? 0.f : ws_ml[prow * 2];
      pl[k] = PW ? 0.f : ws_ml[prow * 2 + 1];
      po[k] = *reinterpret_cast<const merge_f32x4*>(ws_o + prow * D + 4 * d4);
    }
    float Mn = M;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (w0 + k <= d.w_last) Mn = fmaxf(Mn, pm[k]);
    const float mref = (Mn == -INFINITY) ? 0.f : Mn;
    const float rescale = __builtin_amdgcn_exp2f((M - mref) * c);      // 0 while nothing was folded in
    num *= rescale;
    den *= rescale;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (w0 + k <= d.w_last) {
        const float wgt = __builtin_amdgcn_exp2f((pm[k] - mref) * c);  // a piece with no visible key has max -inf
        num += po[k] * wgt;
        den = fmaf(wgt, pl[k], den);
      }
    }
    M = Mn;
  }
  // pointwise: every piece has reference 0, so the weights above are all 1 and num is the plain sum
  const float inv = PW ? inv_norm : 1.0f / den;
  merge_bf16x4 ob;
#pragma unroll
  for (int k = 0; k < 4; ++k) ob[k] = (__bf16)(num[k] * inv);
  *reinterpret_cast<merge_bf16x4*>(out + ((int64_t)d.out_row + (int64_t)qi * H) * D + 4 * d4) = ob;
}

}  // namespace merge_detail
}  // namespace mts
