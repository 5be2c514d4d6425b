// Incremental attention of the fp32 element type (Sec. 2, Eq. 6-7) on the fp32 matrix cores: fp32
// logits, running-max softmax and fp32 accumulation.
//
// A workgroup of 8 wavefronts owns 16 queries of one (user, head); wavefront w takes the 16-token
// sub-blocks w, w + 8, ... of the keys those queries see, and the 8 partial results are combined
// through LDS, so a call needs no workspace and no second launch.
//
// Operand flow: S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_16x16x4_f32.  Its k index is one
// lane group (lane / 16) per step, so a lane's 16-byte granule of 4 consecutive dims serves four
// steps (step j contracts the dims 16 s + 4 gq + j over the lane groups gq); the accumulator then
// holds 4 consecutive tokens of one query per lane, which are the four P.V steps' operands, and
// the pool's [dim][16 tokens] order of V makes the other operand one 16-byte load as well.
//
// Bound: latency for the few-thousand-key calls this type is used for (page id -> K/V -> scores,
// then the combination), and then the two wavefronts of a SIMD, whose products and weights take 0.85 us a sub-block at
// head_dim 32.  The next sub-block's K and V travel while one is computed, requested without a branch (behind a load that
// may not have been made the compiler waits for all of them), and the page ids of 64 sub-blocks came with one load; head_dim
// 64 is held to 128 registers, two workgroups a CU; the softmax form spills the lane's row offset for it, stored and read back once
// outside the keys' loop (recomputed instead, no scratch: calls of long histories 0.99 of the time, of 100 users and more 1.012 to 1.015;
// as 32 bits a lane 1.00 to 1.02 and 0.96 to 0.99).  us a layer, with a branch, a page id a sub-block and the library's exponential /
// now: 16 queries x 272 keys x 4 heads of 32 5.75 / 4.87 (73 with one wavefront per (query, head) and a scalar load per
// element), of 64 8.1 / 6.8, of 128 13.0 / 11.8; 30 x 3030 x 8 of 64 42.5 / 36.9; 40 x 1440 x 8 of 128 43.8 / 37.3; 100 users' 10 x
// 110 x 8 of 64 19.6 / 15.0.  Many users of a few keys are the plain kernel's (f32_takes_plain).
#include <math.h>

#include <type_traits>

#include "mts_internal.hpp"

namespace mts {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int kWaves = 8;
constexpr int kQ = 16;           // queries per workgroup
constexpr int kSub = 16;         // tokens per step of a wavefront

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// max over the 4 lanes that hold the same query (lane, lane^16, lane^32, lane^48)
template <typename F>
__device__ __forceinline__ float over_quad_rows(float v, F f) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_row_max(float v) {
  return over_quad_rows(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float quad_row_sum(float v) {
  return over_quad_rows(v, [](float a, float b) { return a + b; });
}

// Weights are at most 1, the largest logit's is 1: what is below the smallest normal number counts as 0.
__device__ __forceinline__ float exp2_of(float x) { return __builtin_amdgcn_exp2f(x); }

struct F32Args {                 // one argument, see TableWords
  PoolGeom g;
  const float* q;
  float* out;
  float scale, inv_norm;
};

template <int D, bool PW>
__global__ __launch_bounds__(64 * kWaves, D == 128 ? 2 : 4) void attn_f32_kernel(TableWords runs, TableWords pages, CallWords2 call, F32Args args) {
  const int32_t *new_indptr = table(runs[0]), *prefix_lens = table(runs[1]), *page_indptr = table(pages[0]),
                *page_indices = table(pages[1]);
  const int batch = call[0], total_new = call[1];
  const PoolGeom& g = args.g;
  const float* __restrict__ q = args.q;
  float* __restrict__ out = args.out;
  const float scale = args.scale, inv_norm = args.inv_norm;
  // Softmax: references are raw logits, and a weight is 2^(c (z - m)), c = scale log2(e): exactly 1 at the reference, however
  // large the logits are.  (As 2^(c z - m) by one fma, m the rounded c z of the largest, that one's exponent is off by up to half a
  // unit in the last place of c z, and from 2^31 on its weight infinite or 0.  us a layer so / now: 16 queries x 272 keys x 4 heads
  // of 32 4.82 / 4.87, of 64 6.85 / 6.82, of 128 11.2 / 11.8; eleven other calls within 0.7 %.)  Against 64 bits, 24 random
  // calls of 32 to 1900 keys: 4.47e-7 (geometric mean), with the scaled logit, its difference and the library's exponential 4.48e-7.
  const float c = scale * 1.4426950408889634f;
  constexpr int NF = D / 16;       // 16-byte fragments per lane of a sub-block's K, V, of Q and of the output
  __shared__ f32x4 s_o[kWaves / 2][NF][64];
  __shared__ float s_m[kWaves / 2][kQ], s_l[kWaves / 2][kQ];

  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
  const int r = lane & 15, gq = lane >> 4;
  const int H = g.H, S = g.S, h = blockIdx.y;

  // Blocks of user u start at new_indptr[u] / 16 + u: at least ceil(n_u / 16) of them before the next
  // user's, so no prefix sum over the users is needed and the grid stays below total_new / 16 + batch.
  const int blk = blockIdx.x;
  int lo = 0, hi = batch;
  while (hi - lo > 1) {                                 // largest u that starts at or before blk
    const int mid = (lo + hi) >> 1;
    if (new_indptr[mid] / kQ + mid <= blk) lo = mid; else hi = mid;
  }
  const int u = lo, tok0 = new_indptr[u];
  const int n_u = new_indptr[u + 1] - tok0;
  const int q0 = (blk - (tok0 / kQ + u)) * kQ;
  if (q0 < 0 || q0 >= n_u || tok0 + q0 >= total_new) return;    // workgroup-uniform
  const int P = prefix_lens[u];
  const int pbeg = page_indptr[u], npg = page_indptr[u + 1] - pbeg;
  int nq = n_u - q0 < kQ ? n_u - q0 : kQ;
  nq = nq < total_new - tok0 - q0 ? nq : total_new - tok0 - q0;
  const int kv_len = P + q0 + nq;                       // keys the last query sees
  const int n_sb = (kv_len + kSub - 1) / kSub;
  const int sub_mask = (1 << g.sub_shift) - 1;
  const char* head_base = g.layer_base + (int64_t)h * 2 * S * D * 4;
  const int64_t v_off = (int64_t)S * D * 4;

  // lane (r, gq): query q0 + r, dims 16 s + 4 gq .. + 3
  f32x4 qf[NF];
#pragma unroll
  for (int s = 0; s < NF; ++s) {
    qf[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (r < nq) qf[s] = *reinterpret_cast<const f32x4*>(q + ((int64_t)(tok0 + q0 + r) * H + h) * D + 16 * s + 4 * gq);
  }

  // The wavefront's i-th sub-block is number wave + 8 i; a lane holds the page of one, 64 of them at a time.
  const int n_mine = n_sb > wave ? (n_sb - wave - 1) / kWaves + 1 : 0;
  int ids = -1;
  auto load_ids = [&](int first) __attribute__((always_inline)) {
    const int sb = wave + kWaves * (first + lane), lp = sb >> g.sub_shift;
    ids = sb < n_sb && lp < npg ? page_indices[pbeg + lp] : -1;
  };
  f32x4 kf[2][NF], vf[2][NF];
  bool held[2];                                         // the sub-block's page exists
  auto load = [&](auto slot_c, int i) __attribute__((always_inline)) {
    constexpr int p = decltype(slot_c)::value;
    const int sb = wave + kWaves * i;
    int page = __builtin_amdgcn_readlane(ids, i & 63);
    held[p] = (unsigned)page < (unsigned)g.num_pages;
    page = held[p] ? page : 0;                          // no branch: behind a load that may not have been made all are waited for
    const char* kb = head_base + (int64_t)page * g.page_bytes + (int64_t)(sb & sub_mask) * kSub * D * 4;
    // K rows are the tokens in order: token r lies at half (r / 4) % 2, slot (r / 8) * 4 + r % 4
    const char* kl = kb + ((((r >> 2) & 1) * (D / 4) + gq) * 8 + ((r >> 3) << 2) + (r & 3)) * 16;
    const char* vl = kb + v_off + (r * 16 + 4 * gq) * 4;      // dim 16 db + r, tokens 4 gq .. + 3
#pragma unroll
    for (int s = 0; s < NF; ++s) kf[p][s] = *reinterpret_cast<const f32x4*>(kl + s * 4 * 8 * 16);
#pragma unroll
    for (int s = 0; s < NF; ++s) vf[p][s] = *reinterpret_cast<const f32x4*>(vl + s * 16 * 16 * 4);
  };

  f32x4 o[NF];
#pragma unroll
  for (int s = 0; s < NF; ++s) o[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;                         // l: this lane's tokens only
  auto compute = [&](auto slot_c, int i) __attribute__((always_inline)) {
    constexpr int p = decltype(slot_c)::value;
    const int sb = wave + kWaves * i;
    if (!held[p]) return;
    f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NF; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) z = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[p][s][j], qf[s][j], z, 0, 0, 0);
    const int tb = sb * kSub;
    const int visible = P + q0 + r + 1 - (tb + 4 * gq);  // of this lane's 4 tokens, the first `visible`
    f32x4 w;
    if constexpr (PW) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = z[e] * scale;
        w[e] = (e >= visible || x == -INFINITY) ? 0.f : x / (1.0f + expf(-x));   // silu; hidden keys weigh 0
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = e < visible ? z[e] : -INFINITY;
      const float m_new = fmaxf(m, quad_row_max(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]))));
      const float m_ref = m_new == -INFINITY ? 0.f : m_new;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = exp2_of((z[e] - m_ref) * c);
      const float alpha = exp2_of((m - m_ref) * c);
      l = l * alpha + ((w[0] + w[1]) + (w[2] + w[3]));
      m = m_new;
#pragma unroll
      for (int s = 0; s < NF; ++s) o[s] *= alpha;
    }
    if (tb + kSub > P + q0 + 1) {
      // The causal tail: some query must not see some token here.  A weight of 0 does not cancel an
      // infinity or a NaN, so values that not every query sees are finite or are added one by one,
      // and slots past the user's last token (they may hold anything) are cleared.
      bool finite = true;
#pragma unroll
      for (int s = 0; s < NF; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (tb + 4 * gq + j >= P + n_u) vf[p][s][j] = 0.f;
          finite &= fabsf(vf[p][s][j]) < INFINITY;
        }
      if (__builtin_amdgcn_ballot_w64(!finite) != 0) {
#pragma unroll 1
        for (int tg = 0; tg < 4; ++tg)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float wt = __shfl(w[j], r + 16 * tg);                   // token 4 tg + j of query r
            const bool seen = tb + 4 * tg + j <= P + q0 + r;
#pragma unroll
            for (int s = 0; s < NF; ++s)
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                const float vt = __shfl(vf[p][s][j], 4 * gq + k + 16 * tg);
                if (seen) o[s][k] = fmaf(wt, vt, o[s][k]);
              }
          }
        return;
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int s = 0; s < NF; ++s) o[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[p][s][j], w[j], o[s], 0, 0, 0);
  };

  constexpr std::integral_constant<int, 0> slot0{};
  constexpr std::integral_constant<int, 1> slot1{};
  if (n_mine > 0) {
    load_ids(0);
    load(slot0, 0);
    int i = 0;
    for (; i + 1 < n_mine; ++i) {
      if (((i + 1) & 63) == 0) load_ids(i + 1);
      load(slot1, i + 1);
      compute(slot0, i);
#pragma unroll
      for (int s = 0; s < NF; ++s) { kf[0][s] = kf[1][s]; vf[0][s] = vf[1][s]; }
      held[0] = held[1];
    }
    compute(slot0, i);
  }

  // Combination, in wavefront order: wavefronts 4-7 hand theirs to 0-3, whose sums every thread then
  // folds for its share of the 16 x D outputs.
  auto put = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < NF; ++s) s_o[slot][s][lane] = o[s];
    if (!PW && gq == 0) { s_m[slot][r] = m; s_l[slot][r] = l; }
  };
  if (!PW) l = quad_row_sum(l);
  if (wave >= kWaves / 2) put(wave - kWaves / 2);
  __syncthreads();
  if (wave < kWaves / 2) {
    float wa = 1.f, wb = 1.f;
    if (!PW) {
      const float mb = s_m[wave][r], mn = fmaxf(m, mb), m_ref = mn == -INFINITY ? 0.f : mn;
      wa = exp2_of((m - m_ref) * c);
      wb = exp2_of((mb - m_ref) * c);
      l = l * wa + s_l[wave][r] * wb;
      m = mn;
    }
#pragma unroll
    for (int s = 0; s < NF; ++s) o[s] = o[s] * wa + s_o[wave][s][lane] * wb;
    put(wave);                                           // the slot that this wavefront alone has just read
  }
  __syncthreads();
  for (int e = threadIdx.x; e < NF * 64; e += 64 * kWaves) {
    const int s = e >> 6, ln = e & 63, qi = ln & 15;     // dims 16 s + 4 (ln / 16) .. + 3 of query qi
    if (qi >= nq) continue;
    float wgt[kWaves / 2], den = 0.f;
    float mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves / 2; ++w) mx = PW ? 0.f : fmaxf(mx, s_m[w][qi]);
    if (mx == -INFINITY) mx = 0.f;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves / 2; ++w) {
      wgt[w] = PW ? 1.f : exp2_of((s_m[w][qi] - mx) * c);
      if (!PW) den = fmaf(wgt[w], s_l[w][qi], den);
      sum += s_o[w][s][ln] * wgt[w];
    }
    f32x4 res;
#pragma unroll
    for (int k = 0; k < 4; ++k) res[k] = PW ? sum[k] * inv_norm : sum[k] / den;
    *reinterpret_cast<f32x4*>(out + ((int64_t)(tok0 + q0 + qi) * H + h) * D + 16 * s + 4 * (ln >> 4)) = res;
  }
}

template <int D>
void launch_d(dim3 grid, const PoolGeom& g, const BatchDev& b, const float* q, float* out, float scale, float inv_norm,
              hipStream_t stream) {
  auto kern = inv_norm > 0.f ? attn_f32_kernel<D, true> : attn_f32_kernel<D, false>;
  hipLaunchKernelGGL(kern, grid, dim3(64 * kWaves), 0, stream, run_tables(b), page_tables(b), CallWords2{b.batch, b.total_new},
                     F32Args{g, q, out, scale, inv_norm});
}

}  // namespace

hipError_t launch_attn_f32(const PoolGeom& g, const void* q, void* out, const BatchDev& b, float sm_scale,
                           float inv_norm, hipStream_t stream) {
  if (b.total_new <= 0 || b.batch <= 0) return hipSuccess;
  const dim3 grid((unsigned)(b.total_new / kQ + b.batch), (unsigned)g.H, 1);
  const float* qp = static_cast<const float*>(q);
  float* op = static_cast<float*>(out);
  switch (g.D) {
    case 32: launch_d<32>(grid, g, b, qp, op, sm_scale, inv_norm, stream); break;
    case 64: launch_d<64>(grid, g, b, qp, op, sm_scale, inv_norm, stream); break;
    case 128: launch_d<128>(grid, g, b, qp, op, sm_scale, inv_norm, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace mts
