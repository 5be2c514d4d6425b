// Cache-miss / long-segment prefill attention on the matrix cores: the same operation as the
// streaming kernel (Sec. 2, Eq. 6-7; with no cached prefix it is the causal attention of the
// recompute baseline, Sec. 5.1), laid out for the case of MANY new tokens per user, where the
// work is a dense contraction and K/V reuse across queries decides the speed.
//
// A workgroup (4 wavefronts) owns one (user, head, block of 128*NQ new tokens): wavefront w takes
// queries 32*NQ*w .. 32*NQ*(w+1)-1 of the block.  All four walk the same kv tiles, so each 32-token
// K/V tile is fetched from global memory ONCE per workgroup: every wavefront moves a quarter of it
// straight into LDS (16 bytes per lane, no registers), in an order from which all reads back are whole, conflict-free
// operands.  A wavefront's quarter comes from one of the tile's two 16-token sub-blocks, at an address that is one for all
// lanes, and lies as far apart in LDS as in the page: one page id, one multiplication and two m0 a step, and four loads with
// nothing between them.  (Quarters that took both sub-blocks, with 64-bit addresses a lane: 80 instructions more in two
// steps, which at the power limit cost time whatever they overlap with: 1168 -> 1095 us for the call below, one user of 5189
// tokens x 4 heads 49.6 -> 47.6, split and merged.)
// The block's page ids are copied to LDS once, so that no load in the loop depends on another load.
//
// Operand flow: S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x16_bf16; queries are the columns,
// so a lane's 16 scores belong to ONE query, and the order in which a tile's tokens are the rows of
// S^T makes them 8 consecutive tokens of either sub-block: the two operands of P.V without a shuffle.
//
// Pipeline: a stage of the three in LDS holds the values of tile t and the keys of tile t+2.  Step t
// fetches the stage of step t+2, reads its values, multiplies the keys of tile t+1 (in registers since
// the step before) while the vector units take the weights of tile t, then reads the keys of tile t+2
// while the matrix cores work on P.V.  One barrier per step, across which the newest fetch stays in
// flight.
//
// Bound: on random data the chip's power.  16 users x 4096 tokens x 16 heads of 128, one layer: 1014 to
// 1095 us on several cards (1004-1085 TFLOP/s), 780 us on zeros; a library matrix product of 8192^3
// reaches 1250 TFLOP/s here.  With v_mfma_f32_16x16x32_bf16, tiles parked from registers and no
// pipelining across tiles the same call took 1163 to 1200 us (1018 on zeros), 64-dim heads 697 (628
// now).  Tried and slower: 256-query blocks of eight wavefronts (1192 against 1162), raised wavefront priority around the
// matrix work (1-3 %); 64 queries of 128 dims a wavefront, one wavefront a SIMD, matrix and vector instructions dealt out
// one by one (957 on zeros, 1072 to 1127 on random data where this one took 1095; split calls 1.25 times as long).
//
// The softmax reference is fixed, as in the streaming kernel (max of the block's first tile, no
// rescaling; an overflowed denominator makes the whole workgroup redo its block, or its piece of a cut
// one, with the exact max, found by a K-only pass); the denominator sums the rounded weights in fp32
// (v_dot2_f32_bf16 against ones).  Workgroups of one (user, head) land on one XCD, longest block first,
// so that its K/V stays in that XCD's L2 while the blocks re-read it.
//
// SPLIT is the form for calls that would leave the chip idle that way: a single first-time user
// (fewer blocks than CUs, the longest of them the whole launch), or a batch in which some users
// have a few new tokens behind a long history.  The call's tile steps, ordered (user, head, block,
// tile), are one sequence; a persistent launch of two workgroups per CU gives each a contiguous
// share of it (the first on a CU a larger one, see kFirstShare), and a block that a share boundary cuts is written as unnormalised fp32
// pieces that a merge kernel finishes.  Every wavefront derives the schedule by itself from the
// device-resident lengths, in its lanes: a scan over the users, then searches by one comparison a lane
// (positions inside a user are closed forms).  Measured, attention and merge of one layer in a step, means of runs on
// several cards, head_dim 128, unsplit -> split: 1 user x 5189 new tokens x 4 heads 93 -> 45 to 50 us (merge 9.5); 6 users with
// 4-12 K histories and 8-64 new tokens beside 2 first-time ones 190 -> 82 to 92 us (merge 9.8).  What is left there is the block starts (1.2 and 1.5 segments
// a share, about 4 us each) and the fp32 pieces (64 KB each, about 40 and 47 MB written and read back).
//
// A block's start (page ids, keys, queries, reference, first scores) is 3.4 to 4 us, and a CU does little else before the
// first one is done.  It was 5.5, and 2 before it for the schedule, now 0.9: with a prefix sum in LDS, masks and
// addresses computed ahead of the redo loop into 200 spilled scalar registers, the page table's round trip
// before that of the keys, and queries loaded as fragments.  A piece's end took 2.3 us stored row by row, 1.4 in fragment order.  A step of 8 layers, by all of
// it: one user's 5189 tokens x 4 heads 488 -> 465 us (446 since a CU's two shares are unequal, 413 with all of the above), 16 x 4096 x 16 heads
// 10414 -> 10238 (9627).
//
// PW selects the pointwise aggregation out = inv_norm * sum_j silu(c * q.k_j) v_j: no reference
// max, no denominator, no redo; hidden keys carry logit 0 (silu(0) = 0).
#include <math.h>

#include <mutex>
#include <type_traits>

#include "mts_attn_merge.hpp"
#include "mts_attn_rules.hpp"
#include "mts_internal.hpp"

namespace mts {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;   // one 16-byte fragment
typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned u32x2;

using merge_detail::MergeDesc;

constexpr int kTile = 32;        // kv tokens per step
constexpr int kXcds = 8;
constexpr int kMaxIdBytes = 64 * 1024;   // LDS page table of one block
// The queries' own rooms (see the kernel) lie in the LDS of the page table from word `at` on: behind the table, but inside it
// where two workgroups have room on a CU only so, as with 98 to 131 K tokens at 16 a page in a split launch of head_dim 128.  The
// ids that lie there are then filled in when the queries have been read.  Behind any table, two users of 105 and 112 K tokens
// with 900 and 600 new x 8 heads took 941 us, one workgroup on a CU; so 830, and 861 before the queries came by way of LDS.
template <int D, bool BLOCK_REFERENCE>
struct QueryRooms {
  static constexpr int kFree = (BLOCK_REFERENCE ? 3 : 4) * (D / 64);  // rooms of a wavefront in the stages, of its eight
  static constexpr int kOwn = kFree < 8 ? 8 - kFree : 0, kWords = 4 * kOwn * 256;
  static constexpr int kTwo = (80 * 1024 - 3 * 32 * D * 4 - 64) / 4;  // words of a workgroup of two, with three stages and the flags
  static constexpr int at(int id_cap) {
    return id_cap > kTwo - kWords && id_cap <= kTwo ? kTwo - kWords : (id_cap + 3) & ~3;
  }
  static constexpr int64_t bytes(int id_cap) { return kOwn > 0 ? ((int64_t)at(id_cap) + kWords) * 4 : (int64_t)id_cap * 4; }
  static_assert(kTwo % 4 == 0 && kWords < kTwo, "16-byte rooms");
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float fast_silu(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + fast_exp2(-1.4426950408889634f * x));
}

// A wavefront-uniform element of an array that nothing writes while the kernel runs, by a scalar load.
__device__ __forceinline__ int scalar_load(const int32_t* p, int i) {
  typedef const __attribute__((address_space(4))) int32_t* scalar_ptr;
  return ((scalar_ptr)(uintptr_t)p)[i];
}

// over the 2 lanes that hold the same query (lane, lane^32)
__device__ __forceinline__ float pair_max(float v) {
  const unsigned u = __float_as_uint(v);
  auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float pair_sum(float v) {
  const unsigned u = __float_as_uint(v);
  auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// `N` times 16 bytes per lane from global memory, `from` + `lane_at` + k * STRIDE, to LDS byte address `to` (both
// wavefront-uniform) + k * STRIDE + 16 * lane, without passing through registers.  As instructions of its own because the
// compiler, given the builtin, waits for all such loads before any LDS read; here the waits are wait_and_barrier's.
// m0 is declared as overwritten, so that no value of the compiler's own is taken to outlive the statement in it; the
// warning says that the statement does not restore it.  A load must not read a scalar register that a vector instruction wrote
// within the last five wait states, a lane read that brings back a spilled `from` among them, and the compiler does not look into
// the statement: so the load reads a copy that a scalar instruction has made, in the place of the wait state that m0 needs.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int N, int STRIDE>
__device__ __forceinline__ void load_to_lds(const char* from, uint32_t lane_at, uint32_t to) {
  static_assert(N == 1 || N == 2, "one m0 for both");
  uint64_t base;
  if constexpr (N == 1)
    asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
                 : "=&s"(base) : "v"(lane_at), "s"(from), "s"(to) : "m0", "memory");
  else
    asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0\n\tglobal_load_lds_dwordx4 %1, %0 offset:%4"
                 : "=&s"(base) : "v"(lane_at), "s"(from), "s"(to), "n"(STRIDE) : "m0", "memory");
}
#pragma clang diagnostic pop
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// Workgroup barrier that leaves the newest `kInFlight` loads of the wavefront in flight; its LDS
// reads are done, and memory operations stay on their side of it.
template <int kInFlight>
__device__ __forceinline__ void wait_and_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((kInFlight & 15) | ((kInFlight >> 4) << 14) | (7 << 4));   // vmcnt(kInFlight) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The wavefront's LDS reads are done before what follows.
__device__ __forceinline__ void wait_for_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));           // lgkmcnt(0)
  asm volatile("" ::: "memory");
}

// f(0), f(1), ... f(N - 1), each with its argument as a constant
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (N > 0) {
    unrolled<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// SPLIT: a persistent launch over one sequence of tile steps (see the head of the file) instead of
// one workgroup per (user, head, query block).
template <int D, int NST, int NQ, bool PW, bool SPLIT>
__global__ __launch_bounds__(256, 2) void attn_prefill_kernel(PoolGeom g, BatchDev b,
                                                                const uint16_t* __restrict__ q,
                                                                uint16_t* __restrict__ out, float c, float inv_norm,
                                                                int q_blocks_max, int n_pairs, int pair_group, int id_cap,
                                                                int block_cost, int min_steps,
                                                                MergeDesc* __restrict__ ws_desc,
                                                                float* __restrict__ ws_o, float* __restrict__ ws_ml) {
  constexpr int kWaveQ = 32 * NQ;      // queries per wavefront
  constexpr int kBlockQ = 4 * kWaveQ;  // new tokens per workgroup
  constexpr int kBlockTiles = kBlockQ / kTile;
  constexpr int KS = D / 16;           // k-steps of Q.K
  constexpr int DB = D / 32;           // 32-dim blocks of the output
  constexpr int FR = KS + 2 * DB;      // 1 KiB fragments of a tile: K (step), then V (dim block, sub-block)
  constexpr int FQ = FR / 4;           // fragments each wavefront fetches: FQ/2 of K, FQ/2 of V
  static_assert(FQ % 2 == 0 && FQ >= 2 && NST == 3, "fragment split");

  extern __shared__ int s_ids[];       // physical page of every logical page the block reads
  __shared__ u32x4 stage[NST][FR * 64];  // K in KS KiB, then V (k_lane, v_lane and the reads below have the order)
  // A wavefront's queries come by way of LDS, 1 KiB of rows a load: into the wavefront's own room of the stages that are not
  // filled yet, and what does not fit there into rooms beside the page table (QueryRooms).
  constexpr bool kBlockReference = SPLIT && !PW;
  using Rooms = QueryRooms<D, kBlockReference>;
  constexpr int kRooms = Rooms::kFree, kOwnRooms = Rooms::kOwn, kOwnWords = kOwnRooms * 256;
  static_assert(kRooms == (kBlockReference ? 3 : 4) * (FQ / 2) && sizeof(stage) == 3 * 32 * D * 4, "as the launch allows for");
  __shared__ int redo_flag[4];         // of every wavefront

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int r = lane & 31, hf = lane >> 5;
  const int H = g.H, S = g.S;

  // The block (or, SPLIT, the segment of a block) being worked on.
  int u, h, qblk, tok0, n_u, P, pbeg, npg, t_beg = 0, t_end;
  // SPLIT: this workgroup's share [pos, hi) of the call's tile steps
  int wid = 0, pos = 0, lo = 0, hi = 1, pair_end = 0, seg_end = 0;
  PrefillShares shares{2, 1, false};
  // steps of one (user, head): every block counts its tiles and an allowance for its start and end
  auto last_tiles = [&](int prefix, int n) { return (prefix + n + kTile - 1) / kTile; };
  auto steps_before = [&](int prefix, int blk) {                // of blocks [0, blk), all of them full
    return blk * ((prefix + kTile - 1) / kTile + block_cost) + kBlockTiles * (blk * (blk + 1) / 2);
  };
  auto user_steps = [&](int prefix, int n) {
    const int blocks = (n + kBlockQ - 1) / kBlockQ;
    return blocks > 0 ? steps_before(prefix, blocks - 1) + last_tiles(prefix, n) + block_cost : 0;
  };
  // Position of user k's steps in the sequence, from the lanes of a wavefront: inclusive sums over the lanes (scan_lanes).
  // how many of the items 0, 1, ... `count` - 1 start at or before x, less one; `start` rises
  auto last_at_or_before = [&](int count, int x, auto start) __attribute__((always_inline)) {
    int found = 0;
    for (int k = 0; k < count; k += 64) {
      const int here = __builtin_popcountll(__builtin_amdgcn_ballot_w64(k + lane < count && start(k + lane) <= x));
      found += here;
      if (here < 64) break;
    }
    return found - 1;
  };
  int l_tok = 0, l_n = 0, l_P = 0, l_pg = 0, l_npg = 0;         // SPLIT: of this lane's user in the group below
  int l_first = 0;                                              // ... the group's first position
  int l_incl = 0, group_of = -1;                                // ... inclusive sums inside the group; which group
  int g_incl = 0;                                               // inclusive sums over groups: a lane holds one
  // Descriptors per block (n_pairs > 0 of them, as many as the call's bounds allow): sums of the users' blocks as above, and
  // the number of the user's first one
  const bool per_block = SPLIT && n_pairs > 0;
  int gb_incl = 0, lb_incl = 0, first_block = 0;
  auto user_blocks = [&](int n) { return n > 0 ? (n + kBlockQ - 1) / kBlockQ * H : 0; };
  const int users_per_lane = SPLIT ? (b.batch + 63) / 64 : 1;   // of a group
  auto load_user = [&](int k) __attribute__((always_inline)) {
    l_n = 0;
    if (k < b.batch) {
      l_tok = b.new_indptr[k];
      l_n = b.new_indptr[k + 1] - l_tok;
      l_P = b.prefix_lens[k];
      l_pg = b.page_indptr[k];
      l_npg = b.page_indptr[k + 1] - l_pg;
    }
  };
  // the block that holds position x
  int blk_pos = 0;
  auto locate = [&](int x) __attribute__((always_inline)) {
    const int grp = __builtin_popcountll(__builtin_amdgcn_ballot_w64(g_incl <= x));   // the lane whose users hold `pos`
    int user_pos;
    if (users_per_lane == 1) {
      u = grp;
      user_pos = u > 0 ? __builtin_amdgcn_readlane(g_incl, u - 1) : 0;
      if (per_block) first_block = u > 0 ? __builtin_amdgcn_readlane(gb_incl, u - 1) : 0;
    } else {
      // the users of that lane, one a lane
      if (grp != group_of) {
        group_of = grp;
        l_n = 0;
        if (lane < users_per_lane) load_user(grp * users_per_lane + lane);
        l_incl = scan_lanes(user_steps(l_P, l_n) * H);
        if (per_block) lb_incl = scan_lanes(user_blocks(l_n));
        l_first = grp > 0 ? __builtin_amdgcn_readlane(g_incl, grp - 1) : 0;
      }
      u = __builtin_popcountll(__builtin_amdgcn_ballot_w64(l_incl <= x - l_first));
      user_pos = l_first + (u > 0 ? __builtin_amdgcn_readlane(l_incl, u - 1) : 0);
      if (per_block)
        first_block = (grp > 0 ? __builtin_amdgcn_readlane(gb_incl, grp - 1) : 0) +
                      (u > 0 ? __builtin_amdgcn_readlane(lb_incl, u - 1) : 0);
    }
    tok0 = __builtin_amdgcn_readlane(l_tok, u);
    n_u = __builtin_amdgcn_readlane(l_n, u);
    P = __builtin_amdgcn_readlane(l_P, u);
    pbeg = __builtin_amdgcn_readlane(l_pg, u);
    npg = __builtin_amdgcn_readlane(l_npg, u);
    const int head_steps = user_steps(P, n_u);
    h = last_at_or_before(H, x - user_pos, [&](int k) { return k * head_steps; });
    const int head_pos = user_pos + h * head_steps;
    qblk = last_at_or_before((n_u + kBlockQ - 1) / kBlockQ, x - head_pos, [&](int k) { return steps_before(P, k); });
    blk_pos = head_pos + steps_before(P, qblk);
  };
  if constexpr (SPLIT) {
    // Every wavefront works the schedule out by itself, without LDS or barriers: lane i sums the steps of
    // users [i, i + 1) * users_per_lane; up to 64 users that is one each, and nothing is read again.
    int steps = 0, blocks = 0;
    if (users_per_lane == 1) {
      load_user(lane);
      steps = user_steps(l_P, l_n) * H;
      blocks = user_blocks(l_n);
    } else {
      for (int j = 0; j < users_per_lane; ++j) {
        load_user(lane * users_per_lane + j);
        steps += user_steps(l_P, l_n) * H;
        blocks += user_blocks(l_n);
      }
    }
    g_incl = scan_lanes(steps);
    if (per_block) gb_incl = scan_lanes(blocks);
    const int total = __builtin_amdgcn_readlane(g_incl, 63);
    // blockIdx -> XCD is round-robin, and inside an XCD the first half of a full launch's workgroups come first to
    // their CUs, the second half to the same ones.  Every XCD gets one contiguous stretch of the sequence, so
    // that the shares of one (user, head) meet in one L2, and a CU two neighbouring shares.
    const int slots = (int)gridDim.x / kXcds, xcd = (int)blockIdx.x % kXcds, slot = (int)blockIdx.x / kXcds;
    shares = prefill_shares(total, (int)gridDim.x, min_steps, (int)gridDim.x == kPrefillMaxWgs);
    if (shares.paired) {
      wid = 2 * (xcd * (slots / 2) + slot % (slots / 2)) + slot / (slots / 2);
    } else {
      wid = gridDim.x % kXcds == 0 ? xcd * slots + slot : (int)blockIdx.x;
    }
    const int64_t first_step = shares.begin(wid), last_step = shares.end(wid);
    lo = first_step < total ? (int)first_step : total;
    hi = last_step < total ? (int)last_step : total;
    pos = lo;
    if (!per_block) {
      if (tid == 0) ws_desc[wid].valid = 0;
    } else {
      const int k = __builtin_amdgcn_readlane(gb_incl, 63) + (int)blockIdx.x;     // numbers that no block has
      if ((unsigned)k < (unsigned)n_pairs && tid == 0) ws_desc[k].valid = 0;
    }
  } else {
    // blockIdx -> XCD is round-robin: all blocks of one (user, head) share blockIdx % 8.  An XCD
    // takes `pair_group` pairs at a time, the longest causal rows of all of them first.
    const int slot = blockIdx.x / kXcds, per_group = pair_group * q_blocks_max;
    const int in_group = slot % per_group;
    const int pair = (slot / per_group * pair_group + in_group % pair_group) * kXcds + (blockIdx.x % kXcds);
    if (pair >= n_pairs) return;
    qblk = q_blocks_max - 1 - in_group / pair_group;
    u = pair / H;
    h = pair % H;
    tok0 = b.new_indptr[u];
    n_u = b.new_indptr[u + 1] - tok0;
    if (qblk * kBlockQ >= n_u) return;                            // workgroup-uniform
    P = b.prefix_lens[u];
    pbeg = b.page_indptr[u];
    npg = b.page_indptr[u + 1] - pbeg;
  }

  while (pos < hi) {                                              // workgroup-uniform; once without SPLIT
  if constexpr (SPLIT) {
    locate(pos);
  }
  const int Q0 = qblk * kBlockQ;
  const int T_u = P + n_u;                                      // tokens that hold data
  const int blk_end = (n_u < Q0 + kBlockQ) ? n_u : (Q0 + kBlockQ);
  const int tiles_blk = (P + blk_end + kTile - 1) / kTile;      // kv tiles the block's last query sees
  t_end = tiles_blk;
  if constexpr (SPLIT) {
    pair_end = blk_pos + tiles_blk + block_cost;
    seg_end = pair_end < hi ? pair_end : hi;
    // positions count cost units: a block's allowance comes first, then its tiles
    const int c_beg = pos - blk_pos - block_cost, c_end = seg_end - blk_pos - block_cost;
    t_beg = c_beg > 0 ? c_beg : 0;
    t_end = c_end > 0 ? c_end : 0;
    if (t_end <= t_beg) {                                       // only the allowance lies in this share
      pos = seg_end;
      continue;
    }
  }
  const int q0 = Q0 + kWaveQ * wave;                                // this wavefront's queries
  int nq = n_u - q0;
  nq = nq < 0 ? 0 : (nq > kWaveQ ? kWaveQ : nq);
  int tiles_w = nq > 0 ? (P + q0 + nq + kTile - 1) / kTile : 0;
  if (SPLIT && tiles_w > t_end) tiles_w = t_end;
  const int first_query_pos = P + q0;

  // page table of the segment, copied to LDS in the prologue
  const int lp_beg = SPLIT ? (t_beg * 2) >> g.sub_shift : 0;
  const int n_ids = ((t_end * 2 - 1) >> g.sub_shift) + 1 - lp_beg;
  const int block = SPLIT ? first_block + h * ((n_u + kBlockQ - 1) / kBlockQ) + qblk : 0;
  if (n_ids > id_cap) {                // lengths beyond the bound the call stated: no output, no overrun
    if (!SPLIT) return;
    if (per_block && t_beg == 0 && (unsigned)block < (unsigned)n_pairs && tid == 0) ws_desc[block].valid = 0;
    pos = seg_end;
    continue;
  }
  const int sub_mask = (1 << g.sub_shift) - 1;
  const int64_t v_off = (int64_t)S * D * 2;
  const char* head_base = g.layer_base + (int64_t)h * 2 * S * D * 2;

  const int last_tile = t_end - 1;
  // A wavefront moves what comes from one of a tile's two sub-blocks, number wave & 1: one page id a tile, one address
  // that is the same for all lanes.
  // K fragment s: lane (r, hf) holds dims 16 s + 8 hf .. + 7 of tile row r.  The row order makes the 16
  // accumulator values of a lane its tokens 8 hf .. + 7 of sub-block 0, then of sub-block 1.  In LDS, 1 KiB holds the rows
  // of one sub-block of fragments 2 x and 2 x + 1; x = wave / 2 and wave / 2 + 2 are the wavefront's, as far apart there as
  // in the page.
  const uint32_t k_lane = ((((lane >> 3) & 1) * (D / 8) + 4 * (wave >> 1) + (lane >> 4)) * 8 + (lane & 7)) * 16;
  const int k_read = (r >> 4) * (KS / 2 * 64) + hf * 16 + (r & 15);
  // V^T fragment (db, sb): dim 32 db + r, tokens 8 hf .. + 7 of sub-block sb; db = wave / 2 and wave / 2 + 2 are the wavefront's
  const uint32_t v_lane = (uint32_t)v_off + (r * 2 + hf) * 16 + (wave >> 1) * 1024;
  const uint32_t k_lds = lds_address(&stage[0][0]) + ((wave & 1) * (KS / 2) + (wave >> 1) * (KS / 4)) * 1024;
  const uint32_t v_lds = lds_address(&stage[0][0]) + (KS + (wave & 1) + (wave >> 1) * DB) * 1024;
  // a tile's sub-block (past the end: of the last one, whose data is then fetched again, never used), its page
  auto sub_block = [&](int tile) __attribute__((always_inline)) { return (tile < last_tile ? tile : last_tile) * 2 + (wave & 1); };
  auto page_id = [&](int tile) __attribute__((always_inline)) { return s_ids[(sub_block(tile) >> g.sub_shift) - lp_beg]; };
  auto put_id = [&](int i) __attribute__((always_inline)) {
    int id = lp_beg + i < npg ? b.page_indices[pbeg + lp_beg + i] : 0;
    if ((unsigned)id >= (unsigned)g.num_pages) id = 0;
    s_ids[i] = id;
  };
  // A stage holds the keys of tile `tile` and the values of the tile two before it.  Fetches this
  // wavefront's quarter of it straight into LDS; the first two stages of a segment are keys only.
  const char *v_1 = head_base, *v_2 = head_base;                 // of tiles tile - 1 and tile - 2
  auto sub_block_at = [&](int tile, int id) __attribute__((always_inline)) {
    const uint32_t page = (uint32_t)g.page_bytes;                // at most 2 GiB: 65535 heads of 64 x 128 bf16
    return head_base + (uint64_t)(uint32_t)uniform(id) * page + (uint32_t)((sub_block(tile) & sub_mask) * 16 * D * 2);
  };
  auto load = [&](int st, int tile, int id, auto with_v) __attribute__((always_inline)) {
    const char* at = sub_block_at(tile, id);
    load_to_lds<FQ / 2, 1024>(at, k_lane, k_lds + st * (FR * 1024));
    if constexpr (decltype(with_v)::value) load_to_lds<FQ / 2, 2048>(v_2, v_lane, v_lds + st * (FR * 1024));
    v_2 = v_1;
    v_1 = at;
  };

  // Row `row` of the wavefront's 32 NQ queries lies in room row / kRoomRows, its 16-byte pieces turned by the row, so that the
  // 32 rows of a fragment are read without conflicts.
  constexpr int kPieces = D / 8, kRoomRows = 64 / kPieces;
  auto turn = [](int row) __attribute__((always_inline)) { return D == 128 ? row & 15 : (row >> 1) & 7; };
  auto room = [&](int j) __attribute__((always_inline)) -> uint32_t {
    constexpr int N = FQ / 2;
    const int own = (int)lds_address(s_ids + Rooms::at(id_cap)) + (wave * kOwnRooms - kRooms) * 1024;
    return j < N       ? k_lds + 2 * FR * 1024 + j * 1024
           : j < 2 * N ? v_lds + 2 * FR * 1024 + (j - N) * 2048
           : j < 3 * N ? v_lds + FR * 1024 + (j - 2 * N) * 2048
           : j < kRooms ? v_lds + (j - 3 * N) * 2048
                        : (uint32_t)(own + j * 1024);
  };
  {
    // The queries, whose addresses need no page id, in whole rows; those past the user's last repeat it and go nowhere.
    // Loaded as fragments, 32 bytes of 32 rows an instruction, they held up the tiles they came behind: the first block's
    // scores began 5.3 us after the schedule, now 4.0 (6.8 and 5.0 with eight users), later blocks' after 3.4 instead of 4.4.
    // And only what the first scores need is asked for before them: the third stage waits in the queries' room.
    const char* from = reinterpret_cast<const char*>(q + ((int64_t)(tok0 + Q0) * H + h) * D);
    int ln = lane;                                                 // hidden, or eight offsets a lane are kept, spilled, for the next segment
    asm volatile("" : "+v"(ln));
    unrolled<8>([&](auto j_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value;
      const int row = j * kRoomRows + ln / kPieces, at = kWaveQ * wave + row;
      const int there = at < n_u - Q0 ? at : n_u - Q0 - 1;
      load_to_lds<1, 0>(from, (uint32_t)there * (uint32_t)(H * D * 2) + (uint32_t)((ln % kPieces) ^ turn(row)) * 16, room(j));
    });
  }

  bf16x8 qf[NQ][KS];
  f32x16 o[NQ][DB];
  float l[NQ];                     // softmax denominators: this lane's tokens only
  float m[NQ], mcq[NQ];            // reference max: raw logit units / scaled for the base-2 exponent
  float cq[NQ];                    // what scales the logits: c, but for huge ones (row_scale)
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) { m[qb] = -INFINITY; mcq[qb] = 0.f; cq[qb] = c; }

  auto key_fragment = [&](int st, int s, int room = 0) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8, stage[st][(room + (s >> 2) + KS / 4 * (s >> 1 & 1)) * 64 + (s & 1) * 32 + k_read]);
  };
  auto value_fragment = [&](int st, int f) __attribute__((always_inline)) {        // f = 2 db + sb
    return __builtin_bit_cast(bf16x8, stage[st][(KS + (f >> 2) * 2 + (f & 1) + DB * (f >> 1 & 1)) * 64 + lane]);
  };
  // S^T of query block qb; with `masked`, keys the query must not see (causal order among the new
  // tokens) are set to -inf.
  auto scores = [&](const bf16x8 (&kf)[KS], int qb, int tb, bool masked) __attribute__((always_inline)) {
    f32x16 z;
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[qb][s], z, 0, 0, 0);
    if (masked) {
      const int qpos = first_query_pos + 32 * qb + r;
      const int kbase = tb + 8 * hf;
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (kbase + 16 * (e >> 3) + (e & 7) > qpos) z[e] = PW ? 0.f : -INFINITY;
    }
    return z;
  };
  auto max16 = [](const f32x16& z) __attribute__((always_inline)) {
    float v = z[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) v = fmaxf(v, z[e]);
    return v;
  };
  // reference max from the scores of a tile; with nothing visible or all of them -inf, any will do
  auto set_reference = [&](const f32x16& z, int qb) __attribute__((always_inline)) {
    m[qb] = pair_max(max16(z));
    const float ref = m[qb] == -INFINITY ? 0.f : m[qb];
    cq[qb] = merge_detail::row_scale(ref, c);
    mcq[qb] = ref * cq[qb];
  };
  // Weights of a tile from its scores, and their sum.
  auto weights = [&](const f32x16& z, int qb, bf16x8 (&pf)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = z[8 * sb + e];
        if constexpr (PW) pf[sb][e] = (__bf16)fast_silu(x * c);
        else pf[sb][e] = (__bf16)fast_exp2(fmaf(x, cq[qb], -mcq[qb]));
      }
      if constexpr (!PW) {
        // the rounded weights are summed, as P.V does
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const bf16x2 w = {pf[sb][e], pf[sb][e + 1]}, one = {(__bf16)1.0f, (__bf16)1.0f};
          l[qb] = __builtin_amdgcn_fdot2_f32_bf16(w, one, l[qb], false);
        }
      }
    }
  };
  // Step `t`: the scores of tile t+1, whose keys are in registers, go into z_next while the weights
  // of tile t are taken from z; its values come from stage `st`, and so do the keys of tile t+2,
  // which travel to registers while the matrix cores work on P.V.
  // The barrier publishes the stage and retires every read of the one before it, which the fetch
  // for step t+2 overwrites; the fetch for step t+1 stays in flight across it.
  int next_id = 0;                     // page of the tile that the next step fetches
  bf16x8 kf[KS];
  auto move = [&](int t, int st) __attribute__((always_inline)) {
    wait_and_barrier<FQ>();
    load(st == 0 ? NST - 1 : st - 1, t + 4, next_id, std::true_type{});
    next_id = page_id(t + 5);
  };
  auto read_values = [&](int st, bf16x8 (&vf)[2 * DB]) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < 2 * DB; ++f) vf[f] = value_fragment(st, f);
  };
  auto read_keys = [&](int st) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = key_fragment(st, s);
  };
  auto add_values = [&](int qb, const bf16x8 (&vf)[2 * DB], const bf16x8 (&pf)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int sb = 0; sb < 2; ++sb)
#pragma unroll
      for (int db = 0; db < DB; ++db)
        o[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[2 * db + sb], pf[sb], o[qb][db], 0, 0, 0);
  };
  // Tiles past the wavefront's own last query hold no key it may see (the later wavefronts of the block still need
  // them): it only helps to move them.
  // NQ = 1
  auto step = [&](auto masked_c, int t, int st, f32x16& z, f32x16& z_next) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    move(t, st);
    const bool here = !MASKED || t < tiles_w, next = !MASKED || t + 1 < tiles_w;
    bf16x8 vf[2 * DB];
    if (here) read_values(st, vf);
    if (next) z_next = scores(kf, 0, (t + 1) * kTile, MASKED);
    if (here) {
      bf16x8 pf[2];
      weights(z, 0, pf);
      __builtin_amdgcn_sched_barrier(0);
      read_keys(st);
      const int tb = t * kTile;
      if constexpr (MASKED) {                                      // slots past the user's last token may hold anything
        if (tb + kTile > T_u) {
#pragma unroll
          for (int f = 0; f < 2 * DB; ++f)
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (tb + 16 * (f & 1) + 8 * hf + e >= T_u) vf[f][e] = (__bf16)0.0f;
        }
      }
      add_values(0, vf, pf);
    }
  };
  // NQ = 2: the query blocks are half a step apart, so that all of the matrix work has weights to be taken beside it.  On
  // entry p0 are the weights of block 0 and z1 the scores of block 1; z0 holds nothing between steps (both blocks in step keep two
  // sets of scores each, spilled 22 registers in the split form, and took 1-2 % longer: heads of 64, one user's 6000 tokens x 8
  // 62.6 -> 61.5 us a layer, 8 users x 1150 x 8 37.2 -> 36.4).
  auto step_apart = [&](auto masked_c, int t, int st, f32x16& z0, f32x16& z1, bf16x8 (&p0)[2]) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    move(t, st);
    const bool here = !MASKED || t < tiles_w, next = !MASKED || t + 1 < tiles_w;
    bf16x8 vf[2 * DB], p1[2];
    if (here) read_values(st, vf);
    if (next) z0 = scores(kf, 0, (t + 1) * kTile, MASKED);
    if (here) {
      weights(z1, NQ - 1, p1);
      const int tb = t * kTile;
      if constexpr (MASKED) {                                      // slots past the user's last token may hold anything
        if (tb + kTile > T_u) {
#pragma unroll
          for (int f = 0; f < 2 * DB; ++f)
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (tb + 16 * (f & 1) + 8 * hf + e >= T_u) vf[f][e] = (__bf16)0.0f;
        }
      }
      add_values(0, vf, p0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (next) z1 = scores(kf, NQ - 1, (t + 1) * kTile, MASKED);
    if (here) read_keys(st);
    if (next) weights(z0, 0, p0);
    if (here) add_values(NQ - 1, vf, p1);
    __builtin_amdgcn_sched_barrier(0);
  };
  // tiles below hide no key from any query of the block (its first wavefront sees the least)
  int fast_all = (P + Q0 + 1) / kTile;
  if (fast_all > t_end) fast_all = t_end;
  constexpr std::false_type body{};
  constexpr std::true_type tail{};

  for (int attempt = 0; attempt < 2; ++attempt) {                // workgroup-uniform
    // The first tile by a value that the compiler cannot see through: else it computes the masks and addresses of
    // the prologue ahead of this loop, into 200 spilled scalar registers, 1.5 us at each start of a block.
    int zero = 0;
    asm volatile("" : "+s"(zero));
    const int tile0 = t_beg + zero;
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      l[qb] = 0.f;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[qb][db][e] = 0.f;
    }
    if (!PW && attempt == 1) {
      // exact max of every query over its whole visible range: K only, straight from global
      float mx[NQ];
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb) mx[qb] = -INFINITY;
      for (int tile = tile0; tile < tiles_w; ++tile) {         // tiles past tiles_w hold no visible key
        const int sb = tile * 2 + (r >> 4);
        const char* ka = head_base + (int64_t)s_ids[(sb >> g.sub_shift) - lp_beg] * g.page_bytes +
                         (int64_t)(sb & sub_mask) * 16 * D * 2 + (((r >> 3 & 1) * (D / 8) + hf) * 8 + (r & 7)) * 16;
        bf16x8 kf[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) kf[s] = *reinterpret_cast<const bf16x8*>(ka + s * 256);
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) mx[qb] = fmaxf(mx[qb], max16(scores(kf, qb, tile * kTile, true)));
      }
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb) {
        m[qb] = pair_max(mx[qb]);
        const float ref = m[qb] == -INFINITY ? 0.f : m[qb];
        cq[qb] = merge_detail::row_scale(ref, c);
        mcq[qb] = ref * cq[qb];
      }
    }

    // prologue: the keys of the first two tiles, the stage of the first step, the first tile's scores
    // Their pages, and those of the user's first tile, by scalar loads that travel together.
    int id[NST + 1] = {};
    auto tile_at = [&](int k) __attribute__((always_inline)) { return k == NST ? zero : tile0 + k; };
    if (npg > 0) {
#pragma unroll
      for (int k = 0; k <= NST; ++k) {
        const int lp = sub_block(tile_at(k)) >> g.sub_shift;
        id[k] = scalar_load(b.page_indices, pbeg + (lp < npg ? lp : npg - 1));
      }
#pragma unroll
      for (int k = 0; k <= NST; ++k)
        if ((unsigned)id[k] >= (unsigned)g.num_pages || sub_block(tile_at(k)) >> g.sub_shift >= npg) id[k] = 0;
    }
    // SPLIT: the reference of a piece is that of its whole block, the max of the user's first tile.  So its
    // weights are rounded as those of an uncut block, and how a call is cut changes its result by the
    // order of fp32 sums alone.  The tile's keys travel beside the piece's own, into the room of the
    // values that stage 0 does not hold yet; 8 layers of one user's 5189 tokens x 4 heads take 446 us with
    // it and 441 with a reference of each piece's own, six returning users beside two first-time ones 750 and 741.
    if (kBlockReference && attempt == 0) {
      load_to_lds<FQ / 2, 1024>(sub_block_at(zero, id[NST]), k_lane, k_lds + KS * 1024);
    }
    load(0, tile0, id[0], std::false_type{});
    load(1, tile0 + 1, id[1], std::false_type{});
    if (attempt == 0) {
      // behind the first tiles' loads, so that their round trip is shared: the block's page table -> LDS.  Ids the metadata does not back become page 0 (in bounds; such slots lie past the user's last
      // token and are masked).
      const int n_first = kOwnRooms > 0 && n_ids > Rooms::at(id_cap) ? Rooms::at(id_cap) : n_ids;
      for (int i = tid; i < n_first; i += 256) put_id(i);
    }
    wait_and_barrier<0>();
    if (attempt == 0) {
      // Q^T fragments: lane (r, hf) holds query q0 + 32 qb + r, dims 16 s + 8 hf .. + 7.
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb) {
        int row = 32 * qb + r;
        asm volatile("" : "+v"(row));
        const uint32_t at = room(row / kRoomRows) + (row % kRoomRows) * (D * 2);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          typedef const __attribute__((address_space(3))) bf16x8* lds_fragment;
          qf[qb][s] = *(lds_fragment)(uintptr_t)(at + (uint32_t)(((2 * s + hf) ^ turn(row)) * 16));
        }
      }
      wait_for_lds();
      if constexpr (kOwnRooms > 0) {                               // ids of the wavefront's own room, free now; the next barrier shows them
        const int mine = Rooms::at(id_cap) + wave * kOwnWords, end = n_ids < mine + kOwnWords ? n_ids : mine + kOwnWords;
        for (int i = mine + lane; i < end; i += 64) put_id(i);
      }
    }
    load(2, tile0 + 2, id[2], std::true_type{});                   // into the room that the queries have left
    f32x16 za[NQ], zb;
    if (kBlockReference && attempt == 0) {
#pragma unroll
      for (int s = 0; s < KS; ++s) kf[s] = key_fragment(0, s, KS);
#pragma unroll
      for (int qb = 0; qb < NQ; ++qb) set_reference(scores(kf, qb, zero, true), qb);
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = key_fragment(0, s);
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      za[qb] = scores(kf, qb, tile0 * kTile, true);
      if (!PW && !kBlockReference && attempt == 0) set_reference(za[qb], qb);
    }
    wait_and_barrier<FQ>();                                        // stage 0 is read
    next_id = page_id(tile0 + 3);
    load(0, tile0 + 3, next_id, std::true_type{});
    next_id = page_id(tile0 + 4);
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = key_fragment(1, s);

    int tile = tile0, st = 2;
    auto after = [](int st) __attribute__((always_inline)) { return st == NST - 1 ? 0 : st + 1; };
    if (nq == 0) {                                                 // no query of this wavefront's: it only moves tiles
      for (; tile < t_end; ++tile) {
        move(tile, st);
        st = after(st);
      }
    }
    // steady state: fully visible tiles; then the causal tail, and what is left over
    if constexpr (NQ == 1) {
      for (; tile + 2 < fast_all; tile += 2) {
        step(body, tile, st, za[0], zb);
        st = after(st);
        step(body, tile + 1, st, zb, za[0]);
        st = after(st);
      }
      for (; tile < t_end; tile += 2) {
        step(tail, tile, st, za[0], zb);
        st = after(st);
        if (tile + 1 < t_end) step(tail, tile + 1, st, zb, za[0]);
        st = after(st);
      }
    } else {
      bf16x8 p0[2];
      weights(za[0], 0, p0);
      for (; tile + 1 < fast_all; ++tile) {
        step_apart(body, tile, st, za[0], za[NQ - 1], p0);
        st = after(st);
      }
      for (; tile < t_end; ++tile) {
        step_apart(tail, tile, st, za[0], za[NQ - 1], p0);
        st = after(st);
      }
    }
    wait_and_barrier<0>();                                         // no load is in flight, no stage is read

    if constexpr (PW) break;                                     // no statistics, nothing to redo
    // A reference far below the true max shows up as an overflowed (or NaN) denominator of a
    // real query; then every wavefront of the block goes round again.
    // (the numerator overflows first when the values are large: the sum of a query's absolute
    // accumulator values is infinite or NaN as soon as one of them is)
    const merge_detail::RedoLimits limit = merge_detail::redo_limits(SPLIT && (t_beg > 0 || t_end < tiles_blk));
    bool bad = false;
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      l[qb] = pair_sum(l[qb]);
      float mag = 0.f;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) mag += fabsf(o[qb][db][e]);
      bad |= (32 * qb + r < nq) && (!(l[qb] < limit.den) || !(mag < limit.mag));
    }
    // read by everyone before the barriers of the next prologue, written behind them
    const int wave_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
    if (lane == 0) redo_flag[wave] = wave_bad;
    __syncthreads();
    if (!(redo_flag[0] | redo_flag[1] | redo_flag[2] | redo_flag[3])) break;
  }

  auto out4 = [](const f32x16& acc, int g8, float inv) __attribute__((always_inline)) {
    bf16x4 ob;
#pragma unroll
    for (int k = 0; k < 4; ++k) ob[k] = (__bf16)(acc[4 * g8 + k] * inv);
    return ob;
  };
  if (!SPLIT || (t_beg == 0 && t_end == tiles_blk)) {
    if (per_block && (unsigned)block < (unsigned)n_pairs && tid == 0) ws_desc[block].valid = 0;
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      const int qi = 32 * qb + r;
      if (qi < nq) {
        const float inv = PW ? inv_norm : 1.0f / l[qb];
        uint16_t* orow = out + ((int64_t)(tok0 + q0 + qi) * H + h) * D + 8 * hf;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int g8 = 0; g8 < 4; g8 += 2) {
            // accumulator rows 8 g8 + 4 hf .. + 3 of two g8: the query's other lane trades one for one, 16 bytes each
            u32x2 a = __builtin_bit_cast(u32x2, out4(o[qb][db], g8, inv)), b = __builtin_bit_cast(u32x2, out4(o[qb][db], g8 + 1, inv));
            const auto x = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
            const auto y = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
            *reinterpret_cast<u32x4*>(orow + 32 * db + 8 * g8) = u32x4{x[0], y[0], x[1], y[1]};
          }
      }
    }
  } else {
    const int slot = (pos == lo) ? 0 : 1;              // leading or trailing piece of this share
    const int64_t prow = ((int64_t)wid * 2 + slot) * kBlockQ + kWaveQ * wave;
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
      const int qi = 32 * qb + r;
      if (qi < nq) {
        // in fragment order: a store of a wavefront is one run of 1 KB (row by row, 32 of 32 bytes)
        f32x4* po = reinterpret_cast<f32x4*>(ws_o + ((int64_t)wid * 2 + slot) * kBlockQ * D) + (NQ * wave + qb) * DB * 4 * 64 + lane;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int g8 = 0; g8 < 4; ++g8) {
            f32x4 piece;
#pragma unroll
            for (int k = 0; k < 4; ++k) piece[k] = o[qb][db][4 * g8 + k];
            po[(db * 4 + g8) * 64] = piece;
          }
        if (!PW && hf == 0) {
          // a first tile of infinite logits names no reference: what was weighed has been weighed against 0
          ws_ml[(prow + qi) * 2] = m[qb] == -INFINITY && l[qb] != 0.f ? 0.f : m[qb];
          ws_ml[(prow + qi) * 2 + 1] = l[qb];
        }
      }
    }
    if (t_beg == 0 && tid == 0) {
      // this share holds the block's first tile: it owns the merge of all the pieces
      MergeDesc d;
      d.valid = 1;
      d.w_first = wid;
      d.w_last = shares.of(pair_end - 1);
      d.out_row = (tok0 + Q0) * H + h;
      d.nq = blk_end - Q0;
      d.first_slot = slot;
      d.pad[0] = d.pad[1] = 0;
      if (!per_block) ws_desc[wid] = d;
      else if ((unsigned)block < (unsigned)n_pairs) ws_desc[block] = d;
    }
  }
  if constexpr (!SPLIT) break;
  pos = seg_end;
  __syncthreads();                                     // the segment's page table and stages are done with
  }
}

template <int D, int NST, int NQ, bool PW, bool SPLIT>
hipError_t allow_lds() {
  static std::once_flag attr_once;                               // static + dynamic LDS may pass 64 KiB
  static hipError_t attr_status = hipSuccess;
  std::call_once(attr_once, [] {
    attr_status = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_prefill_kernel<D, NST, NQ, PW, SPLIT>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize,
                                      kMaxIdBytes + 16 + QueryRooms<D, SPLIT && !PW>::kWords * 4);
  });
  return attr_status;
}

// Pairs (user, head) that an XCD takes at a time.  One after the other, the last pair's longest block
// starts last and the launch waits for it; all together, the longest blocks of all start first, but
// where their K/V are several times the XCD's 4 MB L2 the blocks no longer find in it what the others
// read.  In between, four to seven, evenly, if the users are about as long as one another; if not, as many
// as half fill the XCD's 64 workgroup slots: the last group's longest blocks are a tail again.
// A step's time against one pair at a time (head_dim 128 unless stated; users x tokens x heads, MB of K/V
// per XCD; 4-7 / all at a time): 8 x 300 x 16 (1) 1.00 / 0.90, 20 x 100-700 x 4 (2) 1.05 / 0.96, 20 x 300 x 8
// of head_dim 64 (2) 1.00 / 0.92, 32 x 400 x 8 (7) 0.96 / 0.89, 12 x 600-2500 x 8 (10) 1.06 / 0.95,
// 8 x 1500 x 8 (6) 0.86 / 0.91; 24 x 550 x 16 (14) 0.99 / 1.01, 32 x 1500 x 16 (49) 0.96 / 1.27, 64 x 600 x 16
// (39) 1.00 / 1.22; unequal and large, 2 / 4-7 / all: 24 x 1000-4000 x 8 (31) 1.05 / 1.17 / 1.12, 32 x 400-1500
// x 16 (30) 0.96 / 1.01 / 1.00, 64 x 100-400 x 16 (16) 0.88 / 0.83 / 0.82.
int prefill_pair_group(const PoolGeom& g, const BatchDev& b, int xcd_pairs, int q_blocks_max) {
  const int64_t mean_len = ((int64_t)b.total_pages * g.S + b.batch - 1) / b.batch;
  if (xcd_pairs * mean_len * g.D * 4 <= (12ll << 20)) return xcd_pairs;
  if (4ll * b.max_new * b.batch > 5ll * b.total_new)             // the longest new segment above 1.25 times the mean
    return q_blocks_max >= 32 ? 1 : (32 / q_blocks_max < xcd_pairs ? 32 / q_blocks_max : xcd_pairs);
  const int groups = xcd_pairs >= 4 ? xcd_pairs / 4 : 1;
  return (xcd_pairs + groups - 1) / groups;
}

template <int D, int NST, int NQ, bool PW>
hipError_t launch_one(const PoolGeom& g, const BatchDev& b, const AttnPlan& plan, const uint16_t* q, uint16_t* out,
                      float c, float inv_norm, int64_t id_bytes, void* workspace, hipStream_t stream) {
  constexpr int kBlockQ = 128 * NQ;
  if (plan.prefill_wgs > 0) {
    const hipError_t attr = allow_lds<D, NST, NQ, PW, true>();
    if (attr != hipSuccess) return attr;
    char* ws = static_cast<char*>(workspace);
    MergeDesc* ws_desc = reinterpret_cast<MergeDesc*>(ws);
    float* ws_o = reinterpret_cast<float*>(ws + plan.ws_desc_bytes);
    float* ws_ml = ws_o + (int64_t)plan.prefill_wgs * 2 * kBlockQ * D;
    // A descriptor per block where that is not more than one per share: the merge then launches no workgroups that find none.
    const int64_t blocks = (int64_t)g.H * (b.total_new / kBlockQ + b.batch);   // at most
    // (in eights, an XCD's in a row: the merge reads pieces on the XCD that wrote most of them)
    const int descs = blocks <= plan.prefill_wgs / 8 * 8 ? (int)((blocks + 7) / 8 * 8) : 0;
    const int64_t lds_bytes = QueryRooms<D, !PW>::bytes((int)(id_bytes / 4));
    hipLaunchKernelGGL((attn_prefill_kernel<D, NST, NQ, PW, true>), dim3((unsigned)plan.prefill_wgs), dim3(256),
                       (size_t)lds_bytes, stream, g, b, q, out, c, inv_norm, 1, descs, 1,
                       (int)(id_bytes / 4), plan.pair_cost, plan.min_tiles, ws_desc, ws_o, ws_ml);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return merge_detail::launch_merge<D, PW, true>(out, c, inv_norm, kBlockQ, g.H, plan.prefill_wgs,
                                                   descs > 0 ? descs : blocks, ws_desc, ws_o, ws_ml, stream, descs > 0);
  }
  const hipError_t attr = allow_lds<D, NST, NQ, PW, false>();
  if (attr != hipSuccess) return attr;
  int q_blocks_max = (b.max_new + kBlockQ - 1) / kBlockQ;
  if (q_blocks_max < 1) q_blocks_max = 1;
  const int n_pairs = b.batch * g.H;
  const int xcd_pairs = (n_pairs + kXcds - 1) / kXcds;
  const int pair_group = prefill_pair_group(g, b, xcd_pairs, q_blocks_max);
  const int64_t grid = (int64_t)((xcd_pairs + pair_group - 1) / pair_group * pair_group) * kXcds * q_blocks_max;
  if (grid <= 0 || grid > 0x7fffffffll) return hipErrorInvalidValue;
  const int64_t lds_bytes = QueryRooms<D, false>::bytes((int)(id_bytes / 4));
  hipLaunchKernelGGL((attn_prefill_kernel<D, NST, NQ, PW, false>), dim3((unsigned)grid), dim3(256),
                     (size_t)lds_bytes,
                     stream, g, b, q, out, c, inv_norm, q_blocks_max, n_pairs, pair_group, (int)(id_bytes / 4), 0, 0, nullptr, nullptr,
                     nullptr);
  return hipGetLastError();
}

}  // namespace

bool attn_prefill_applicable(const PoolGeom& g, const BatchDev& b) {
  if (g.es != 2 || (g.D != 64 && g.D != 128)) return false;
  const int64_t ids = ((int64_t)b.max_total_len + g.S - 1) / g.S + 4;
  return ids * 4 <= kMaxIdBytes;
}

// New tokens per workgroup block (the template's 128 * NQ below).
int attn_prefill_block(const PoolGeom& g) { return g.D == 64 ? 256 : 128; }

hipError_t launch_attn_prefill(const PoolGeom& g, const AttnPlan& plan, const void* q, void* out, const BatchDev& b,
                               float sm_scale, float inv_norm, void* workspace, hipStream_t stream) {
  if (b.total_new <= 0 || b.batch <= 0) return hipSuccess;
  if (!attn_prefill_applicable(g, b)) return hipErrorInvalidValue;
  const bool pw = inv_norm > 0.f;
  // softmax logits are exponentiated in base 2; the pointwise scale stays in natural units
  const float c = pw ? sm_scale : sm_scale * 1.4426950408889634f;
  // table entries one block may touch: its tiles end at most one tile past max_total_len
  const int64_t id_bytes = (((int64_t)b.max_total_len + g.S - 1) / g.S + 4) * 4;
  const uint16_t* qp = reinterpret_cast<const uint16_t*>(q);
  uint16_t* op = reinterpret_cast<uint16_t*>(out);
  // Two wavefronts per SIMD in both shapes (<= 256 registers each): one wavefront alone issues
  // in order and leaves its LDS operand reads and MFMA -> VALU dependencies exposed.  At
  // D = 128 that means 32 queries per wavefront (64-register accumulator) and 128-query blocks, at
  // D = 64 twice that.
  switch (g.D) {
    case 64:
      return pw ? launch_one<64, 3, 2, true>(g, b, plan, qp, op, c, inv_norm, id_bytes, workspace, stream)
                : launch_one<64, 3, 2, false>(g, b, plan, qp, op, c, 0.f, id_bytes, workspace, stream);
    case 128:
      return pw ? launch_one<128, 3, 1, true>(g, b, plan, qp, op, c, inv_norm, id_bytes, workspace, stream)
                : launch_one<128, 3, 1, false>(g, b, plan, qp, op, c, 0.f, id_bytes, workspace, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mts
