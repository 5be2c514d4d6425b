// Byte-exact KV movement between the contiguous layout and the paged pool:
//   unpack - Cache Scattering (Sec. 3.2 step 3, scatter kernel of Sec. 4.2)
//   append - Cache Update     (Sec. 3.2 step 5, Alg. 1 step 8.2)
//   pack   - gather kernel of the offload path (Sec. 3.2 step 6, Sec. 4.2)
//
// All three are HBM-bound permutations of 16-byte granules (K) and of elements (V, whose pool
// layout is [dim][token]); see kv_move_kernel for how the work is split.
#include <type_traits>

#include "mts_copy_rules.hpp"
#include "mts_internal.hpp"

namespace mts {
namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));          // one granule, opaque
template <typename T> struct ElemVec;                                // one granule, as elements
template <> struct ElemVec<uint16_t> { typedef uint16_t type __attribute__((ext_vector_type(8))); };
template <> struct ElemVec<uint32_t> { typedef uint32_t type __attribute__((ext_vector_type(4))); };

// Element of a table that no kernel of this file writes: a scalar load whatever surrounds it (the
// index is wavefront-uniform).
template <typename I>
__device__ __forceinline__ I scalar_load(const I* p) {
  return *(const __attribute__((address_space(4))) I*)(uintptr_t)p;
}

// One granule past the caches' retention (KEEP = false: nothing reads it again soon) or the ordinary way.
template <bool KEEP>
__device__ __forceinline__ u32x4 load_granule(const void* p) {
  if constexpr (KEEP) return *reinterpret_cast<const u32x4*>(p);
  else return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
template <bool KEEP>
__device__ __forceinline__ void store_granule(void* p, u32x4 v) {
  if constexpr (KEEP) *reinterpret_cast<u32x4*>(p) = v;
  else __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
}

enum { MODE_UNPACK = 0, MODE_APPEND = 1, MODE_PACK = 2 };

// How a launch's units, (sub-block of a run, head) and layer, are numbered.  kRuns: blockIdx.y is the run.  kPlanes: the same,
// K and V of a masked unit by a wavefront of its own (append_by_planes).  kFlat: an append's units follow one another and each
// wavefront finds its user (append_flat).
enum class Units { kRuns, kPlanes, kFlat };

constexpr int kBulkWaves = 4;      // wavefronts (= units) per bulk workgroup

// The two sides of a move, strides from one layer to the next.
template <typename T>
struct MoveSides {
  PoolGeom g;
  const T *src_a, *src_b;
  T* dst_contig;
  int64_t pool_layer_stride, contig_layer_stride;     // bytes, elements
};

// One wavefront moves one (16-token sub-block, head): the contiguous side moves in whole rows
// (D*es bytes per token and head), the pool side in whole 16-byte granules in pool order, so that
// BOTH sides of every copy are 16-byte-per-lane accesses over full cache lines; the reordering
// in between - the K granule permutation and the V transpose - goes through a wavefront-private
// LDS tile of 16 rows (padded by one granule, which keeps the strided accesses off a single
// bank).  Workgroups [0, bulk_blocks) take the sub-blocks that a run covers completely; those
// behind them take partly covered sub-blocks with the same code under a token mask: rows outside
// the run are neither read nor written, K granules of other tokens are skipped and a V granule
// that the run covers only in part is written piece by piece, so no slot outside the run
// is ever written.
// `runs`: seg_user and seg_pos of a segment list (`run_tok`: seg_tok_indptr) or an append's new_indptr and prefix_lens;
// `pages`: page_indptr and page_indices.
// PAST: which rows travel past the caches' retention (mts_copy_rules.hpp; an append's own rule is at KEEP).
template <typename T, int MODE, int DCH, RowsPast PAST, Units UNITS>
__global__ __launch_bounds__(256) void kv_move_kernel(TableWords runs, TableWords pages, CallWords call, const int64_t* run_tok,
                                                      MoveSides<T> sides) {
  const int32_t *run_user = table(runs[0]), *run_pos = table(runs[1]), *page_indptr = table(pages[0]),
                *page_indices = table(pages[1]);
  const int batch = call[0], H = call[1], bulk_blocks = call[2];
  constexpr int G = 16 / sizeof(T);
  constexpr int D = DCH * G;
  constexpr int PITCH = D + G;       // LDS row pitch in elements (one granule of padding)
  constexpr int NIT = 16 * DCH / 64; // 64-granule rounds per 16-token sub-block
  constexpr int dch = DCH;
  constexpr bool PLANES = UNITS == Units::kPlanes, FLAT = UNITS == Units::kFlat;
  const int s = blockIdx.y;
  // several layers in one launch: blockIdx.z picks the layer on both sides
  PoolGeom& g = sides.g;
  const int S = g.S;
  g.layer_base += (int64_t)blockIdx.z * sides.pool_layer_stride;
  const T* src_a = sides.src_a + (int64_t)blockIdx.z * sides.contig_layer_stride;
  const T* src_b = MODE == MODE_APPEND ? sides.src_b + (int64_t)blockIdx.z * sides.contig_layer_stride : nullptr;
  T* dst_contig = MODE == MODE_PACK ? sides.dst_contig + (int64_t)blockIdx.z * sides.contig_layer_stride : nullptr;

  // Which sub-block this wavefront moves
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  // unit = 4 * block + wave of a part, as (sub-block, head) = (unit / H, unit % H) in 32 bits
  const bool in_bulk = (int)blockIdx.x < bulk_blocks;
  const unsigned blk = in_bulk ? blockIdx.x : blockIdx.x - (unsigned)bulk_blocks;
  int64_t k;
  int h, plane = 0;
  if (const unsigned inverse = (unsigned)call[3]) {              // two divisions were 0.1 to 0.3 us of a short launch
    unsigned unit = blk * kBulkWaves + (unsigned)wave;
    if (PLANES) { plane = unit & 1; unit >>= 1; }
    const unsigned quotient = __umulhi(2 * unit, inverse);
    k = quotient;
    h = (int)(unit - quotient * (unsigned)H);
  } else {
    const unsigned blk_q = blk / (unsigned)H, rest = (blk - blk_q * (unsigned)H) * kBulkWaves + (unsigned)wave;
    const unsigned rest_q = rest / (unsigned)H;
    k = (int64_t)blk_q * kBulkWaves + rest_q;
    h = (int)(rest - rest_q * (unsigned)H);
  }

  // Resolve the run: user, first pool token, length, and the contiguous K / V planes.  A step's append
  // moves little and costs its chain of memory round trips, so whatever can travel together does: the
  // tables are read by scalar loads (nothing here writes them), all of a run's bounds at once, then the
  // page id, then the rows without waiting for it.  Left to itself the compiler made eight or nine
  // round trips of these four (each masked pair of rows waited for): an append of one user's 32 rows of
  // 4 heads of 128 5.1 -> 4.2 us, of 64 users' 8-64 rows of 8 heads of 64 7.7 -> 6.5.
  int u, pos, pbeg, pend;
  int64_t n, t0;
  bool user_ok = true;                                          // an append's grid has one row per user
  if constexpr (FLAT) {
    // User u's sub-blocks start at (its first row) / 16 + 2 u: its rows touch at most as many as there are before the next
    // user's, so no sum over the users is needed.  The lanes look at 64 users at a time, or at every so many of them.
    int first = 0, count = batch;
    const int rows0 = scalar_load(run_user);
    while (count > 64) {
      const int every = (count + 63) / 64, k64 = first + lane * every;
      const bool at_or_before = lane * every < count && (run_user[k64] - rows0) / 16 + 2 * k64 <= k;
      const uint64_t some = __builtin_amdgcn_ballot_w64(at_or_before);
      const int step = (some ? 63 - __builtin_clzll(some) : 0) * every;
      first += step;
      count = count - step < every ? count - step : every;
    }
    int l_r0 = 0, l_r1 = 0, l_pos = 0, l_pbeg = 0, l_pend = 0;
    if (lane < count) {
      l_r0 = run_user[first + lane];
      l_r1 = run_user[first + lane + 1];
      l_pos = run_pos[first + lane];
      l_pbeg = page_indptr[first + lane];
      l_pend = page_indptr[first + lane + 1];
    }
    const uint64_t some = __builtin_amdgcn_ballot_w64(lane < count && (l_r0 - rows0) / 16 + 2 * (first + lane) <= k);
    const int at = some ? 63 - __builtin_clzll(some) : 0;
    u = first + at;
    const int r0 = __builtin_amdgcn_readlane(l_r0, at);
    t0 = r0;
    n = (int64_t)__builtin_amdgcn_readlane(l_r1, at) - t0;
    pos = __builtin_amdgcn_readlane(l_pos, at);
    pbeg = __builtin_amdgcn_readlane(l_pbeg, at);
    pend = __builtin_amdgcn_readlane(l_pend, at);
    k -= (r0 - rows0) / 16 + 2 * u;                             // of this user's
  } else if (MODE == MODE_APPEND) {
    u = s;
    int r0 = scalar_load(run_user + u), r1 = scalar_load(run_user + u + 1);
    pos = scalar_load(run_pos + u);
    pbeg = scalar_load(page_indptr + u);
    pend = scalar_load(page_indptr + u + 1);
    asm volatile("" : "+s"(r0), "+s"(r1), "+s"(pos), "+s"(pbeg), "+s"(pend));   // one wait for all of them
    t0 = r0;
    n = (int64_t)r1 - t0;
  } else {
    u = scalar_load(run_user + s);
    pos = scalar_load(run_pos + s);
    t0 = scalar_load(run_tok + s);
    int64_t t1 = scalar_load(run_tok + s + 1);
    asm volatile("" : "+s"(u), "+s"(pos), "+s"(t0), "+s"(t1));
    n = t1 - t0;
    user_ok = u >= 0 && u < batch;
    const int uc = user_ok ? u : 0;
    pbeg = scalar_load(page_indptr + uc);
    pend = scalar_load(page_indptr + uc + 1);
  }
  const int npg = pend - pbeg;

  const T* k_plane;
  const T* v_plane;
  T* k_out = nullptr;
  T* v_out = nullptr;
  if (MODE == MODE_APPEND) {
    k_plane = src_a + t0 * H * D;
    v_plane = src_b + t0 * H * D;
  } else {
    const int64_t base = t0 * 2 * H * D;
    k_plane = src_a + base;
    v_plane = k_plane + n * H * D;
    if (MODE == MODE_PACK) {
      k_out = dst_contig + base;
      v_out = k_out + n * H * D;
    }
  }
  const bool run_ok = user_ok && n > 0 && pos >= 0;
  const int64_t npos = run_ok ? n : 1, ppos = run_ok ? pos : 0;
  const int64_t first_sb = ppos >> 4, last_sb = (ppos + npos - 1) >> 4;
  // 16-token sub-blocks the run covers completely: [full_lo, full_hi) in units of sub-blocks
  const int64_t full_lo = (ppos + 15) >> 4;
  int64_t full_hi = (ppos + npos) >> 4;
  if (full_hi < full_lo || (!FLAT && bulk_blocks == 0)) full_hi = full_lo;   // a launch of short runs: every sub-block takes the masked form

  // ... and which of its 16 tokens belong to the run
  int64_t sb;
  bool masked = !in_bulk;
  if constexpr (FLAT) {
    sb = first_sb + k;
    if (!run_ok || k < 0 || sb > last_sb) return;
    masked = sb < full_lo || sb >= full_hi;
  } else if (in_bulk) {
    // whole sub-blocks: one wavefront per (sub-block, head)
    sb = full_lo + k;
    if (!run_ok || sb >= full_hi) return;                       // wavefront-uniform; no block barrier below
  } else {
    // the sub-blocks the whole-sub-block part leaves: all of a run's when the launch has no such
    // part (k-th sub-block of the run), else the partly covered ones at its two ends
    if (bulk_blocks == 0) {
      sb = first_sb + k;
    } else {
      const bool head_part = first_sb < full_lo;                            // unit 0: partly covered first
      const bool tail_part = last_sb >= full_hi && !(head_part && last_sb == first_sb);   // unit 1: last
      sb = (k == 0 && head_part) ? first_sb : ((k == 1 && tail_part) ? last_sb : -1);
    }
    if (!run_ok || sb < 0 || sb > last_sb) return;
  }
  const int64_t sbase = sb << 4;
  int t_lo = 0, t_hi = 16;                                      // tokens of the sub-block inside the run
  if (masked) {
    t_lo = (int)(ppos > sbase ? ppos - sbase : 0);
    t_hi = (int)(ppos + npos < sbase + 16 ? ppos + npos - sbase : 16);
  }
  __shared__ __attribute__((aligned(16))) T tile[kBulkWaves][16 * PITCH];
  // masked_c: compile-time copy of `masked`, so that the whole-sub-block form carries no checks; planes_c: K, V or both
  auto move_sub_block = [&](auto masked_c, auto planes_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    constexpr bool KP = decltype(planes_c)::value & 1, VP = decltype(planes_c)::value & 2;
    // A short append's rows are written for late readers: stored the plain way they fill an L2 that writes
    // them back at the kernel's end and push out what the next kernel reads; a step of 64 returning users 247 ->
    // 230 us, 256 users 1109 -> 1064.  A whole prefill's append keeps its rows, the attention that follows
    // reads them all: 16 x 4096 rows x 16 heads of 128, a step of 8 layers, 10.45 ms kept, 10.6 not.
    constexpr bool KEEP = MODE == MODE_APPEND ? !MASKED : PAST != RowsPast::kReadAndWritten;
    constexpr bool KEEP_READ = MODE != MODE_APPEND && PAST == RowsPast::kNone;
    const int64_t row0 = sbase - ppos;                          // contiguous-side row of the sub-block's token 0
    T* lt = tile[wave];                                         // [16 tokens][PITCH]: K first, then V
    // LDS operations of one wavefront execute in order; the fence only pins the compiler's order
    auto wave_sync = [] {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    auto in_run = [&](int t) { return !MASKED || (t >= t_lo && t < t_hi); };
    typedef typename ElemVec<T>::type EV;
    u32x4 kg[NIT], vg[NIT];
    const int64_t lp = sb >> g.sub_shift;
    if (lp >= npg) return;
    const int page = scalar_load(page_indices + pbeg + lp);
    const bool page_ok = (unsigned)page < (unsigned)g.num_pages;
    const int sub = (int)(sb & ((S >> 4) - 1));
    char* head = g.layer_base + (int64_t)page * g.page_bytes;
    T* kblk = reinterpret_cast<T*>(head + head_block_offset(0, h, S, D, sizeof(T))) + (int64_t)sub * 16 * D;
    T* vblk = reinterpret_cast<T*>(head + head_block_offset(1, h, S, D, sizeof(T))) + (int64_t)sub * 16 * D;
    if (MODE != MODE_PACK) {
      // rows in (whole D*es-byte runs); a row outside the run repeats one inside it and goes nowhere
#pragma unroll
      for (int j = 0; j < NIT; ++j) {
        const int gi = j * 64 + lane, c = gi % dch;
        int t = gi / dch;
        if (MASKED) t = t < t_lo ? t_lo : (t < t_hi ? t : t_hi - 1);
        const int64_t off = (row0 + t) * H * D + (int64_t)h * D + c * G;
        if constexpr (KP) kg[j] = load_granule<KEEP_READ>(k_plane + off);
        if constexpr (VP) vg[j] = load_granule<KEEP_READ>(v_plane + off);
      }
      if constexpr (KP) {
#pragma unroll
        for (int j = 0; j < NIT; ++j) {
          const int gi = j * 64 + lane, t = gi / dch, c = gi % dch;
          *reinterpret_cast<u32x4*>(lt + t * PITCH + c * G) = kg[j];
        }
        wave_sync();
#pragma unroll
        for (int j = 0; j < NIT; ++j) {
          const int p = j * 64 + lane;                          // K granule in pool order
          const int half = p / (dch * 8), c = (p / 8) % dch, slot = p % 8;
          const int t = ((slot >> 2) << 3) + half * 4 + (slot & 3);
          kg[j] = *reinterpret_cast<const u32x4*>(lt + t * PITCH + c * G);
        }
      }
      if constexpr (KP && VP) wave_sync();
      if constexpr (VP) {
#pragma unroll
        for (int j = 0; j < NIT; ++j) {
          const int gi = j * 64 + lane, t = gi / dch, c = gi % dch;
          *reinterpret_cast<u32x4*>(lt + t * PITCH + c * G) = vg[j];
        }
        wave_sync();
#pragma unroll
        for (int j = 0; j < NIT; ++j) {
          const int p = j * 64 + lane;                          // V granule: G tokens of one dim
          const int d = p / (16 / G), part = p % (16 / G);
          EV o;
#pragma unroll
          for (int e = 0; e < G; ++e) o[e] = lt[(part * G + e) * PITCH + d];
          vg[j] = __builtin_bit_cast(u32x4, o);
        }
      }
      if (!page_ok) return;                                     // here, so that the rows do not wait for the page id
#pragma unroll
      for (int j = 0; j < NIT; ++j) {
        const int p = j * 64 + lane;
        if constexpr (KP) {
          const int slot = p % 8, half = p / (dch * 8);
          const int t = ((slot >> 2) << 3) + half * 4 + (slot & 3);       // token of K granule p
          if (in_run(t)) store_granule<KEEP>(kblk + (int64_t)p * G, kg[j]);
        }
        if constexpr (VP) if (!MASKED || (t_lo == 0 && t_hi == 16)) store_granule<KEEP>(vblk + (int64_t)p * G, vg[j]);
      }
      if constexpr (VP && MASKED) {
        // V granule p holds tokens part*G .. part*G+G-1 of one dim: of a sub-block that the run covers in part it is whole
        // if the run covers all of them, else it goes in the widest aligned pieces that the run covers - no slot outside the
        // run is written.  Which pieces those are is the same for all lanes of a part.  (Element by element, eight stores of
        // 2 bytes a lane: an append of one user's 32 rows of 4 heads of 128 4.05 -> 3.65 us, of 128 users' 1 row 5.1 -> 4.7.)
        if (t_lo == 0 && t_hi == 16) return;
        const int own = lane % (16 / G);                        // the part of this lane's granules, whatever j
#pragma unroll
        for (int part = 0; part < 16 / G; ++part) {
          const int lo = t_lo - part * G, hi = t_hi - part * G;
          auto covers = [&](int first, int count) { return lo <= first && first + count <= hi; };
          auto misses = [&](int first, int count) { return hi <= first || first + count <= lo; };
          auto store_piece = [&](int first, auto piece) {       // elements `first` .. of the granules, as wide as `piece`
            typedef decltype(piece) Piece;
            constexpr int kCount = sizeof(Piece) / sizeof(T);
            if (own != part) return;
#pragma unroll
            for (int j = 0; j < NIT; ++j) {
              const EV o = __builtin_bit_cast(EV, vg[j]);
              T e[kCount];
#pragma unroll
              for (int k = 0; k < kCount; ++k) e[k] = o[first + k];
              *reinterpret_cast<Piece*>(vblk + (int64_t)(j * 64 + lane) * G + first) = __builtin_bit_cast(Piece, e);
            }
          };
          constexpr int kHalf = G / 2, kQuarter = 4 / sizeof(T);           // elements of 8 and of 4 bytes
          if (misses(0, G)) continue;
          if (covers(0, G)) {
            if (own == part) {
#pragma unroll
              for (int j = 0; j < NIT; ++j) store_granule<KEEP>(vblk + (int64_t)(j * 64 + lane) * G, vg[j]);
            }
            continue;
          }
#pragma unroll
          for (int half = 0; half < G; half += kHalf) {
            if (misses(half, kHalf)) continue;
            if (covers(half, kHalf)) {
              store_piece(half, uint64_t{});
              continue;
            }
#pragma unroll
            for (int quarter = half; quarter < half + kHalf; quarter += kQuarter) {
              if (covers(quarter, kQuarter)) {
                store_piece(quarter, uint32_t{});
              } else if constexpr (kQuarter > 1) {
#pragma unroll
                for (int e = quarter; e < quarter + kQuarter; ++e)
                  if (covers(e, 1)) store_piece(e, T{});
              }
            }
          }
        }
      }
    } else {
      if (!page_ok) return;
      // granules in, in pool order; whole rows out
#pragma unroll
      for (int j = 0; j < NIT; ++j) {
        const int p = j * 64 + lane;
        kg[j] = *reinterpret_cast<const u32x4*>(kblk + (int64_t)p * G);
        vg[j] = *reinterpret_cast<const u32x4*>(vblk + (int64_t)p * G);
      }
#pragma unroll
      for (int j = 0; j < NIT; ++j) {
        const int p = j * 64 + lane;
        const int half = p / (dch * 8), c = (p / 8) % dch, slot = p % 8;
        const int t = ((slot >> 2) << 3) + half * 4 + (slot & 3);
        *reinterpret_cast<u32x4*>(lt + t * PITCH + c * G) = kg[j];
      }
      wave_sync();
#pragma unroll
      for (int j = 0; j < NIT; ++j) {
        const int gi = j * 64 + lane, t = gi / dch, c = gi % dch;
        kg[j] = *reinterpret_cast<const u32x4*>(lt + t * PITCH + c * G);
      }
      wave_sync();
#pragma unroll
      for (int j = 0; j < NIT; ++j) {
        const int p = j * 64 + lane;
        const int d = p / (16 / G), part = p % (16 / G);
        const EV iv = __builtin_bit_cast(EV, vg[j]);
#pragma unroll
        for (int e = 0; e < G; ++e) lt[(part * G + e) * PITCH + d] = iv[e];
      }
      wave_sync();
#pragma unroll
      for (int j = 0; j < NIT; ++j) {
        const int gi = j * 64 + lane, t = gi / dch, c = gi % dch;
        if (in_run(t)) {
          const int64_t off = (row0 + t) * H * D + (int64_t)h * D + c * G;
          store_granule<KEEP>(k_out + off, kg[j]);
          store_granule<KEEP>(v_out + off, *reinterpret_cast<const u32x4*>(lt + t * PITCH + c * G));
        }
      }
    }
  };
  if constexpr (PLANES) {
    if (plane == 0) move_sub_block(std::true_type{}, std::integral_constant<int, 1>{});
    else move_sub_block(std::true_type{}, std::integral_constant<int, 2>{});
  } else {
    constexpr std::integral_constant<int, 3> both{};
    if (masked) move_sub_block(std::true_type{}, both);
    else move_sub_block(std::false_type{}, both);
  }
}

template <typename T, int MODE, int DCH>
void launch_typed(const PoolGeom& g, const SegDev& segs, const BatchDev& b, dim3 grid, int bulk_blocks,
                  const void* a, const void* bsrc, void* dst, int64_t pool_layer_stride,
                  int64_t contig_layer_stride_bytes, unsigned inverse, Units units, hipStream_t stream) {
  constexpr RowsPast kBoth = RowsPast::kReadAndWritten, kRead = RowsPast::kRead, kNone = RowsPast::kNone;
  auto kern = kv_move_kernel<T, MODE, DCH, MODE != MODE_PACK || gather_past_caches(DCH * 16) ? kBoth : kNone, Units::kRuns>;
  if constexpr (MODE == MODE_UNPACK) {
    const RowsPast past = scatter_past_caches((int64_t)segs.num_segs * segs.max_seg_tokens, (int64_t)b.total_pages * g.S,
                                              2ll * g.H * g.D * g.es, grid.z);
    if (past != kBoth) kern = past == kRead ? kv_move_kernel<T, MODE, DCH, kRead, Units::kRuns> : kv_move_kernel<T, MODE, DCH, kNone, Units::kRuns>;
  }
  constexpr bool kAppend = MODE == MODE_APPEND;
  if constexpr (kAppend) {
    if (units == Units::kPlanes) kern = kv_move_kernel<T, MODE, DCH, kBoth, Units::kPlanes>;
    if (units == Units::kFlat) kern = kv_move_kernel<T, MODE, DCH, kBoth, Units::kFlat>;
  }
  hipLaunchKernelGGL(kern, grid, dim3(256, 1, 1), 0, stream,
                     kAppend ? run_tables(b) : table_words(segs.seg_user, segs.seg_pos), page_tables(b),
                     CallWords{b.batch, g.H, bulk_blocks, (int)inverse}, segs.seg_tok_indptr,
                     MoveSides<T>{g, (const T*)a, (const T*)bsrc, (T*)dst, pool_layer_stride,
                                  contig_layer_stride_bytes / (int64_t)sizeof(T)});
}

template <int MODE>
hipError_t launch_move(const PoolGeom& g, const SegDev& segs, const BatchDev& b, int runs,
                       int64_t max_run_tokens, const void* a, const void* bsrc, void* dst,
                       hipStream_t stream, int layers = 1, int64_t pool_layer_stride = 0,
                       int64_t contig_layer_stride_bytes = 0) {
  if (runs <= 0 || max_run_tokens <= 0 || layers <= 0) return hipSuccess;
  if (layers > 65535) return hipErrorInvalidValue;
  const int G = 16 / g.es;
  // One wavefront per (16-token sub-block, head).  Runs of at least kBulkRun tokens: the sub-blocks a
  // run covers completely (of the longest run) take the unmasked form, the at most two partly
  // covered ones at its ends the masked form.  Shorter runs (a step's few new tokens): every
  // sub-block a run touches, at most ceil(max / 16) + 1, takes the masked form.
  const bool bulk = max_run_tokens >= kBulkRun;
  const int64_t bulk_units = bulk ? (max_run_tokens / 16) * (int64_t)g.H : 0;
  const int64_t bulk_blocks = (bulk_units + kBulkWaves - 1) / kBulkWaves;
  const int64_t end_units = (bulk ? 2 : (max_run_tokens + 15) / 16 + 1) * (int64_t)g.H;
  int64_t blocks = bulk_blocks + (end_units + kBulkWaves - 1) / kBulkWaves;
  const int64_t flat_units = MODE == MODE_APPEND ? ((int64_t)b.total_new / 16 + 2ll * b.batch) * g.H : 0;
  const int64_t flat_blocks = (flat_units + kBulkWaves - 1) / kBulkWaves;
  const bool flat = MODE == MODE_APPEND && append_flat(max_run_tokens, blocks * runs * layers, flat_blocks * layers);
  // unit / H = the upper word of 2 * unit * inverse while unit * H < 2^31
  const int64_t most_units = (flat ? flat_units : bulk_units > end_units ? bulk_units : end_units) + kBulkWaves;
  const unsigned inverse = 2 * most_units * g.H < (1ll << 31) ? (unsigned)(((1ull << 31) + g.H - 1) / g.H) : 0;
  const bool planes = MODE == MODE_APPEND && !flat && !bulk && inverse != 0 && append_by_planes(g.D * g.es, end_units * runs * layers);
  const Units units = flat ? Units::kFlat : planes ? Units::kPlanes : Units::kRuns;
  if (flat) {
    blocks = flat_blocks;
    runs = 1;
  } else if (planes) {
    blocks = (end_units * 2 + kBulkWaves - 1) / kBulkWaves;
  }
  if (blocks > 0x7fffffffll) return hipErrorInvalidValue;
  dim3 grid((unsigned)blocks, (unsigned)runs, (unsigned)layers);
  const int dch = g.D / G;
#define MTS_MOVE_CASE(T, DCH_) \
  case DCH_: launch_typed<T, MODE, DCH_>(g, segs, b, grid, flat ? 0 : (int)bulk_blocks, a, bsrc, dst, pool_layer_stride, \
                                         contig_layer_stride_bytes, inverse, units, stream); break;
  if (g.es == 2) {
    switch (dch) {
      MTS_MOVE_CASE(uint16_t, 4) MTS_MOVE_CASE(uint16_t, 8) MTS_MOVE_CASE(uint16_t, 16)
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (dch) {
      MTS_MOVE_CASE(uint32_t, 8) MTS_MOVE_CASE(uint32_t, 16) MTS_MOVE_CASE(uint32_t, 32)
      default: return hipErrorInvalidValue;
    }
  }
#undef MTS_MOVE_CASE
  return hipGetLastError();
}

}  // namespace

hipError_t launch_unpack(const PoolGeom& g, const void* staging, const SegDev& segs, const BatchDev& b,
                         hipStream_t stream, int layers, int64_t pool_layer_stride, int64_t staging_layer_stride) {
  return launch_move<MODE_UNPACK>(g, segs, b, segs.num_segs, segs.max_seg_tokens, staging, nullptr,
                                  nullptr, stream, layers, pool_layer_stride, staging_layer_stride);
}

hipError_t launch_pack(const PoolGeom& g, void* staging_out, const SegDev& segs, const BatchDev& b,
                       hipStream_t stream, int layers, int64_t pool_layer_stride, int64_t staging_layer_stride) {
  return launch_move<MODE_PACK>(g, segs, b, segs.num_segs, segs.max_seg_tokens, staging_out, nullptr,
                                staging_out, stream, layers, pool_layer_stride, staging_layer_stride);
}

hipError_t launch_append(const PoolGeom& g, const void* k_new, const void* v_new, const BatchDev& b,
                         hipStream_t stream, int layers, int64_t pool_layer_stride, int64_t rows_layer_stride) {
  SegDev none{};
  return launch_move<MODE_APPEND>(g, none, b, b.batch, b.max_new, k_new, v_new, nullptr, stream, layers,
                                  pool_layer_stride, rows_layer_stride);
}

}  // namespace mts
