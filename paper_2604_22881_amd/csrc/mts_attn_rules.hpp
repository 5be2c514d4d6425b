// Where the forms of the attention change over, and how a split prefill launch is shared out: rules on sizes.
#pragma once
#include <stdint.h>

namespace mts {

// Whether a call of one query tile per user loads its K/V tiles past the caches' retention.
// It pays (8-11 % of the step at head_dim 64, 2-10 % at 128) where nothing of a tile is read again:
// * The layers of a step together are larger than what the last-level cache (256 MB) hands to the next
//   step.  Step time, past the caches / ordinary, of 290, 320, 350, 380 MB over 1 layer: 1.05 1.00 0.95 0.90 at
//   head_dim 64, 1.15 1.11 1.00 0.98 at 128; over 2 layers 1.04 1.00 0.94 0.92 and 1.16 1.10 1.06 1.00.
// * Users are long.  The ring of a segment loads its last tile again and again past the segment's end, which
//   costs nothing while caches hold it: users of 40, 130, 200, 300, 450 tokens 1.12 1.05 0.99 0.96 0.94 at head_dim
//   64 (8 layers of 150 MB; 1.02 at 200 and 1.00 at 260 in 2 layers of 1 GB), of 40, 200, 450, 700, 1000 tokens
//   1.27 1.08 1.01 0.98 0.96 at 128 (4 layers of 260, 2 of 520 MB), whose ring and tiles are larger.
// * The call is long enough for its bandwidth to matter: 4 layers of 135, 170, 210, 260, 400 MB 0.93 0.91 0.91
//   0.91 0.90 at head_dim 64, 1.02 1.01 0.99 0.98 0.96 at 128.
constexpr bool kv_past_caches(int head_dim, int64_t call_bytes, int64_t layers, int64_t tokens_per_user) {
  return head_dim == 128 ? call_bytes >= (192ll << 20) && call_bytes >= (368ll << 20) / layers && tokens_per_user >= 768
                         : call_bytes >= (128ll << 20) && call_bytes >= (320ll << 20) / layers && tokens_per_user >= 256;
}

// Whether the pieces of a (query tile, head) that lie in one workgroup's shares are folded inside the
// workgroup.  It saves partials and merge work, and costs a launch of few workgroups, which ends with its
// longest chain, the barrier and the serial fold.  Step of 8 layers, us, folded / not:
// * launches of 384 wavefronts and more: 16 users x 1000 keys + 16 new x 4 heads of 128 190 / 198, 32 x 600 + 24 x 4
//   of 128 229 / 258, 16 x 300 + 64 x 8 of 64 172 / 176, 64 x 64 + 64 x 8 of 64 189 / 202; below, 1 x 300 + 64 x 4 of
//   128 164 / 147, 16 x 300 + 64 x 4 of 128 223 / 206, 1 x 1500 + 50 x 8 of 64 138 / 132;
// * pairs of so many pieces that the merge is the longer chain: 32 and more, 1 x 6400 + 32 x 4 of 128 191 / 197;
//   8 and more where pieces are small, 4 x 1000 + 32 x 8 of 64 pointwise 116 / 125, 1 x 700 + 16 x 4 of 32 94 / 99.
constexpr bool joins_pieces(int64_t waves, int64_t pairs, int head_dim, int q_tile, bool pointwise) {
  return waves >= 384 || waves >= 32 * pairs || (waves >= 8 * pairs && q_tile <= 32 && (pointwise || head_dim == 32));
}

// How the streaming kernel divides a call's (query tile, head)s, `pairs` of at most `max_tiles` 32-token tiles: even
// shares of wavefronts; a workgroup per pair; or a workgroup per equal piece of a pair, and a merge launch.
// Step time over that of even shares, whole pairs / pieces, of 1000 random calls of up to 100 MB a layer (geometric
// means; q: queries per tile; the kernels of pairs and pieces take 0.95 to 1.00 of the time they took then):
// * Up to 256 pairs a CU holds one, whose keys it alone reads: head_dim 128 16-32 tiles 0.77 / 0.89, 32-40 0.84 / 0.88,
//   40-52 0.92 / 0.88, 64-80 1.16 / 0.90; 64, q <= 32 32-40 0.80 / 0.92, 40-52 0.84 / 0.94, 52-64 0.90 / 0.95, 80-110 1.04 / 0.94;
//   32 0.73 / 0.93, 0.82 / 0.95, 64-80 0.89 / 0.94, 80-110 0.97 / 0.92; q > 32, both, 24-32 0.77 / 0.88, 32-40 0.88 / 0.92,
//   64-80 1.1 / 0.95.
// * Up to 512 pairs two share a CU where registers allow, and the longest ones are the launch's end: 8-32 tiles
//   head_dim 128, q <= 16 0.88 to 0.92 of even shares, more queries 0.95 to 1.05; 64 0.71 to 0.85 (longer ones 0.91 to 1.2), 32
//   0.67 to 0.75.  Beyond, a CU starts one after the other: head_dim 64, q <= 16 up to 16 tiles 0.82 to 0.9, more queries 0.97 to
//   1.09; 32, q <= 32 up to 32 tiles 0.79 to 0.88, q > 32 0.92 to 1.03; 128 0.91 to 1.5.
// * Pieces: 40 tiles and more, head_dim 128 up to 160 MB a layer 0.89 to 0.95, 200-300 MB 0.94 to 1.02; 64 up to 80 MB 0.93 to 0.95, 120
//   MB 0.84 to 1.04, 160 MB 1.07 to 1.17.  Each pair rounds its pieces up, so of many pairs the longest ones wait: 97-128
//   pairs 0.94 to 1.24, 129-255 0.98 to 1.26.
// * Staged users' tiles take longer, and of few pairs theirs are the longest: from three quarters of these lengths, all head sizes,
//   1-2 users whole pairs 0.88 to 1.21 / pieces 0.83 to 0.89 of the time before either (up to 32 pairs), 3-8 users 0.79 to
//   1.13 / 0.85 to 0.96; more pairs 0.74 to 1.05 / 0.83 to 0.91.
// * head_dim 32: K/V are little to read, and a launch of many tiles ends with the CUs that the rounding of the pieces
//   left more of them, each wavefront of more than 32 queries with one tile in flight.  By tiles of the call, thousands, more than
//   32 queries: softmax up to 6 0.85 to 1.02, 6-8 0.93 to 1.02, 8-10 0.92 to 1.07, 10-14 0.99 to 1.24, 14-31 0.98 to
//   1.32; pointwise up to 6 0.88 to 0.95, 6-8 0.96 to 1.13, 11-19 1.05 to 1.38.  Staged, 16 queries: up to 8 0.88 to 1.07,
//   8-18 0.97 to 1.18; more: up to 16 0.85 to 1.00, 17-38 0.97 to 1.13.  Else up to the 20 of 80 MB 0.92 to 1.08.
enum class StreamForm { kShares, kWholePairs, kPieces };
enum class StreamCall { kSoftmax, kPointwise, kStaged };
// `q_tiles`: query tiles of a user, each of which reads the call's bytes
constexpr StreamForm stream_form(int head_dim, int q_tile, int64_t pairs, int64_t max_tiles, int64_t call_bytes, int64_t q_tiles = 1,
                                 StreamCall call = StreamCall::kSoftmax) {
  const int64_t whole = pairs <= 256   ? (head_dim == 128 ? 36 : q_tile > 32 ? 44 : head_dim == 64 ? 52 : 68)
                        : pairs <= 512 ? (head_dim == 32 ? 32 : head_dim == 64 || q_tile <= 16 ? 24 : 0)
                        : pairs > 2048 ? 0
                        : head_dim == 32 ? (q_tile <= 32 ? 32 : 0)
                                         : (head_dim == 64 && q_tile <= 16 ? 16 : 0);
  if (max_tiles <= (call == StreamCall::kStaged && pairs <= 32 ? whole * 3 / 4 : whole)) return StreamForm::kWholePairs;
  if (pairs > 96 || call_bytes > (head_dim == 128 ? 160ll << 20 : 80ll << 20)) return StreamForm::kShares;
  if (head_dim != 32) return StreamForm::kPieces;
  const int64_t tiles = call_bytes / (128 * head_dim) * q_tiles;          // a tile of K/V of a head is 128 * head_dim bytes
  const int64_t most = call == StreamCall::kStaged ? (q_tile > 16 ? 16384 : 8192)
                       : q_tile <= 32              ? INT64_MAX
                                                   : (call == StreamCall::kPointwise ? 6144 : 8192);
  return tiles <= most ? StreamForm::kPieces : StreamForm::kShares;
}

// Least share of a wavefront of the streaming kernel, in units of the schedule: a whole tile of the onload buffer, so that
// every share between a pair's first and last has a piece of it.  mts_attn_tuning takes any number; four of them, a
// workgroup's, are held in 32 bits.
constexpr int least_share(int min_tiles, int tile_cost) {
  return min_tiles < tile_cost ? tile_cost : min_tiles < INT32_MAX / 4 ? min_tiles : INT32_MAX / 4;
}

// Shares of a split prefill launch: workgroup `wid` of it takes the tile steps [begin(wid), end(wid)) of the call's
// sequence of `total`.  Shares 2 k and 2 k + 1 are a CU's two in a launch that fills the chip, and there the first is
// the larger one, kFirstShare per cent of both: the workgroup that came first is served first (of equal shares the first
// ended after 59 us of a launch and the second after 72).  A step by the first one's part, 50 / 58 / 62 / 66 / 70 per cent: one
// user's 5189 tokens x 4 heads of 128 445, 441, 439, 446, 461 us; beside two of 4-6 K six users behind 5-11 K 764, 742, 749,
// 757, 771; 12000 x 4 of 64 846, 811, 796, 830, 822; 2 of 4-6 K and 25 behind 600 x 8 of 64 920, 891, 899, 921, 953.
constexpr int kFirstShare = 60;
struct PrefillShares {
  int per_two, per_first;      // steps of shares 2 k and 2 k + 1 together, of the first of them
  bool paired;                 // the two are a CU's, and unequal
  constexpr int64_t begin(int wid) const { return (int64_t)(wid >> 1) * per_two + (wid & 1) * per_first; }
  constexpr int64_t end(int wid) const { return begin(wid) + ((wid & 1) ? per_two - per_first : per_first); }
  constexpr int of(int pos) const {                             // the share that holds step `pos`
    const int two = pos / per_two;
    return 2 * two + (pos - two * per_two >= per_first);
  }
};
// `min_steps`, the least share, may be any positive number: where twice it does not fit, share 1 ends past every step.
constexpr PrefillShares prefill_shares(int total, int wgs, int min_steps, bool fills_chip) {
  if (fills_chip && total / wgs >= min_steps) {
    const int two = (total - 1) / (wgs / 2) + 1, first = two * kFirstShare / 100 + 1;
    return {two, first < two ? first : two - 1, true};
  }
  int first = (total - 1) / wgs + 1;
  if (first < min_steps) first = min_steps;
  return {first < (1 << 30) ? 2 * first : INT32_MAX, first, false};
}

// Whether an fp32 call goes to the plain kernel.  A workgroup of the matrix-core kernel is eight wavefronts that
// find their user, read at least one 16-token sub-block and combine: 6.3, 8, 19.5 ns of the whole chip at head_dim
// 32, 64, 128 however short the user is.  The plain kernel pays per (query, key).  us, matrix cores / plain, at 1000 users x 8
// heads, 1 new token of 8 keys, 1 of 32, 1 of 48, 2 of 32, 4 of 16: head_dim 32 51 / 14, 50 / 35, 52 / 51, 53 / 61, 56 / 64; 64
// 63 / 22, 68 / 68, 78 / 108, 74 / 123, 69 / 104; 128 166 / 90, 175 / 338, 191 / 510, 191 / 590, 191 / 494; at 256 users of 32
// keys 14 / 15, 19 / 18, 42 / 29.  `max_new` times all keys and `total_new` times the longest user's both bound the (query, key)
// pairs of the call, by half as much again where lengths differ, twice where new tokens do too; the limits are for
// such calls: 64 a workgroup less 8 a query at head_dim 32; 38 and 7 more a query, 64 at most, at 64 (58 random calls between this and
// the 64 of the time when a workgroup took 14 ns, matrix cores over plain: 0.56 to 1.05 and one of 1.10; 1.00 to 1.35 just below it); 68 less 16
// at 128, and 18 where K/V come from beyond the caches (1.65 to 1.95 just below).  A call that does not fill the chip waits for the plain kernel's longest chain of keys, 0.3 us each: 16 users x
// 1000 keys 13 / 301 at head_dim 32.
constexpr bool f32_takes_plain(int head_dim, int64_t heads, int64_t users, int64_t total_new, int64_t max_new,
                               int64_t max_len, int64_t page_tokens) {
  const int64_t blocks = total_new / 16 + users;
  if (300 * max_len + 3000 >= blocks * heads * (head_dim == 32 ? 7 : head_dim == 64 ? 11 : 22)) return false;
  const bool far = head_dim == 128 && page_tokens * heads * 1024 > (96ll << 20);
  const int64_t more = 7 * total_new < 26 * blocks ? 7 * total_new : 26 * blocks;      // head_dim 64's, up to 64 a workgroup in all
  const int64_t room = head_dim == 64 ? blocks * 38 + more
                                      : blocks * (head_dim == 32 ? 64 : far ? 18 : 68) - total_new * (head_dim == 32 ? 8 : far ? 0 : 16);
  return total_new * max_len < room || (max_new <= room / (page_tokens > 0 ? page_tokens : 1) && max_new * page_tokens < room);
}

}  // namespace mts
