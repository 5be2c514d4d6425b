// The rules by which the attention chooses its forms, at sizes on both sides of each line;
// compiling it is the check.
#include "../../paper_2604_22881_amd/csrc/mts_attn_rules.hpp"

using mts::f32_takes_plain;
using mts::joins_pieces;
using mts::kv_past_caches;
using mts::least_share;
using mts::prefill_shares;
using mts::PrefillShares;
using mts::stream_form;
using mts::StreamCall;
using mts::StreamForm;
constexpr int64_t MB = 1000000;

// bound by reading K/V: past the caches
static_assert(kv_past_caches(64, 219 * MB, 4, 1600), "64 users of about 1600 tokens");
static_assert(kv_past_caches(64, 1400 * MB, 4, 2600), "");
static_assert(kv_past_caches(128, 1300 * MB, 8, 10000), "");
static_assert(kv_past_caches(128, 860 * MB, 8, 3300), "");
static_assert(kv_past_caches(128, 400 * MB, 1, 3000), "");
// the layers stay in the last-level cache from step to step
static_assert(!kv_past_caches(128, 13 * MB, 8, 6400), "");
static_assert(!kv_past_caches(128, 135 * MB, 1, 1000), "");
static_assert(!kv_past_caches(128, 260 * MB, 1, 2000), "");
static_assert(!kv_past_caches(64, 260 * MB, 1, 4000), "");
static_assert(!kv_past_caches(64, 135 * MB, 2, 2000), "");
// many short users: a segment's last tile is loaded several times
static_assert(!kv_past_caches(128, 170 * MB, 4, 64), "1300 users of 40 tokens in 32-token pages");
static_assert(!kv_past_caches(128, 445 * MB, 4, 64), "");
static_assert(!kv_past_caches(64, 445 * MB, 4, 64), "");
static_assert(!kv_past_caches(128, 520 * MB, 2, 450), "");
static_assert(kv_past_caches(128, 520 * MB, 2, 1000), "");
static_assert(!kv_past_caches(64, 520 * MB, 2, 200), "");
static_assert(kv_past_caches(64, 520 * MB, 2, 300), "");
// the largest values of the arguments do not overflow
static_assert(kv_past_caches(64, 1ll << 62, INT32_MAX, 1ll << 37), "");

// launches that fill the chip fold pieces inside workgroups, a single user's do not ...
static_assert(joins_pieces(400, 128, 64, 16, false) && joins_pieces(1024, 4, 128, 64, false), "");
static_assert(!joins_pieces(20, 4, 128, 64, false) && !joins_pieces(112, 8, 64, 64, false), "");
static_assert(!joins_pieces(336, 64, 128, 64, false) && !joins_pieces(152, 32, 64, 16, true), "");
// ... unless the merge of their many pieces is the longer chain
static_assert(joins_pieces(212, 4, 128, 32, false) && joins_pieces(336, 32, 64, 32, true) && joins_pieces(36, 4, 32, 16, false), "");
static_assert(!joins_pieces(336, 32, 64, 32, false) && !joins_pieces(60, 4, 32, 64, false), "");

// small calls: whole pairs up to the length that one CU reads in time ...
static_assert(stream_form(128, 32, 4, 36, 1 * MB) == StreamForm::kWholePairs && stream_form(64, 32, 256, 52, 90 * MB) == StreamForm::kWholePairs, "");
static_assert(stream_form(64, 64, 16, 44, 5 * MB) == StreamForm::kWholePairs && stream_form(32, 16, 16, 68, 5 * MB) == StreamForm::kWholePairs, "");
static_assert(stream_form(128, 16, 512, 24, 90 * MB) == StreamForm::kWholePairs && stream_form(32, 32, 2048, 32, 90 * MB) == StreamForm::kWholePairs, "");
// ... then pieces, of few pairs and while reading K/V is not yet the most of it
static_assert(stream_form(128, 32, 4, 37, 1 * MB) == StreamForm::kPieces && stream_form(64, 64, 96, 45, 80 * MB) == StreamForm::kPieces, "");
static_assert(stream_form(128, 32, 96, 300, 160 * MB) == StreamForm::kPieces && stream_form(64, 32, 96, 300, 84 * MB) == StreamForm::kShares, "");
static_assert(stream_form(128, 32, 97, 37, 30 * MB) == StreamForm::kShares && stream_form(128, 32, 96, 400, 168 * MB) == StreamForm::kShares, "");
// (the pairs of the piece tests, on the pool's rows and on staged ones)
static_assert(stream_form(32, 16, 15, 96, 1 * MB) == StreamForm::kPieces && stream_form(64, 64, 30, 98, 2 * MB) == StreamForm::kPieces, "");
static_assert(stream_form(128, 64, 42, 98, 4 * MB) == StreamForm::kPieces && stream_form(64, 16, 2, 376, 3 * MB) == StreamForm::kPieces, "");
// ... and, of head_dim 32, while they are few tiles, each query tile's own counted
static_assert(stream_form(32, 64, 96, 300, 32 << 20) == StreamForm::kPieces && stream_form(32, 64, 96, 300, 33 << 20) == StreamForm::kShares, "");
static_assert(stream_form(32, 48, 8, 800, 16 << 20, 2) == StreamForm::kPieces && stream_form(32, 48, 8, 800, 17 << 20, 2) == StreamForm::kShares, "");
static_assert(stream_form(32, 64, 8, 800, 24 << 20, 1, StreamCall::kPointwise) == StreamForm::kPieces, "");
static_assert(stream_form(32, 64, 8, 800, 25 << 20, 1, StreamCall::kPointwise) == StreamForm::kShares, "");
static_assert(stream_form(32, 64, 8, 800, 64 << 20, 1, StreamCall::kStaged) == StreamForm::kPieces, "");
static_assert(stream_form(32, 32, 8, 800, 65 << 20, 1, StreamCall::kStaged) == StreamForm::kShares, "");
static_assert(stream_form(32, 16, 8, 800, 32 << 20, 1, StreamCall::kStaged) == StreamForm::kPieces, "");
static_assert(stream_form(32, 16, 8, 800, 33 << 20, 1, StreamCall::kStaged) == StreamForm::kShares, "");
static_assert(stream_form(32, 32, 96, 300, 80 << 20) == StreamForm::kPieces && stream_form(64, 64, 96, 300, 80 << 20, 2) == StreamForm::kPieces, "");
// staged histories: few whole pairs are shorter ones
static_assert(stream_form(64, 32, 32, 39, 5 * MB, 1, StreamCall::kStaged) == StreamForm::kWholePairs, "");
static_assert(stream_form(64, 32, 32, 40, 5 * MB, 1, StreamCall::kStaged) == StreamForm::kPieces, "");
static_assert(stream_form(64, 32, 33, 52, 5 * MB, 1, StreamCall::kStaged) == StreamForm::kWholePairs, "");
static_assert(stream_form(64, 32, 32, 52, 5 * MB) == StreamForm::kWholePairs, "");
// pairs that take their turns on a CU
static_assert(stream_form(128, 32, 257, 1, 10 * MB) == StreamForm::kShares && stream_form(128, 16, 513, 1, 10 * MB) == StreamForm::kShares, "");
static_assert(stream_form(64, 32, 513, 1, 10 * MB) == StreamForm::kShares && stream_form(64, 16, 513, 16, 90 * MB) == StreamForm::kWholePairs, "");
static_assert(stream_form(32, 16, 2049, 1, 10 * MB) == StreamForm::kShares && stream_form(32, 48, 513, 1, 10 * MB) == StreamForm::kShares, "");
static_assert(stream_form(64, 64, 1ll << 30, 1ll << 26, 1ll << 62) == StreamForm::kShares, "");

// a wavefront's least share is a whole tile, and a workgroup's four fit 32 bits
static_assert(least_share(1, 1) == 1 && least_share(1, 2) == 2 && least_share(4, 2) == 4 && least_share(1 << 28, 1) == 1 << 28, "");
static_assert(4ll * least_share(1 << 29, 1) <= INT32_MAX && 4ll * least_share(INT32_MAX, 2) <= INT32_MAX, "");

// split prefill: the shares are the sequence, one after the other, and every step finds its own
constexpr bool shares_cover(int total, int wgs, int min_steps, bool fills_chip) {
  const PrefillShares s = prefill_shares(total, wgs, min_steps, fills_chip);
  if (s.begin(0) != 0 || s.end(wgs - 1) < total) return false;
  for (int w = 0; w < wgs; ++w) {
    const int64_t lo = s.begin(w), hi = s.end(w);
    if (lo < 0 || hi < lo || (w + 1 < wgs && s.begin(w + 1) != hi)) return false;
    if (!fills_chip && hi < total && hi - lo < min_steps) return false;
    if (lo < total && (hi == lo || s.of((int)lo) != w || s.of((int)((hi < total ? hi : total) - 1)) != w)) return false;
  }
  return true;
}
static_assert(shares_cover(1, 512, 12, true) && shares_cover(511, 512, 1, true) && shares_cover(512, 512, 1, true), "");
static_assert(shares_cover(513, 512, 1, true) && shares_cover(1537, 512, 3, true) && shares_cover(26624, 512, 12, true), "");
static_assert(shares_cover(26624, 510, 12, false) && shares_cover(100, 7, 3, false) && shares_cover(100, 1, 1, false), "");
static_assert(shares_cover(INT32_MAX, 512, 12, true) && shares_cover(INT32_MAX, 128, 1, false), "");
// the least share may be any number that the tuning takes: everything in the first share, or in two
static_assert(shares_cover(26624, 512, 1 << 29, true) && shares_cover(26624, 512, (1 << 30) - 1, true), "");
static_assert(shares_cover(26624, 512, 1 << 30, true) && shares_cover(26624, 512, INT32_MAX, true), "");
static_assert(shares_cover(26624, 7, 1 << 30, false) && shares_cover(1, 1, INT32_MAX, false), "");
static_assert(shares_cover(INT32_MAX, 512, 1 << 30, true) && shares_cover(INT32_MAX, 8, INT32_MAX, false), "");

// fp32: many users of a few keys, in pages of 16 and 64 tokens ...
static_assert(f32_takes_plain(32, 8, 1000, 1000, 1, 8, 16000) && f32_takes_plain(32, 8, 1000, 1000, 1, 32, 32000), "");
static_assert(f32_takes_plain(64, 8, 1000, 1000, 1, 8, 16000) && f32_takes_plain(64, 8, 4000, 16000, 4, 16, 64000), "");
static_assert(f32_takes_plain(128, 8, 256, 256, 1, 32, 8192) && f32_takes_plain(128, 8, 4000, 4000, 1, 4, 64000), "");
static_assert(f32_takes_plain(64, 8, 1000, 1000, 1, 8, 64000), "");
static_assert(f32_takes_plain(64, 8, 1000, 1000, 1, 100, 16000), "one longer user among them");
// ... but no longer ones, no few, and none with many queries
static_assert(!f32_takes_plain(32, 8, 1000, 1000, 1, 96, 96000) && !f32_takes_plain(64, 8, 1000, 4000, 4, 32, 32000), "");
static_assert(!f32_takes_plain(64, 8, 1000, 1000, 1, 48, 48000) && !f32_takes_plain(64, 8, 1000, 2000, 2, 32, 32000), "");
static_assert(!f32_takes_plain(64, 8, 1000, 8000, 8, 13, 16000), "never beyond 64 a workgroup");
static_assert(!f32_takes_plain(128, 8, 1000, 1000, 1, 32, 32000) && !f32_takes_plain(128, 2, 1000, 4000, 4, 8, 16000), "");
static_assert(!f32_takes_plain(32, 4, 1, 1, 1, 300, 304) && !f32_takes_plain(64, 8, 8, 8, 1, 8, 128), "");
static_assert(!f32_takes_plain(64, 8, 1000, 1000, 1, 3000, 16000), "the launch would wait for the longest");
static_assert(!f32_takes_plain(32, 8, 1000, 64000, 64, 64, 64000), "");
// the largest values of the arguments do not overflow
static_assert(!f32_takes_plain(128, 65535, INT32_MAX, INT32_MAX, INT32_MAX, 1 << 22, 1ll << 37), "");
