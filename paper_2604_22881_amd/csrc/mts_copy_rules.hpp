// Which copies move their rows past the caches' retention: host-only rules on sizes.  Stored the plain way, many
// rows fill an L2 that writes them back at the kernel's end; few find room in the last-level cache (256 MB).
// Times are those past the caches over plain ones, of copies repeated on the same buffers.
#pragma once
#include <stdint.h>

namespace mts {

enum class RowsPast { kNone, kRead, kReadAndWritten };

// Scatter, by the bytes of all layers of the launch.
// * Stores: 100-120 MB 1.07, 140-270 MB 1.08 to 1.18, 300 MB 1.03, 360 MB and more 0.91 to 0.98; below, with plain
//   loads beside them, 1.05 to 1.08 at 27-90 MB and nothing under that.
// * Loads: where rows and pool pages together are more than the cache, plain loads push out what the stores put
//   there; of both plain, 180-360 MB take 0.73 to 0.99 of the time with loads past the caches.
// `run_tokens` (runs times the longest) and `held_tokens` (the batch's pages) both bound the tokens that are moved.
constexpr RowsPast scatter_past_caches(int64_t run_tokens, int64_t held_tokens, int64_t token_bytes, int64_t layers) {
  const int64_t tokens = held_tokens > 0 && held_tokens < run_tokens ? held_tokens : run_tokens;
  return tokens >= (336ll << 20) / token_bytes / layers   ? RowsPast::kReadAndWritten
         : tokens >= (160ll << 20) / token_bytes / layers ? RowsPast::kRead
                                                          : RowsPast::kNone;
}

// Gather, by the bytes of a token's row of one head: rows of 128 and more 0.99 to 1.00 up to 100 MB, 0.95 at 130,
// 0.79 to 0.81 at 180-260, 0.94 to 0.98 beyond; rows of 64, half a cache line each, 1.10 to 1.21 at 35-115 MB,
// 1.03 to 1.08 beyond 330.
constexpr bool gather_past_caches(int row_bytes) { return row_bytes >= 128; }

// Whether K and V of a short append's sub-block are moved by a wavefront each, `units` of them (sub-block, head, user,
// layer) in the launch.  A launch of few is its longest chain, half as long then: rows of 256 bytes and more 0.74 to 0.97
// of the time up to 9 000 units, 1.00 to 1.05 at 19 000 and more; of 128 bytes 0.93 to 0.97 up to 500, 1.02 to 1.12
// at 1 100 to 6 000 (more wavefronts, each with little to do); of 64 bytes 1.00 to 1.06.
constexpr bool append_by_planes(int row_bytes, int64_t units) {
  return row_bytes >= 256 ? units <= 16384 : row_bytes == 128 && units <= 1024;
}

// The shortest longest run of a launch whose whole sub-blocks take a form of their own, without a token mask.
constexpr int64_t kBulkRun = 128;

// Whether an append's workgroups are numbered through the users' rows, `flat` of them at most, and not by the longest user's for
// each user, `rectangle` of them: a workgroup that finds nothing to move costs the launch up to a nanosecond, finding one's user
// half a microsecond.  Of 70 random calls of 2 to 180 users, one to four of them with 100 to 4000 rows, times flat over
// rectangle, by how many workgroups fewer: under 128 1.02 to 1.17, 128 to 511 0.82 to 1.06, 512 and more 0.48 to 1.01 and
// one of 1.07 (60 users of 40 rows beside one of 200, 8 heads of 128; 1.006 with the attention behind it, where the others are 0.92 to 1.00).
// A launch of short runs leaves few out, and its whole sub-blocks would be kept in the L2 that the next kernel needs: eight calls of
// 64 to 512 users of 1 to 127 rows, with their attention, 1.00 to 1.04; stored past it, 0.99 to 1.00.
constexpr bool append_flat(int64_t longest_run, int64_t rectangle, int64_t flat) {
  return longest_run >= kBulkRun && rectangle - flat >= 512;
}

}  // namespace mts
