// Compiles if the copies' size rules lie where they were measured.
#include "../../paper_2604_22881_amd/csrc/mts_copy_rules.hpp"

using mts::append_by_planes;
using mts::append_flat;
using mts::gather_past_caches;
using mts::scatter_past_caches;

using mts::RowsPast;
constexpr RowsPast none = RowsPast::kNone, read = RowsPast::kRead, both = RowsPast::kReadAndWritten;

// 12 histories of 5000 tokens, 4 heads of 128, 8 layers: 983 MB; in one launch per layer, 123 MB each
static_assert(scatter_past_caches(60000, 90000, 2048, 8) == both && scatter_past_caches(60000, 90000, 2048, 1) == none, "");
// many short runs of one long one's bound: the batch's pages bound them
static_assert(scatter_past_caches(1024 * 1024, 16384, 2048, 4) == none && scatter_past_caches(1024 * 1024, 0, 2048, 4) == both, "");
static_assert(scatter_past_caches(43007, 1 << 30, 2048, 4) == read && scatter_past_caches(43008, 1 << 30, 2048, 4) == both, "");
static_assert(scatter_past_caches(20479, 1 << 30, 2048, 4) == none && scatter_past_caches(20480, 1 << 30, 2048, 4) == read, "");
static_assert(!gather_past_caches(64) && gather_past_caches(128) && gather_past_caches(512), "");
static_assert(append_by_planes(256, 16384) && !append_by_planes(512, 16385), "");
static_assert(append_by_planes(128, 1024) && !append_by_planes(128, 1025) && !append_by_planes(64, 1), "");
static_assert(append_flat(128, 1024, 512) && !append_flat(128, 1024, 513) && !append_flat(4000, 100, 200), "");
static_assert(!append_flat(127, 1 << 20, 512), "short runs: their whole sub-blocks would be kept in the L2");
