// Tuned launch parameters, looked up per request.
//
// Section 4.4: an offline exhaustive search fixes the scheduling parameters
// per configuration, separately for graph and non-graph execution; the
// tuned values are defaults that environment variables override.  Here the
// search is done by the package's autotuner, which writes a text table:
//
//   # dtype op ranks graph log2_lo log2_hi tile groups_per_cu interleave waves batch unroll
//   f32     sum 8   0     24      28      4096   1             1          4     16    4
//
// dtype in {i32, f32, bf16, e4m3, e5m2, mxfp8,
// bf16pair, *}, op in {sum, max, *}, ranks a number
// or *, graph 0 / 1 / *, and [log2_lo, log2_hi] the range of
// floor(log2(bytes per rank of the whole request)); the trailing interleave
// (tile layout, default 0; 1 = bands of the launch's workgroups, n >= 2 =
// bands of n tiles), waves-per-workgroup (default 4), publish-batch (default
// 16) and unroll (rows in flight per lane, 2 or 4, default 4) columns may be
// omitted, from the right.  The first matching row wins.  Host-only C++17.
#pragma once
#include <cstdint>
#include <string>
#include <vector>

namespace pcoll {

struct TuneRow {
  int dtype = -1, op = -1, ranks = -1, graph = -1;  // -1 = any
  int log2_lo = 0, log2_hi = 63;
  int tile_elems = 0, groups_per_cu = 0, interleave = 0, group_waves = 4;
  int publish_batch = 16;
  int unroll = 4;
};

struct TuneChoice {
  int tile_elems;
  int groups_per_cu;
  int interleave;
  int group_waves;
  int publish_batch;
  int unroll;
  bool matched = false;  // a row of the table matched
};

// Parses a table; malformed lines are skipped.  Returns the rows.
std::vector<TuneRow> parse_tune_table(const std::string& text);

// First matching row, or (matched = false) a plain default, in whose place the
// runtime takes shape_rule.
TuneChoice tune_lookup(const std::vector<TuneRow>& rows, int dtype, int op,
                       int ranks, int graph, uint64_t bytes_per_rank);

// The launch shape where the table has no row: from the payload type, the
// ranks and the size alone.
TuneChoice shape_rule(int dtype, int ranks, uint64_t bytes_per_rank);

// Launch shape of the direct kernel: `groups` workgroups of `waves`
// wavefronts, one for each of the span_tiles tiles of tile_rows rows of every
// span; `band` the tile layout, `lds` reserved per workgroup and never used.
struct DirectShape {
  uint32_t tile_rows;
  uint32_t span_tiles;
  uint64_t groups;
  uint32_t band;
  int waves;
  unsigned lds;
};
// What a caller's environment sets of it; values out of range count as unset.
struct DirectOverride {
  int tile_elems = 0;   // > 0: elements per tile
  int groups = 0;       // > 0: no more workgroups than this (one per span)
  int interleave = -1;  // >= 0: the layout, as in a request's configuration
  int group_waves = 0;  // 1..8
};
DirectShape direct_shape(int dtype, int ranks, uint64_t count, uint64_t span,
                         const DirectOverride& o);

}  // namespace pcoll
