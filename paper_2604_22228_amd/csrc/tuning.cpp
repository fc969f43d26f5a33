// Tuned-table parsing and lookup (see tuning.hpp).
#include "tuning.hpp"

#include <algorithm>
#include <sstream>

namespace pcoll {

namespace {

int parse_dtype(const std::string& s) {
  if (s == "*") return -1;
  if (s == "i32") return 0;
  if (s == "f32") return 1;
  if (s == "bf16") return 2;
  if (s == "e4m3") return 3;
  if (s == "e5m2") return 4;
  if (s == "mxfp8") return 5;
  if (s == "bf16pair") return 6;
  return -2;
}

int parse_op(const std::string& s) {
  if (s == "*") return -1;
  if (s == "sum") return 0;
  if (s == "max") return 1;
  return -2;
}

bool parse_int_or_any(const std::string& s, int* v) {
  if (s == "*") {
    *v = -1;
    return true;
  }
  try {
    size_t used = 0;
    *v = std::stoi(s, &used);
    return used == s.size();
  } catch (...) {
    return false;
  }
}

bool match(int want, int have) { return want == -1 || want == have; }

}  // namespace

std::vector<TuneRow> parse_tune_table(const std::string& text) {
  std::vector<TuneRow> rows;
  std::istringstream in(text);
  std::string line;
  while (std::getline(in, line)) {
    auto hash = line.find('#');
    if (hash != std::string::npos) line.resize(hash);
    std::istringstream ls(line);
    std::string f[12];
    int nf = 0;
    while (nf < 12 && (ls >> f[nf])) ++nf;
    std::string extra;
    if (nf < 8 || (ls >> extra)) continue;
    TuneRow r;
    r.dtype = parse_dtype(f[0]);
    r.op = parse_op(f[1]);
    if (r.dtype == -2 || r.op == -2) continue;
    if (!parse_int_or_any(f[2], &r.ranks) || !parse_int_or_any(f[3], &r.graph))
      continue;
    if (!parse_int_or_any(f[4], &r.log2_lo) ||
        !parse_int_or_any(f[5], &r.log2_hi))
      continue;
    if (!parse_int_or_any(f[6], &r.tile_elems) ||
        !parse_int_or_any(f[7], &r.groups_per_cu))
      continue;
    if (nf >= 9 && (!parse_int_or_any(f[8], &r.interleave) ||
                    r.interleave < 0 || r.interleave > (1 << 20)))
      continue;
    if (nf >= 10 && (!parse_int_or_any(f[9], &r.group_waves) ||
                     r.group_waves < 1 || r.group_waves > 8))
      continue;
    if (nf >= 11 && (!parse_int_or_any(f[10], &r.publish_batch) ||
                     r.publish_batch < 1 || r.publish_batch > 64))
      continue;
    if (nf == 12 && (!parse_int_or_any(f[11], &r.unroll) ||
                     (r.unroll != 2 && r.unroll != 4)))
      continue;
    if (r.log2_lo < 0) r.log2_lo = 0;
    if (r.log2_hi < 0) r.log2_hi = 63;
    if (r.tile_elems <= 0 || r.tile_elems % 1024 != 0 || r.groups_per_cu <= 0)
      continue;
    rows.push_back(r);
  }
  return rows;
}

TuneChoice tune_lookup(const std::vector<TuneRow>& rows, int dtype, int op,
                       int ranks, int graph, uint64_t bytes_per_rank) {
  int lg = 0;
  while (lg < 63 && (bytes_per_rank >> (lg + 1)) != 0) ++lg;
  for (const auto& r : rows) {
    if (match(r.dtype, dtype) && match(r.op, op) && match(r.ranks, ranks) &&
        match(r.graph, graph) && lg >= r.log2_lo && lg <= r.log2_hi)
      return {r.tile_elems, r.groups_per_cu, r.interleave, r.group_waves,
              r.publish_batch, r.unroll, true};
  }
  // built-in default: 16 KiB of output per tile, two groups per CU
  // (element bytes: 2 for bf16 and bf16 pairs, 1 for the 8-bit floats)
  const int elem = dtype == 2 || dtype == 6 ? 2
                                            : (dtype >= 3 && dtype <= 5 ? 1 : 4);
  return {16384 / elem, 2, 0, 4, 16, 4};
}

// Rows are 1 KiB of each rank.  A tile costs its group about 4 us of
// latency, and all groups claim tiles from one counter, which gives out 60 a
// microsecond: tiles want many bytes, the more rows the fewer ranks.  Beyond
// that small tiles are better, since the tiles reduced at the same time then
// stay close together in every rank's memory and the last ones end together.
// Microseconds per epoch at 16 / 32 / 64 rows per tile:
//   fp32   1 rank  2^26 elements  264 / 126 /  97     4 ranks 2^26  305 / 232 / 224
//   fp32   2 ranks 2^26           273 / 149 / 138     3 ranks 2^25  132 /  96 / 102
//   fp32   8 ranks 2^24           106 / 109 / 118    16 ranks 2^22   63 /  65 /  66
//   bf16   2 ranks 2^27           273 / 148 / 137     4 ranks 2^26  141 / 116 / 125
//   bf16   8 ranks 2^24            65 /  67 /  68
//   e4m3   2 ranks 2^28           276 / 177 / 174     4 ranks 2^27  148 / 138 / 147
//   e4m3   8 ranks 2^26           134 / 141 / 138     8 ranks 2^23   36 /  35 /  44
// A message of fewer than 64 (8-bit: 128) such tiles gets smaller ones, down
// to a row per wavefront, so that it is read by more compute units at once:
// fp32, 8 ranks, 2^18 elements, 8 / 16 / 32 rows 17.1 / 16.2 / 19.0 us; e4m3,
// 8 ranks, 2^20, 4 / 8 / 16 / 32 rows 21.9 / 20.3 / 22.5 / 28.2 us.
//
// At 7 and 8 ranks a message of more than 256 and at most 512 tiles of 16 rows
// gets tiles of 32, one for each workgroup of the 256 compute units instead of
// two for some: a second tile costs its claim and a latency.  Kernel us at 16
// / 32 rows: fp32, 8 ranks, 4500 rows 18.1 / 17.4, 6000 20.0 / 19.0, 8192 23.1
// / 21.9, 9000 24.6 / 26.2; bf16 8192 23.2 / 22.6, bf16 pair 27.4 / 25.8.  (At
// 16 ranks fp32 6000 29.0 / 28.3 but 8192 33.6 / 34.2, bf16 37.4 / 38.9.)
//
// One group of 8 wavefronts per compute unit at every size (kernel us with one
// / two, fp32, 8 ranks: 2^20 elements 16.2 / 16.3, 2^21 22.4 / 25.0, 2^22 33.9
// / 38.8, 2^24 99 / 111; two of 4 wavefronts as two of 8), two where arithmetic
// must hide behind the loads of others (8-bit: e4m3 2 ranks 2^28 174 against
// 217 us, 8 ranks 2^26 138 / 126, 9 ranks 154 / 140).  From 10 ranks on (MX
// blocks: 9) the registers allow three wavefronts per SIMD or two, and the
// launch's residency cap leaves one group; three groups of 4 wavefronts in its
// place are slower, but for e4m3 at 10 to 13 ranks and 2^26 with tiles of half
// the rows (one of 8 / three of 4: 12 ranks 2^24 57 / 77 us, 2^26 192 / 181; MX
// 160 / 175).  Rows in flight per lane: as many as a wavefront has in a tile, at
// most 2 from 5 ranks on (6 ranks 2^26: 304 against 307 us).
TuneChoice shape_rule(int dtype, int ranks, uint64_t bytes_per_rank) {
  const bool bits8 = dtype >= 3 && dtype <= 5;
  const uint64_t rows = (bytes_per_rank + 1023) / 1024;
  uint64_t tile;
  if (bits8)
    tile = ranks <= 6 || rows <= 16384 ? 32 : 16;
  else
    tile = ranks <= 2 ? 64 : (ranks <= 6 ? 32 : 16);
  if (!bits8 && tile == 16 && ranks <= 8 && rows > 4096 && rows <= 8192)
    tile = 32;
  uint64_t fit = rows / (bits8 ? 128 : 64) / 8 * 8;
  if (fit < 8) fit = 8;
  if (tile > fit) tile = fit;
  const int row_elems = bits8 ? 1024 : (dtype == 2 || dtype == 6 ? 512 : 256);
  return {(int)tile * row_elems, bits8 ? 2 : 1, bits8 ? 0 : 8, 8, 64,
          ranks >= 5 && ranks <= 8 ? 2 : 4, false};
}

// Launch shape of the direct kernel: workgroups of 4 wavefronts, a row each
// per wavefront, two for 4-byte elements once the message has 4096 rows (512
// tiles, two per compute unit).  Small tiles spread a small message over the
// whole chip and keep its parallel streams close together; the hardware hands
// out the next one at no cost.  Measured at 8 ranks, 4 / 8 rows per tile: fp32
// 4 MiB per rank 8.8 / 8.0 us, 256 MiB 397 / 395 us; bf16 2 MiB 6.7 / 6.8 us,
// 128 MiB 189 / 196 us; e4m3 2^24 elements 32.3 / 32.6 us.  (The persistent
// kernel's tiles, 32 rows by 8 wavefronts: 9.7, 406, 8.4, 205, 32.2 us.)  Bands
// of 8 tiles: up to 2 % over consecutive rows from 64 MiB per rank on, no
// difference below.
//
// Large messages of many streams run best with two of these workgroups per
// compute unit, not the three to eight that the registers allow (bf16 and
// compensated sums to plain fp32 and int32): fewer places of each buffer are
// open in memory at once.  Reserving LDS that nothing uses keeps it at two;
// then 8 rows per tile and bands of 16.  Unreserved / two workgroups: fp32,
// 8 ranks, 256 MiB each 398 / 364 us (6.6 TB/s), 64 MiB 102 / 97 us, 4 ranks
// 128 MiB 112 / 103 us; 12 ranks 128 MiB 297 / 266 us; bf16, 8 ranks, 32 MiB
// 55 / 51 us; int32, 16 ranks, 16 MiB 55 / 52 us.  No gain below 128 MiB of
// inputs (fp32, 8 ranks, 16 MiB: 27.6 / 27.7 us), a loss with fewer streams
// (fp32, 1 rank, 128 MiB: 44 / 56 us) and for the 8-bit types, which need the
// wavefronts for their arithmetic (e4m3 110 / 135 us).
DirectShape direct_shape(int dtype, int ranks, uint64_t count, uint64_t span,
                         const DirectOverride& o) {
  const bool bits8 = dtype >= 3 && dtype <= 5;
  const uint64_t elem = bits8 ? 1 : (dtype == 2 || dtype == 6 ? 2 : 4);
  const uint64_t row_elems = 1024 / elem;
  const uint64_t rows = (count + row_elems - 1) / row_elems;
  const uint64_t spans = (count + span - 1) / span;
  const uint64_t span_rows = (span + row_elems - 1) / row_elems;
  DirectShape s{};
  s.waves = 4;
  if (!bits8 && ranks >= 4 && count * elem * (uint64_t)ranks >= (1ull << 27)) {
    s.tile_rows = 8;
    s.band = 16;
    s.lds = 64000;
  } else {
    s.tile_rows = elem == 4 && rows >= 4096 ? 8 : 4;
    s.band = 8;
  }
  // a shape of the caller's own takes no reserved LDS: how many of its
  // workgroups fit is the caller's choice too
  const bool waves = o.group_waves >= 1 && o.group_waves <= 8;
  if (waves) s.waves = o.group_waves;
  if (o.tile_elems > 0)
    s.tile_rows = (uint32_t)std::max<uint64_t>(
        1, (uint64_t)o.tile_elems / row_elems);
  if (o.groups > 0)
    s.tile_rows = (uint32_t)std::min(
        span_rows, std::max<uint64_t>(s.tile_rows,
                                      (rows + (uint64_t)o.groups - 1) /
                                          (uint64_t)o.groups));
  if (waves || o.tile_elems > 0 || o.groups > 0) s.lds = 0;
  for (;; s.tile_rows *= 2u) {
    s.span_tiles = (uint32_t)((span_rows + s.tile_rows - 1) / s.tile_rows);
    s.groups = spans * s.span_tiles;
    // a grid has fewer than 2^32 threads: larger tiles for what would need
    // more (64 GiB a rank in bf16 and the 8-bit types, 128 GiB in 4-byte
    // ones); one tile a span always fits
    if (s.groups * (64ull * (uint64_t)s.waves) < (1ull << 32)) break;
  }
  if (o.interleave >= 0 && o.interleave <= (1 << 20))
    s.band = o.interleave == 1 ? (uint32_t)std::min<uint64_t>(s.groups, 1u << 20)
                               : (uint32_t)o.interleave;
  return s;
}

}  // namespace pcoll
