// Tile reducers: one wavefront reduces `n` consecutive elements of one
// bucket, starting at element `e0`, over the P rank contributions, in rank
// order 0..P-1 per element (the operation is elementwise, so any split into
// tiles gives the same result, which is why partitions may be reduced in
// any arrival order).
//
// Layout: every rank buffer and output is 16-byte aligned and every
// partition starts on a 128-byte line of its bucket (partition lengths are
// planned in whole lines; 256 elements for the 8-bit floats), so a row of a
// 128-byte aligned buffer covers whole lines.  Each lane streams 16-byte vectors
// (dwordx4), 64 lanes cover 1 KiB per rank per step, and U steps form one
// batch of U * P loads per lane.  Up to 16 loads the compiler mostly issues a
// batch before its first add; in larger ones it starts the first steps' adds
// while loads are still to come (most in flight: fp32, 8 ranks, U = 4 12 of
// 32; int32, 16 ranks, U = 2 10 of 32, U = 1 13 of 16; a single step of 4
// ranks 2 of 4).  A scheduling barrier that keeps every load first is slower
// (fp32, 8 ranks, 256 MiB each 375 -> 386 us, int32, 16 ranks, 64 MiB 188 ->
// 192 us).  Loads and stores carry the nontemporal hint: the data are touched
// once.  The ragged end (< 16 bytes) of a bucket is done element by element.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "layout.hpp"
#include "persistent.hpp"

namespace pcoll {
namespace dev {

// ------------------------------------------------------------ accumulators
// Float sum in binary32, plain or Sum2.  Non-finite values follow IEEE
// arithmetic; once the running sum is not finite the TwoSum errors are
// NaN, so the compensated result is the running sum itself (plain and
// compensated sums then agree).  FINITE: the inputs and sums are known to
// be finite (the 8-bit payloads), which spares that test.
template <bool COMP, bool FINITE = false>
struct FSum {
  float s, c;
  __device__ __forceinline__ void init(float v) { s = v; c = 0.0f; }
  __device__ __forceinline__ void add(float v) {
    if (COMP) {  // Sum2 (Ogita, Rump, Oishi 2005): carry the exact errors
      float e;
      two_sum(s, v, s, e);
      c = c + e;
    } else {
      s = s + v;
    }
  }
  __device__ __forceinline__ float get() const {
    if (!COMP) return s;
    if (FINITE) return s + c;
    return __builtin_isfinite(s) ? s + c : s;
  }
};

// Float max: the maximum operation of IEEE 754-2019 (NaN if any input is
// NaN, +0 above -0), one v_maximum3_f32 on gfx950.  It is commutative and
// associative, so the rank order does not change the result.
struct FMax {
  float m;
  __device__ __forceinline__ void init(float v) { m = v; }
  __device__ __forceinline__ void add(float v) {
    m = __builtin_elementwise_maximum(m, v);
  }
  __device__ __forceinline__ float get() const { return m; }
};

struct ISum {
  uint32_t s;  // two's-complement wrap
  __device__ __forceinline__ void init(uint32_t v) { s = v; }
  __device__ __forceinline__ void add(uint32_t v) { s = s + v; }
  __device__ __forceinline__ uint32_t get() const { return s; }
};

struct IMax {
  int32_t m;
  __device__ __forceinline__ void init(uint32_t v) { m = (int32_t)v; }
  __device__ __forceinline__ void add(uint32_t v) {
    m = (int32_t)v > m ? (int32_t)v : m;
  }
  __device__ __forceinline__ uint32_t get() const { return (uint32_t)m; }
};

// ------------------------------------------------------------------ codecs
// 32-bit words: the value is the word (float bits or int32).
struct Word32 {
  static constexpr int kPerVec = 4;
  static constexpr int kBytes = 4;
  using Val = uint32_t;
  __device__ __forceinline__ static uint32_t get(const uint4& v, int j) {
    return j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w));
  }
};

__device__ __forceinline__ float as_f(uint32_t u) { return __uint_as_float(u); }

// bfloat16 -> float is exact (the upper half of a binary32).
__device__ __forceinline__ float bf16_to_f(uint32_t h) {
  return __uint_as_float(h << 16);
}
// Two floats -> a word of two bfloat16 codes (a in the low half), round
// to nearest even (ties to the even code, subnormals kept, overflow to
// infinity) with gfx950's v_cvt_pk_bf16_f32; every NaN becomes the quiet
// NaN 0x7FC0 (sign and payload dropped) by converting the quiet NaN of
// binary32 with an empty payload in its place.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f_to_bf16x2(float a, float b) {
  const float qnan = __uint_as_float(0x7fc00000u);
  const f32x2_t v = {__builtin_isnan(a) ? qnan : a,
                     __builtin_isnan(b) ? qnan : b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ uint32_t f_to_bf16(float f) {
  return f_to_bf16x2(f, 0.0f) & 0xffffu;
}

// The two 8-bit formats: largest finite value (the block scale maps a
// block's amax onto it), the hardware decode of a code pair, and the encode
// of four values into one word (code j in byte j).  The gfx950 conversions
// round to nearest even, subnormals included, but do not saturate; values
// are clamped to +-kMax first, so that the encode saturates as the formats'
// definitions ask.
__device__ __forceinline__ float clamp_abs(float v, float m) {
  return __builtin_amdgcn_fmed3f(v, -m, m);
}

struct Fp8E4M3 {
  static constexpr float kMax = 448.0f;
  static constexpr float kQuantum = 0x1p-9f;  // every value is a multiple
  __device__ __forceinline__ static float dec(uint32_t w) {  // its low byte
    return __builtin_amdgcn_cvt_f32_fp8((int)w, 0);
  }
  // four values that round to at most kMax
  __device__ __forceinline__ static uint32_t enc4_small(float a, float b,
                                                        float c, float d) {
    const int w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
  }
  template <bool HI>
  __device__ __forceinline__ static auto dec_pair(uint32_t w) {
    return __builtin_amdgcn_cvt_pk_f32_fp8((int)w, HI);
  }
  __device__ __forceinline__ static uint32_t enc4(float a, float b, float c,
                                                  float d) {
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp_abs(a, kMax),
                                            clamp_abs(b, kMax), 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp_abs(c, kMax), clamp_abs(d, kMax),
                                        w, true);
    return (uint32_t)w;
  }
};
struct Fp8E5M2 {
  static constexpr float kMax = 57344.0f;
  static constexpr float kQuantum = 0x1p-16f;
  __device__ __forceinline__ static float dec(uint32_t w) {
    return __builtin_amdgcn_cvt_f32_bf8((int)w, 0);
  }
  __device__ __forceinline__ static uint32_t enc4_small(float a, float b,
                                                        float c, float d) {
    const int w = __builtin_amdgcn_cvt_pk_bf8_f32(a, b, 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(c, d, w, true);
  }
  template <bool HI>
  __device__ __forceinline__ static auto dec_pair(uint32_t w) {
    return __builtin_amdgcn_cvt_pk_f32_bf8((int)w, HI);
  }
  __device__ __forceinline__ static uint32_t enc4(float a, float b, float c,
                                                  float d) {
    int w = __builtin_amdgcn_cvt_pk_bf8_f32(clamp_abs(a, kMax),
                                            clamp_abs(b, kMax), 0, false);
    w = __builtin_amdgcn_cvt_pk_bf8_f32(clamp_abs(c, kMax), clamp_abs(d, kMax),
                                        w, true);
    return (uint32_t)w;
  }
};

// ---------------------------------------------------- 16-byte vector tiles
// Reduces one 16-byte vector per rank into one 16-byte output vector.
template <class Acc, int P, int Kind>
struct VecCombine;

// Kind 0: 32-bit float lanes; Kind 1: 32-bit int lanes; Kind 2: bf16 lanes.
template <class Acc, int P>
struct VecCombine<Acc, P, 0> {
  __device__ __forceinline__ static uint4 run(const uint4 (&x)[P]) {
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Acc a;
      a.init(as_f(Word32::get(x[0], j)));
#pragma unroll
      for (int r = 1; r < P; ++r) a.add(as_f(Word32::get(x[r], j)));
      o[j] = __float_as_uint(a.get());
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
  }
};

template <class Acc, int P>
struct VecCombine<Acc, P, 1> {
  __device__ __forceinline__ static uint4 run(const uint4 (&x)[P]) {
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Acc a;
      a.init(Word32::get(x[0], j));
#pragma unroll
      for (int r = 1; r < P; ++r) a.add(Word32::get(x[r], j));
      o[j] = a.get();
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
  }
};

template <class Acc, int P>
struct VecCombine<Acc, P, 2> {
  __device__ __forceinline__ static uint4 run(const uint4 (&x)[P]) {
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Acc lo, hi;
      uint32_t w = Word32::get(x[0], j);
      lo.init(bf16_to_f(w & 0xffffu));
      hi.init(bf16_to_f(w >> 16));
#pragma unroll
      for (int r = 1; r < P; ++r) {
        w = Word32::get(x[r], j);
        lo.add(bf16_to_f(w & 0xffffu));
        hi.add(bf16_to_f(w >> 16));
      }
      o[j] = f_to_bf16x2(lo.get(), hi.get());
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
  }
};

// bf16 pair output of a binary32 sum y: hi = bf16(y), lo = bf16(y - hi).
// The difference is exact in binary32 (hi is y rounded to fewer bits in
// the same binade), so hi + lo carries y to 16 significant bits.  When hi
// is not finite (y is NaN, infinite or beyond bf16's range), lo = +0, so
// that hi + lo is hi.
__device__ __forceinline__ uint32_t bf16_pair(float y, uint32_t& lo) {
  const uint32_t hi = f_to_bf16(y);
  lo = (hi & 0x7f80u) == 0x7f80u ? 0u : f_to_bf16(y - bf16_to_f(hi));
  return hi;
}

// Kind 3: bf16 lanes in, the pair (hi, lo) out: run() returns the hi
// vector and leaves the lo vector in `low`.
template <class Acc, int P>
struct VecCombine<Acc, P, 3> {
  __device__ __forceinline__ static uint4 run(const uint4 (&x)[P],
                                              uint4& low) {
    uint32_t o[4], l[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Acc a, b;
      uint32_t w = Word32::get(x[0], j);
      a.init(bf16_to_f(w & 0xffffu));
      b.init(bf16_to_f(w >> 16));
#pragma unroll
      for (int r = 1; r < P; ++r) {
        w = Word32::get(x[r], j);
        a.add(bf16_to_f(w & 0xffffu));
        b.add(bf16_to_f(w >> 16));
      }
      uint32_t la, lb;
      const uint32_t ha = bf16_pair(a.get(), la);
      const uint32_t hb = bf16_pair(b.get(), lb);
      o[j] = ha | (hb << 16);
      l[j] = la | (lb << 16);
    }
    low = make_uint4(l[0], l[1], l[2], l[3]);
    return make_uint4(o[0], o[1], o[2], o[3]);
  }
};

// Scalar path for the last (< 16 bytes) elements of a bucket.
template <class Acc, int P, int Kind>
__device__ __forceinline__ void combine_scalar(const char* const (&in)[P],
                                               char* out, char* out2,
                                               uint32_t i) {
  if constexpr (Kind == 3) {
    Acc a;
    a.init(bf16_to_f(reinterpret_cast<const uint16_t*>(in[0])[i]));
#pragma unroll
    for (int r = 1; r < P; ++r)
      a.add(bf16_to_f(reinterpret_cast<const uint16_t*>(in[r])[i]));
    uint32_t lo;
    st_out(reinterpret_cast<uint16_t*>(out) + i,
           (uint16_t)bf16_pair(a.get(), lo));
    st_out(reinterpret_cast<uint16_t*>(out2) + i, (uint16_t)lo);
  } else if constexpr (Kind == 2) {
    Acc a;
    a.init(bf16_to_f(reinterpret_cast<const uint16_t*>(in[0])[i]));
#pragma unroll
    for (int r = 1; r < P; ++r)
      a.add(bf16_to_f(reinterpret_cast<const uint16_t*>(in[r])[i]));
    st_out(reinterpret_cast<uint16_t*>(out) + i, (uint16_t)f_to_bf16(a.get()));
  } else if constexpr (Kind == 0) {
    Acc a;
    a.init(as_f(reinterpret_cast<const uint32_t*>(in[0])[i]));
#pragma unroll
    for (int r = 1; r < P; ++r)
      a.add(as_f(reinterpret_cast<const uint32_t*>(in[r])[i]));
    st_out(reinterpret_cast<uint32_t*>(out) + i, __float_as_uint(a.get()));
  } else {
    Acc a;
    a.init(reinterpret_cast<const uint32_t*>(in[0])[i]);
#pragma unroll
    for (int r = 1; r < P; ++r)
      a.add(reinterpret_cast<const uint32_t*>(in[r])[i]);
    st_out(reinterpret_cast<uint32_t*>(out) + i, a.get());
  }
}

// Rows of a lane's batch: enough loads in flight, bounded register use.  DEEP
// (the default) takes 4 rows up to 8 ranks and 2 above (at 16 ranks 1.4 %
// faster than 1, with no spills); the shallow form takes half of that from 3
// ranks on, which needs fewer registers and leaves more room for kernels that
// run beside the reduction.
template <int P, bool DEEP>
struct Unroll {
  static constexpr int value = P <= 2 ? 4 : (P <= 8 ? (DEEP ? 4 : 2) : (DEEP ? 2 : 1));
};

// Rows of a tile.  A partition is cut into rows of 64 lanes x 16 bytes
// (kRowElems elements) and into nt tiles of rpt = ceil(rows / nt) rows;
// tile lt takes rows base + k * stride, k = 0, 1, ...
//  * consecutive layout (band 0): rows [lt rpt, (lt + 1) rpt);
//  * banded interleave (band B > 0): tiles are grouped into bands of B
//    consecutive tiles, band b owning rows [b B rpt, (b B + nb) rpt) (nb =
//    its tile count, B but the last), and tile j of the band takes every
//    nb-th row of it starting at row j.  The tiles running at the same time
//    (consecutive claims) then stream side by side through one band, and
//    each tile's rows stay within B rpt rows, so a tile touches few pages
//    whatever the partition's size.
struct RowSet {
  uint32_t base, stride, limit;  // rows base + k * stride, k < limit
  // nrows: rows this set may use (whole rows); rpt: ceil(all rows of the
  // partition / nt)
  __device__ __forceinline__ RowSet(uint32_t lt, uint32_t nt, uint32_t rpt,
                                    uint32_t band, uint32_t nrows) {
    if (band) {
      const uint32_t b = lt / band, j = lt - b * band;
      const uint32_t nb = min(band, nt - b * band);
      const uint32_t b0 = b * band * rpt;
      const uint32_t b1 = min(b0 + nb * rpt, nrows);
      base = b0 + j;
      stride = nb;
      limit = base < b1 ? (b1 - 1 - base) / nb + 1 : 0;
    } else {
      const uint32_t rows_per_tile = rpt;
      base = lt * rows_per_tile;
      stride = 1;
      limit = base < nrows ? min(rows_per_tile, nrows - base) : 0;
    }
  }
  __device__ __forceinline__ uint32_t row(uint32_t k) const {
    return base + k * stride;
  }
};

// Whether tile lt owns row q < nt * rpt (used for the ragged end of a
// partition), in the layout of RowSet.
__device__ __forceinline__ bool owns_row(uint32_t q, uint32_t lt, uint32_t nt,
                                         uint32_t rpt, uint32_t band) {
  if (!band) return q / rpt == lt;
  const uint64_t span = (uint64_t)band * rpt;  // rows of a full band
  const uint32_t b = (uint32_t)(q / span);
  const uint32_t nb = min(band, nt - b * band);
  return b * band + (uint32_t)(q - b * span) % nb == lt;
}

template <class Acc, int Kind, bool DEEP = true>
struct VecTile {
  static constexpr int kElemBytes = Kind >= 2 ? 2 : 4;
  static constexpr int kPerVec = 16 / kElemBytes;
  static constexpr uint32_t kRowElems = 64 * kPerVec;
  template <int P, bool DIRECT>
  static constexpr int waves() { return 2; }

  // Reduces wavefront `wave`'s rows of the tile: rows k = wave, wave +
  // nwaves, ... of the tile's row set; wavefront 0 also does the
  // partition's ragged end if this tile owns it.
  template <int P, class Bucket>
  __device__ __forceinline__ static void run(Bucket bd,
                                             uint64_t poff, uint64_t plen,
                                             uint32_t lt, uint32_t nt,
                                             uint32_t inter, uint32_t wave,
                                             uint32_t nwaves) {
    const uint32_t lane = lane_id();
    const uint4* in[P];
#pragma unroll
    for (int r = 0; r < P; ++r)
      in[r] = reinterpret_cast<const uint4*>(
          static_cast<const char*>(bd->in[r]) + poff * kElemBytes);
    uint4* out = reinterpret_cast<uint4*>(static_cast<char*>(bd->out) +
                                          poff * kElemBytes);
    // Kind 3: the low halves of the pairs go to the second output
    uint4* out2 = Kind == 3 ? reinterpret_cast<uint4*>(
                                  static_cast<char*>(bd->out_scale) +
                                  poff * kElemBytes)
                            : nullptr;
    // row q: each rank's 1 KiB at a wave-uniform address, 16 bytes a lane
    auto fetch = [&](uint32_t q, uint4(&xx)[P]) {
#pragma unroll
      for (int r = 0; r < P; ++r) xx[r] = ld_stream(in[r] + (size_t)q * 64u + lane);
    };
    auto emit = [&](uint32_t q, const uint4(&xx)[P]) {
      if constexpr (Kind == 3) {
        uint4 low;
        st_row(out + (size_t)q * 64u, lane, VecCombine<Acc, P, 3>::run(xx, low));
        st_row(out2 + (size_t)q * 64u, lane, low);
      } else {
        st_row(out + (size_t)q * 64u, lane, VecCombine<Acc, P, Kind>::run(xx));
      }
    };
    const uint32_t nv = (uint32_t)(plen / kPerVec);  // whole vectors
    const uint32_t full = nv / 64;                    // whole rows
    const uint32_t all = (uint32_t)((plen + kRowElems - 1) / kRowElems);
    const uint32_t rpt = (all + nt - 1) / nt;
    const RowSet rows(lt, nt, rpt, inter, full);
    // bf16 max holds more temporaries per value than the sums (the NaN
    // handling of IEEE maximum): at 4 rows in flight it would spill
    constexpr int U0 = Unroll<P, DEEP>::value;
    constexpr bool kBf16Max = Kind == 2 && std::is_same<Acc, FMax>::value;
    constexpr int U = kBf16Max && U0 > 2 ? 2 : U0;
    // U rows at a time, then U / 2, then one: whatever is left of a tile is
    // loaded in batches as large as it allows
    uint32_t k = wave;
    auto batch = [&](auto depth) {
      constexpr int D = decltype(depth)::value;
      for (; k + (D - 1) * nwaves < rows.limit; k += D * nwaves) {
        uint4 x[D][P];
#pragma unroll
        for (int u = 0; u < D; ++u) fetch(rows.row(k + u * nwaves), x[u]);
#pragma unroll
        for (int u = 0; u < D; ++u) emit(rows.row(k + u * nwaves), x[u]);
      }
    };
    batch(std::integral_constant<int, U>{});
    if constexpr (U > 2) batch(std::integral_constant<int, U / 2>{});
    if constexpr (U > 1) batch(std::integral_constant<int, 1>{});
    // the partition's ragged end: a partial row and the last < 16 bytes,
    // done by the tile that owns row `full`
    if (wave != 0 || full >= all || !owns_row(full, lt, nt, rpt, inter))
      return;
    if (full * 64u + lane < nv) {
      uint4 x[P];
      fetch(full, x);
      emit(full, x);
    }
    const uint32_t tail = (uint32_t)(plen - (uint64_t)nv * kPerVec);
    if (lane < tail) {
      const char* inb[P];
#pragma unroll
      for (int r = 0; r < P; ++r) inb[r] = reinterpret_cast<const char*>(in[r]);
      combine_scalar<Acc, P, Kind>(inb, reinterpret_cast<char*>(out),
                                   reinterpret_cast<char*>(out2),
                                   nv * kPerVec + lane);
    }
  }
};

// ------------------------------------------------------ 8-bit float tiles
// Each lane owns 16 consecutive codes; a row of 16 lanes owns one block of
// 256 elements and its scale.  Inputs: y = sum_r fl(dec(q_r) * s_r) in
// binary32 (plain or Sum2), then per block amax = max |y|, s = fl(amax /
// max) (max = 448 for e4m3, 57344 for e5m2; s = 1 if that is not a normal
// number), codes enc(fl(y * fl(1/s))).
// Tiles start on block boundaries (tile and partition lengths are multiples
// of 256); only a bucket's last block can be short.
// One word's four values times the block scale (one multiply each, or one
// fused with + 0).
template <class Fmt, bool PLUS0 = false>
__device__ __forceinline__ void dec4(uint32_t w, float scale, float (&o)[4]) {
  auto lo = Fmt::template dec_pair<false>(w);
  auto hi = Fmt::template dec_pair<true>(w);
  const float v[4] = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
  for (int j = 0; j < 4; ++j)
    o[j] = PLUS0 ? __builtin_fmaf(v[j], scale, 0.0f) : v[j] * scale;
}

// Rank-order sum of word k of every rank's codes, plain or Sum2.  dec(word,
// rank, values) decodes one rank's word.  AGAIN: the rarely taken branch of
// a caller that has decoded the same words the same way already; the empty
// asm keeps the compiler from holding those values in registers for it.
template <bool COMP, bool AGAIN, int P, class Dec>
__device__ __forceinline__ void sum_word(const uint4 (&raw)[P], int k,
                                         Dec&& dec, float (&y)[4]) {
  FSum<COMP, true> acc[4];
#pragma unroll
  for (int r = 0; r < P; ++r) {
    float d[4];
    uint32_t w = Word32::get(raw[r], k);
    if (AGAIN) asm("" : "+v"(w));
    dec(w, r, d);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (r == 0)
        acc[j].init(d[j]);
      else
        acc[j].add(d[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) y[j] = acc[j].get();
}

// Max over the 16 lanes of a block: rotations within a DPP row (through LDS
// shuffles each step waits for a round trip: direct kernel, e4m3, 3 ranks, 2^26
// values, 70 against 66 us).
__device__ __forceinline__ float row16_max(float v) {
  const auto step = [&](auto ctrl) {
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(
                     __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf,
                     false)));
  };
  step(std::integral_constant<int, 0x128>{});  // row_ror:8
  step(std::integral_constant<int, 0x124>{});
  step(std::integral_constant<int, 0x122>{});
  step(std::integral_constant<int, 0x121>{});
  return v;
}

// Sum2's result of value i (0..15) of the lane.
template <class Fmt, int P>
__device__ __forceinline__ float sum2_at(const uint4 (&raw)[P],
                                         const float (&s_in)[P], uint32_t i) {
  FSum<true, true> acc;
#pragma unroll
  for (int r = 0; r < P; ++r) {
    const uint32_t lo = __builtin_amdgcn_perm(raw[r].y, raw[r].x, i & 7u);
    const uint32_t hi = __builtin_amdgcn_perm(raw[r].w, raw[r].z, i & 7u);
    const float d = Fmt::dec(i < 8u ? lo : hi) * s_in[r];
    if (r == 0)
      acc.init(d);
    else
      acc.add(d);
  }
  return acc.get();
}

// The compensated row of the 8-bit formats from plain sums, from 3 ranks on
// (below, Sum2 has at most one addition to compensate).
//
// Sum2 in binary32 costs seven dependent operations per rank and value.  But
// the row's outputs are 8-bit codes and one scale per block, and few of them
// depend on the correction.  Sum2 returns fl(s + c) with s the plain sum and
// c the sum of its rounding errors, each at most u |s_r| (u = 2^-24, s_r the
// partial sums): |c| <= E M with M the largest |s_r| and E = u (P - 1), and a
// little for c's own rounding.  Every step from s to a code is monotonic, so
//   * the codes of fl(s - E M) and fl(s + E M), where equal, are the code;
//   * the scale needs the exact largest magnitude: each lane takes Sum2 of
//     the largest of its 16 plain sums, and these settle the block's amax if
//     no lane's second largest can exceed it;
//   * the values whose two codes differ (about 1 in 30,000 of gradient-like
//     data) take Sum2 one by one.
// Returns false where this settles nothing, and the whole row takes Sum2:
// infinities or NaN, near ties for the largest in one lane, many open codes.
//
// Where all scales of a lane are powers of two, its sums are multiples of
// the smallest scale times the format's quantum and often lie halfway between
// two codes; below 2^24 such multiples they are exact (E = 0).  e5m2 codes
// span too much for that: such rows take Sum2 at once.
//
// Bound: VALU issue (686 instructions a row at 8 ranks, 0.78 per CU and cycle)
// beside the memory streams.  e4m3, 128 buckets, 2^30 values, 8 ranks: 1.90 ms
// with Sum2 for every value, 1.60 ms this way (5.5 TB/s); one message of 2^25
// values, 16 ranks, 144 us (binary64 sums, which these kernels must not use,
// 160).  With 3 ranks it costs what Sum2 does (2^26 values, direct kernel 64 /
// 68 us), with 4 less (74 / 84).  A ragged last row in the direct kernel, 16
// ranks: Sum2 6.8, this way 5.7 us.  Rows that end in Sum2 pay for both: every
// value equal, 8 ranks, 80 -> 122 us.  The row's sums are kept for the codes, so
// registers decide the occupancy: a word at a time, the codes through ld_row
// (141 -> 120 VGPRs, four wavefronts per SIMD).
template <class Fmt, int P>
__device__ __forceinline__ bool row_from_plain(const uint4 (&raw)[P],
                                               const float (&s_in)[P],
                                               uint32_t (&w)[4], float& so) {
  uint32_t mant = 0u;
#pragma unroll
  for (int r = 0; r < P; ++r) mant |= __float_as_uint(s_in[r]);
  const bool pow2 = (mant & 0x7fffffu) == 0u;
  if constexpr (Fmt::kQuantum < 0x1p-9f) {
    if (__builtin_expect(__ballot(pow2) != 0, 0)) {
      uint32_t any = 0u;  // blocks of zeros have equal scales
#pragma unroll
      for (int r = 0; r < P; ++r)
        any |= (raw[r].x | raw[r].y | raw[r].z | raw[r].w) & 0x7f7f7f7fu;
      if (__ballot(pow2 && any != 0u) != 0) return false;
    }
  }
  float y[16], M[16];
  uint32_t m1 = 0u, m2 = 0u;  // the largest |y|, the index in the low bits,
                              // and the second largest
  float mx = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int r = 0; r < P; ++r) {
      float d[4];
      if (r == 0)
        // + 0 turns a sum of nothing but -0 into Sum2's +0
        dec4<Fmt, true>(Word32::get(raw[r], k), s_in[r], d);
      else
        dec4<Fmt>(Word32::get(raw[r], k), s_in[r], d);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = 4 * k + j;
        y[i] = r == 0 ? d[j] : y[i] + d[j];
        if (r > 0) M[i] = r == 1 ? fabsf(y[i]) : fmaxf(M[i], fabsf(y[i]));
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = 4 * k + j;
      const uint32_t x = (__float_as_uint(y[i]) & 0x7ffffff0u) | (uint32_t)i;
      m2 = max(min(m1, m2), min(max(m1, m2), x));  // the median
      m1 = max(m1, x);
      mx = fmaxf(mx, M[i]);
    }
    // one word at a time: the other words' terms would only hold registers
    __builtin_amdgcn_sched_barrier(0);
  }
  constexpr float kE = (float)(P - 1) * 0x1.0002p-24f;
  constexpr float kExact = 0x1p24f * Fmt::kQuantum;
  float E = kE;
  if (__ballot(pow2) != 0) {
    uint32_t least = ~0u;  // the smallest scale's bits, twice, less 1: zeros
                           // come last
#pragma unroll
    for (int r = 0; r < P; ++r)
      least = min(least, (__float_as_uint(s_in[r]) << 1) - 1u);
    if (pow2 && mx < __uint_as_float((least + 1u) >> 1) * kExact) E = 0.0f;
  }
  const float amax = row16_max(fabsf(sum2_at<Fmt>(raw, s_in, m1 & 15u)));
  // below 2^-118 the scale is 1 whatever amax is
  const float second = __builtin_fmaf(mx, E, __uint_as_float(m2 | 15u));
  const bool ok = m1 < 0x7f800000u && amax < __builtin_inff() &&
                  second <= fmaxf(amax, 0x1p-118f);
  if (__builtin_expect(__ballot(!ok) != 0, 0)) return false;
  so = amax / Fmt::kMax;
  if (!(so >= 0x1p-126f)) so = 1.0f;
  const float inv = 1.0f / so;
  // |y| * inv is at most kMax and a few of its ulps, so nothing saturates
  uint32_t open = 0u, lo[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float a[4], b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = 4 * k + j;
      a[j] = __builtin_fmaf(M[i], -E, y[i]) * inv;
      b[j] = __builtin_fmaf(M[i], E, y[i]) * inv;
    }
    lo[k] = Fmt::enc4_small(a[0], a[1], a[2], a[3]);
    w[k] = Fmt::enc4_small(b[0], b[1], b[2], b[3]);
    open |= lo[k] ^ w[k];
    __builtin_amdgcn_sched_barrier(0);
  }
  if (__builtin_expect(__ballot(open != 0u) == 0, 1)) return true;
  uint32_t todo = 0u;  // a bit for each open value
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (((lo[i / 4] ^ w[i / 4]) >> (8 * (i % 4)) & 0xffu) != 0u)
      todo |= 1u << i;
  if (__ballot(__popc(todo) > 2) != 0) return false;
  while (__ballot(todo != 0u) != 0) {
    const uint32_t i = todo ? (uint32_t)__ffs((int)todo) - 1u : 0u;
    const float v = sum2_at<Fmt>(raw, s_in, i) * inv;
    const uint32_t code = Fmt::enc4_small(v, 0.0f, 0.0f, 0.0f) & 0xffu;
    const uint32_t at = 8u * (i & 3u);
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
      if (todo && i / 4u == k) w[k] = (w[k] & ~(0xffu << at)) | (code << at);
    todo &= todo - 1u;
  }
  return true;
}

__device__ __forceinline__ uint4 load_codes(const uint8_t* p, uint32_t have) {
  if (have >= 16u) return ld_stream(reinterpret_cast<const uint4*>(p));
  uint32_t w[4] = {0u, 0u, 0u, 0u};
  for (uint32_t j = 0; j < have; ++j) w[j >> 2] |= (uint32_t)p[j] << (8 * (j & 3));
  return make_uint4(w[0], w[1], w[2], w[3]);
}

template <bool COMP, class Fmt>
struct Fp8Tile {
  static constexpr uint32_t kRowElems = 1024;  // 64 lanes x 16 codes
  // Wavefronts per SIMD that the registers are kept to, without spills: the
  // loads of others hide behind a row's arithmetic (8 ranks, 2^26 values,
  // direct kernel, four instead of five 117 -> 122 us).
  template <int P, bool DIRECT>
  static constexpr int waves() {
    if (!COMP || P < 3) return 2;
    if (DIRECT)
      return P == 3 ? 7 : (P <= 5 ? 6 : (P <= 8 ? 5 : (P <= 12 ? 4 : 3)));
    return P <= 9 ? 4 : 3;
  }

  // Row q: lane l owns codes el .. el + 16 of block blk.  FULL: the
  // whole row is inside the bucket (every lane has 16 codes), which spares
  // the per-lane length checks; otherwise `have` codes (0..16).
  template <int P, bool FULL>
  __device__ __forceinline__ static void row(const uint8_t* const (&in)[P],
                                             const float* const (&sc)[P],
                                             uint8_t* out, float* osc,
                                             uint32_t q, uint32_t have) {
    const uint32_t el = q * kRowElems + lane_id() * 16u;
    const uint32_t blk = el / 256u;
    uint4 raw[P];
    float s_in[P];
#pragma unroll
    for (int r = 0; r < P; ++r) {
      if (FULL) {
        raw[r] = ld_row(in[r] + (size_t)q * kRowElems, lane_id());
        s_in[r] = sc[r][blk];
      } else {
        raw[r] = have ? load_codes(in[r] + el, have) : make_uint4(0, 0, 0, 0);
        s_in[r] = have ? sc[r][blk] : 0.0f;
      }
    }
    // every rank's codes and scale are requested before the first is used,
    // so that one memory latency covers the row
    if (FULL) __builtin_amdgcn_sched_barrier(0);
    const auto dec = [&](uint32_t w, int r, float(&d)[4]) {
      dec4<Fmt>(w, s_in[r], d);
    };
    uint32_t w[4];
    float so;
    bool done = false;
    // codes past the end are zeros, which change no sum and no maximum
    if constexpr (COMP && P >= 3)
      done = row_from_plain<Fmt>(raw, s_in, w, so);
    if (!done) {
      float y[16];
      float amax = 0.0f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float v[4];
        sum_word<COMP, COMP && P >= 3>(raw, k, dec, v);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          y[4 * k + j] = v[j];
          if (FULL || (uint32_t)(4 * k + j) < have)
            amax = fmaxf(amax, fabsf(v[j]));
        }
      }
      amax = row16_max(amax);
      so = amax / Fmt::kMax;
      if (!(so >= 0x1p-126f)) so = 1.0f;
      const float inv = 1.0f / so;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        w[k] = Fmt::enc4(y[4 * k] * inv, y[4 * k + 1] * inv,
                         y[4 * k + 2] * inv, y[4 * k + 3] * inv);
    }
    if (FULL || have == 16u) {
      st_row(out + (size_t)q * kRowElems, lane_id(),
             make_uint4(w[0], w[1], w[2], w[3]));
    } else if (have) {
      for (uint32_t j = 0; j < have; ++j)
        st_out(out + el + j, (uint8_t)(w[j >> 2] >> (8 * (j & 3))));
    }
    if ((FULL || have) && (lane_id() & 15u) == 0u) st_out(osc + blk, so);
  }

  template <int P, class Bucket>
  __device__ __forceinline__ static void run(Bucket bd,
                                             uint64_t poff, uint64_t plen,
                                             uint32_t lt, uint32_t nt,
                                             uint32_t inter, uint32_t wave,
                                             uint32_t nwaves) {
    const uint32_t lane = lane_id();
    const uint8_t* in[P];
    const float* sc[P];
#pragma unroll
    for (int r = 0; r < P; ++r) {
      in[r] = static_cast<const uint8_t*>(bd->in[r]) + poff;
      sc[r] = static_cast<const float*>(bd->in_scale[r]) + poff / 256u;
    }
    uint8_t* out = static_cast<uint8_t*>(bd->out) + poff;
    float* osc = static_cast<float*>(bd->out_scale) + poff / 256u;
    const uint32_t n = (uint32_t)plen;
    const uint32_t nrows = (n + kRowElems - 1) / kRowElems;
    const RowSet rows(lt, nt, (nrows + nt - 1) / nt, inter, nrows);
    for (uint32_t k = wave; k < rows.limit; k += nwaves) {
      const uint32_t q = rows.row(k);
      if ((q + 1u) * kRowElems <= n) {  // uniform: the row is whole
        row<P, true>(in, sc, out, osc, q, 16u);
      } else {
        const uint32_t el = q * kRowElems + lane * 16u;
        const uint32_t have = el < n ? (n - el < 16u ? n - el : 16u) : 0u;
        row<P, false>(in, sc, out, osc, q, have);
      }
    }
  }
};

template <bool COMP>
using E4M3Tile = Fp8Tile<COMP, Fp8E4M3>;
template <bool COMP>
using E5M2Tile = Fp8Tile<COMP, Fp8E5M2>;

// ------------------------------------------------------------- MX blocks
// OCP MX blocks with e4m3 elements: 32 codes share one E8M0 scale byte b,
// the value of a code being dec(q) * 2^(b - 127) (exact in binary32).  The
// gfx950 scaled conversions take such a scale as a binary32 operand whose
// exponent field is b: v_cvt_scalef32_pk_f32_fp8 multiplies a decoded pair
// by 2^(b - 127), v_cvt_scalef32_pk_fp8_f32 divides a pair by it and rounds
// to nearest even (without saturating).
typedef float mx_f32x2 __attribute__((ext_vector_type(2)));
typedef short mx_i16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float e8m0_operand(uint32_t b) {
  return __uint_as_float(b << 23);
}

// Scale byte of a block whose largest magnitude is amax: e + 127 for the
// smallest e >= -127 with amax <= 448 * 2^e = 1.75 * 2^(e + 8).  For
// amax = f * 2^E (f in [1, 2)) that is e = E - 8 when f <= 1.75 (fraction
// field <= 0x600000), else E - 7; zero and subnormal amax (E < -126) give
// -127.  The codes of the block then never exceed 448 in magnitude.
__device__ __forceinline__ uint32_t mx_scale_byte(float amax) {
  const uint32_t u = __float_as_uint(amax);
  const int e = (int)(u >> 23) - 135 + ((u & 0x7fffffu) > 0x600000u ? 1 : 0);
  return u < 0x00800000u ? 0u : (uint32_t)(max(e, -127) + 127);
}

// A word's four codes scaled by the operand of byte b.
__device__ __forceinline__ void mx_dec4(uint32_t w, float scale,
                                        float (&o)[4]) {
  const mx_f32x2 lo =
      __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w, scale, false);
  const mx_f32x2 hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w, scale, true);
  o[0] = lo[0];
  o[1] = lo[1];
  o[2] = hi[0];
  o[3] = hi[1];
}

// Terms of at most 448, counted in their smallest scale's quantum 2^-9, add up
// below 2^31 if the ranks' scales, relative to the smallest, add up to this at
// most; so do P ranks' with scale bytes mx_spread(P) apart.
constexpr uint32_t kMxUnits = ((1u << 31) - 1u) / (448u * 512u);
constexpr uint32_t mx_spread(int P) {
  uint32_t d = 0;
  while (((uint32_t)P << (d + 1)) <= kMxUnits) ++d;
  return d;
}

// Whether any byte of w is a NaN code, in bit 7 of each byte, or-ed to acc:
// adding 1 to a byte changes its sign bit only if the other bits are set (a
// carry out of a byte comes from a NaN there).
__device__ __forceinline__ uint32_t mx_nan(uint32_t acc, uint32_t w) {
  return __builtin_amdgcn_bitop3_b32(acc, w + 0x01010101u, w,
                                     0xf0 | (0xcc ^ 0xaa));
}

// Codes of y[0..16) / 2^(b - 127), four per word (code j in byte j).
__device__ __forceinline__ uint4 mx_enc16(const float (&y)[16], float scale) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    mx_i16x2 t = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(
        mx_i16x2{0, 0}, y[4 * k], y[4 * k + 1], scale, false);
    t = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(t, y[4 * k + 2],
                                                 y[4 * k + 3], scale, true);
    w[k] = __builtin_bit_cast(uint32_t, t);
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// 4 codes (a dword, first value in the low byte) scaled by the operand.
__device__ __forceinline__ uint32_t mx_enc4(const float (&y)[4], float scale) {
  mx_i16x2 t = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(mx_i16x2{0, 0}, y[0],
                                                        y[1], scale, false);
  t = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(t, y[2], y[3], scale, true);
  return __builtin_bit_cast(uint32_t, t);
}

// Largest magnitude over a pair of lanes (2j, 2j + 1): one block.
__device__ __forceinline__ float pair_max(float v) {
  const int o = __builtin_amdgcn_mov_dpp(__float_as_int(v), 0xb1, 0xf, 0xf,
                                         false);  // quad_perm [1, 0, 3, 2]
  return fmaxf(v, __int_as_float(o));
}

// Each lane owns 16 consecutive codes, half of a block; lanes 2j and 2j + 1
// of a row share block j and its scale byte.  y = sum_r dec(q_r) *
// 2^(b_r - 127) in binary32 (plain or Sum2), per block the scale byte of
// max |y| (mx_scale_byte), codes RNE(y / 2^(b - 127)).  Partitions start on
// block boundaries (their lengths are multiples of 32); only a bucket's
// last block can be short.
template <bool COMP>
struct MxTile {
  static constexpr uint32_t kRowElems = 1024;  // 64 lanes x 16 codes
  template <int P, bool DIRECT>
  static constexpr int waves() { return 2; }

  template <int P, bool FULL>
  __device__ __forceinline__ static void row(const uint8_t* const (&in)[P],
                                             const uint8_t* const (&sc)[P],
                                             uint8_t* out, uint8_t* osc,
                                             uint32_t q, uint32_t have) {
    const uint32_t el = q * kRowElems + lane_id() * 16u;
    const uint32_t blk = el / 32u;
    uint4 raw[P];
    uint32_t b_in[P];
#pragma unroll
    for (int r = 0; r < P; ++r) {
      if (FULL) {
        raw[r] = ld_stream(reinterpret_cast<const uint4*>(
                               in[r] + (size_t)q * kRowElems) + lane_id());
        b_in[r] = sc[r][blk];
      } else {
        raw[r] = have ? load_codes(in[r] + el, have) : make_uint4(0, 0, 0, 0);
        b_in[r] = have ? sc[r][blk] : 0u;
      }
    }
    if (FULL) __builtin_amdgcn_sched_barrier(0);
    uint32_t base = 0u;  // of the scale bytes in b_in
    const auto dec = [&](uint32_t w, int r, float(&d)[4]) {
      mx_dec4(w, e8m0_operand(b_in[r] + base), d);
    };
    float y[16];
    float amax = 0.0f;
    // From 3 ranks on the compensated sum goes through integers.  Every term
    // is a multiple of g = 2^-9 2^(bmin - 127), of 4 significant bits and at
    // most 448 * 2^(bmax - 127), so for bmax - bmin <= 23 and up to 16 ranks
    // Sum2's errors add up to at most 135 u 448 2^(bmax - 127) <= 2^24 g: its
    // correction is exact and its result the exact sum rounded once; and for
    // scales close enough (8 ranks: 2^10) the sum in units of g fits 32 bits.
    // Above byte 240 a partial sum could leave binary32's range.  Other rows,
    // and those with NaN codes, take Sum2.  32 buckets, 2^28 values, 8 ranks:
    // 0.61 ms with Sum2, 0.53 this way (5.7 TB/s); scales 2^20 apart, 2^25
    // values, 89 against 77 us.
    bool sum2 = COMP;
    if constexpr (COMP && P >= 3) {
      uint32_t bmin = b_in[0], bmax = b_in[0], nan = 0u;
#pragma unroll
      for (int r = 1; r < P; ++r) {
        bmin = min(bmin, b_in[r]);
        bmax = max(bmax, b_in[r]);
      }
#pragma unroll
      for (int r = 0; r < P; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k) nan = mx_nan(nan, Word32::get(raw[r], k));
      bool exact = bmax <= 240u && bmax - bmin <= mx_spread(P);
      if (__ballot(!exact) != 0) {
        // all-zero blocks carry byte 0: their scale does not count
        const uint32_t none = 256u;
        bmin = 255u;
        bmax = 0u;
#pragma unroll
        for (int r = 0; r < P; ++r) {
          const bool zero = ((raw[r].x | raw[r].y | raw[r].z | raw[r].w) &
                             0x7f7f7f7fu) == 0u && b_in[r] != 255u;
          if (zero) b_in[r] = none;
          bmin = min(bmin, b_in[r]);
          bmax = max(bmax, zero ? 0u : b_in[r]);
        }
        if (bmin > bmax) bmin = bmax = 127u;
        // and the other ranks may lie further apart the fewer are far up
        uint32_t sum = 0u;
#pragma unroll
        for (int r = 0; r < P; ++r) {
          if (b_in[r] == none) b_in[r] = bmin;
          sum += 1u << min(b_in[r] - bmin, 14u);
        }
        exact = bmax <= 240u && sum <= kMxUnits;
      }
      // from here on relative to the smallest, times 2^9
      base = bmin - 136u;
#pragma unroll
      for (int r = 0; r < P; ++r) b_in[r] -= base;
      sum2 = __ballot(!exact || (nan & 0x80808080u) != 0u) != 0;
      if (!sum2) {
        // 2^(bmin - 136), which may be subnormal
        const float unit = __builtin_ldexpf(1.0f, (int)bmin - 136);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          int n[4];
#pragma unroll
          for (int r = 0; r < P; ++r) {
            float d[4];
            mx_dec4(Word32::get(raw[r], k), e8m0_operand(b_in[r]), d);
#pragma unroll
            for (int j = 0; j < 4; ++j)
              n[j] = r == 0 ? (int)d[j] : n[j] + (int)d[j];
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) y[4 * k + j] = (float)n[j] * unit;
          // one word at a time: the other words' terms would only hold
          // registers
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (!(COMP && P >= 3) || sum2) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float v[4];
        sum_word<COMP, false>(raw, k, dec, v);
#pragma unroll
        for (int j = 0; j < 4; ++j) y[4 * k + j] = v[j];
        if (COMP) __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (FULL || (uint32_t)j < have) amax = fmaxf(amax, fabsf(y[j]));
    amax = pair_max(amax);
    const uint32_t b = mx_scale_byte(amax);
    const uint4 codes = mx_enc16(y, e8m0_operand(b));
    if (FULL || have == 16u) {
      st_row(out + (size_t)q * kRowElems, lane_id(), codes);
    } else if (have) {
      const uint32_t w[4] = {codes.x, codes.y, codes.z, codes.w};
      for (uint32_t j = 0; j < have; ++j)
        st_out(out + el + j, (uint8_t)(w[j >> 2] >> (8 * (j & 3))));
    }
    if ((FULL || have) && (lane_id() & 1u) == 0u) st_out(osc + blk, (uint8_t)b);
  }

  template <int P, class Bucket>
  __device__ __forceinline__ static void run(Bucket bd,
                                             uint64_t poff, uint64_t plen,
                                             uint32_t lt, uint32_t nt,
                                             uint32_t inter, uint32_t wave,
                                             uint32_t nwaves) {
    const uint32_t lane = lane_id();
    const uint8_t* in[P];
    const uint8_t* sc[P];
#pragma unroll
    for (int r = 0; r < P; ++r) {
      in[r] = static_cast<const uint8_t*>(bd->in[r]) + poff;
      sc[r] = static_cast<const uint8_t*>(bd->in_scale[r]) + poff / 32u;
    }
    uint8_t* out = static_cast<uint8_t*>(bd->out) + poff;
    uint8_t* osc = static_cast<uint8_t*>(bd->out_scale) + poff / 32u;
    const uint32_t n = (uint32_t)plen;
    const uint32_t nrows = (n + kRowElems - 1) / kRowElems;
    const RowSet rows(lt, nt, (nrows + nt - 1) / nt, inter, nrows);
    for (uint32_t k = wave; k < rows.limit; k += nwaves) {
      const uint32_t q = rows.row(k);
      if ((q + 1u) * kRowElems <= n) {  // uniform: the row is whole
        row<P, true>(in, sc, out, osc, q, 16u);
      } else {
        const uint32_t el = q * kRowElems + lane * 16u;
        const uint32_t have = el < n ? (n - el < 16u ? n - el : 16u) : 0u;
        row<P, false>(in, sc, out, osc, q, have);
      }
    }
  }
};

}  // namespace dev
}  // namespace pcoll
