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
// (dwordx4), 64 lanes cover 1 KiB per rank per step, and U steps are issued
// back to back so that U * P loads are in flight per lane before the first
// add.  Loads and stores carry the nontemporal hint: the data are touched
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

// Rows each lane loads at once: enough loads in flight, bounded register
// use.  DEEP (the default) keeps 4 rows in flight up to 8 ranks and 2 above
// (at 16 ranks 1.4 % faster than 1, with no spills); the shallow form keeps
// half of that from 3 ranks on, which needs fewer registers and leaves more
// room for kernels that run beside the reduction.
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
    // U rows at a time, then U / 2, then one: whatever is left of a tile has
    // as many loads in flight as it can
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
// One word's four values times the block scale (one multiply each).
template <class Fmt>
__device__ __forceinline__ void dec4(uint32_t w, float scale, float (&o)[4]) {
  auto lo = Fmt::template dec_pair<false>(w);
  auto hi = Fmt::template dec_pair<true>(w);
  o[0] = lo[0] * scale;
  o[1] = lo[1] * scale;
  o[2] = hi[0] * scale;
  o[3] = hi[1] * scale;
}

// Rank-order sum of word k of every rank's codes, plain or Sum2.  dec(word,
// rank, values) decodes one rank's word.  AGAIN: the rarely taken branch of
// a caller that has decoded the same words already; the empty asm keeps the
// compiler from holding those values in registers for it.
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

// Whether the compensated sums of the 8-bit payloads go through binary64
// (below): from 3 ranks on (64 buckets of e4m3, 2^29 values: 3 ranks 342 ->
// 314 us, 4 ranks 423 -> 383 us, 16 ranks 1569 -> 1393 us).  At 1 and 2 ranks
// Sum2 has no addition, or one, to compensate and costs less than the route.
template <bool COMP, int P>
constexpr bool kSumF64 = COMP && P >= 3;

// What the binary64 route needs to know of a lane's terms.
struct TermBound {
  float t;   // a sum whose nonzero terms are all larger than t in magnitude
             // is Sum2's exact case (see sum_word_f64)
  double b;  // how far Sum2's s + c can be from the binary64 sum
};

// All terms of the lane are at most big = kMax max|s_r| in magnitude.  Where
// a partial sum of P such terms could overflow, nothing is settled through
// binary64 (t and b infinite).
template <class Fmt, int P>
__device__ __forceinline__ TermBound term_bound(const float (&s_in)[P]) {
  // sum_{r=2}^{P-1} r (r + 3) / 2
  constexpr int kC = ((P - 1) * P * (2 * P - 1) / 6 - 1 +
                      3 * (P * (P - 1) / 2 - 1)) / 2;
  float smax = fabsf(s_in[0]);
#pragma unroll
  for (int r = 1; r < P; ++r) smax = fmaxf(smax, fabsf(s_in[r]));
  const bool far = !(smax < 0x1p126f / (Fmt::kMax * (float)P));
  const float big = far ? __builtin_inff() : smax * Fmt::kMax;
  return {big * ((float)(P * (P + 1) / 2) * 0x1p-24f),
          (double)big * ((double)(kC + P) * 0x1p-48)};
}

// The Sum2 result of word k's four values, computed through binary64.
//
// Sum2 in binary32 costs seven dependent operations per rank and value,
// which made these kernels wait for the VALU and not for memory.  A
// binary64 running sum D costs two (convert, add), at the same rate, and
// Sum2's result follows from it.  With u = 2^-24, E the exact sum and m the
// bound on every |p_r|, Sum2 returns fl32(s + c) where s + sum e_r = E
// exactly, |e_r| <= u (r + 1) m, and only c's own additions round:
//   * every nonzero term larger than t = u m P (P + 1) / 2: the terms, so
//     the e_r and c, are multiples of g >= u min|p_r|, and sum |e_r| < 2^24
//     g: c is exact, so is D, and the result is D rounded;
//   * else |s + c - E| <= u^2 m sum_{r=2}^{P-1} r (r + 3) / 2, and D is off
//     by far less: with b the sum of both, D - b and D + b that round to the
//     same binary32 value give the result, rounding being monotonic;
//   * else Sum2 itself, for the word.
// D's own ties are common (the terms have 24 bits each, so D often needs
// just one more: 9 % of values), which is why the first test comes first: a
// term below t appears in 0.2 % of gradient-like values, and one word in 20
// then needs the third (which tells zero terms from small ones), one in 50
// the last.  Sum2 never returns -0, which D rounds to only when every term
// is -0: the second and third test give +0 there.
//
// Row of 1024 values at 8 ranks without its memory traffic, per SIMD: Sum2
// 1776 ns, this about 980 ns.  The e4m3 kernel on 128 buckets, 2^30 values
// in all, 8 ranks: 1.90 -> 1.65 ms (4.6 -> 5.3 TB/s), 5 % above the same
// kernel with plain sums: what bounds it now is the memory streams.
template <int P, class Dec>
__device__ __forceinline__ void sum_word_f64(const uint4 (&raw)[P], int k,
                                             Dec&& dec, const TermBound& tb,
                                             float (&y)[4]) {
  double D[4];
  float least[4];
#pragma unroll
  for (int r = 0; r < P; ++r) {
    float d[4];
    dec(Word32::get(raw[r], k), r, d);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      D[j] = r == 0 ? (double)d[j] : D[j] + (double)d[j];
      least[j] = r == 0 ? fabsf(d[j]) : fminf(least[j], fabsf(d[j]));
    }
  }
  bool close = false;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    y[j] = (float)D[j];
    close |= !(least[j] > tb.t);
  }
  if (__builtin_expect(__ballot(close) == 0, 1)) return;
  bool open[4];
  bool any = false;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float lo = (float)(D[j] - tb.b), hi = (float)(D[j] + tb.b);
    open[j] = !(least[j] > tb.t) && !(lo == hi);
    if (lo == hi) y[j] = hi;
    any |= open[j];
  }
  if (__ballot(any) == 0) return;
  // the smallest nonzero term: twice the magnitude's bits less one, which
  // puts zero last
  uint32_t nz[4] = {~0u, ~0u, ~0u, ~0u};
#pragma unroll
  for (int r = 0; r < P; ++r) {
    float d[4];
    uint32_t w = Word32::get(raw[r], k);
    asm("" : "+v"(w));  // decoded again, not kept (see sum_word)
    dec(w, r, d);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      nz[j] = min(nz[j], (__float_as_uint(d[j]) << 1) - 1u);
  }
  any = false;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool exact = nz[j] >= __float_as_uint(tb.t) << 1;
    if (open[j] && exact) y[j] = (float)D[j] + 0.0f;
    any |= open[j] && !exact;
  }
  if (__ballot(any) != 0) sum_word<true, true>(raw, k, dec, y);
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
        raw[r] = ld_stream(reinterpret_cast<const uint4*>(
                               in[r] + (size_t)q * kRowElems) + lane_id());
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
    float y[16];
    float amax = 0.0f;
    const auto keep = [&](int k, const float(&v)[4]) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        y[4 * k + j] = v[j];
        if (FULL || (uint32_t)(4 * k + j) < have)
          amax = fmaxf(amax, fabsf(v[j]));
      }
    };
    if constexpr (kSumF64<COMP, P>) {
      const TermBound tb = term_bound<Fmt>(s_in);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float v[4];
        sum_word_f64(raw, k, dec, tb, v);
        keep(k, v);
      }
      // infinite codes (e5m2): what Sum2 makes of them
      if (__builtin_expect(__ballot(amax == __builtin_inff()) != 0, 0)) {
        amax = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float v[4];
          sum_word<true, true>(raw, k, dec, v);
          keep(k, v);
        }
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float v[4];
        sum_word<COMP, false>(raw, k, dec, v);
        keep(k, v);
      }
    }
    // max over the 16 lanes of the block
    amax = fmaxf(amax, __shfl_xor(amax, 8, 16));
    amax = fmaxf(amax, __shfl_xor(amax, 4, 16));
    amax = fmaxf(amax, __shfl_xor(amax, 2, 16));
    amax = fmaxf(amax, __shfl_xor(amax, 1, 16));
    float so = amax / Fmt::kMax;
    if (!(so >= 0x1p-126f)) so = 1.0f;
    const float inv = 1.0f / so;
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      w[k] = Fmt::enc4(y[4 * k] * inv, y[4 * k + 1] * inv, y[4 * k + 2] * inv,
                       y[4 * k + 3] * inv);
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

// Whether the exact sum, rounded once, is what Sum2 returns for a lane's
// values (32 buckets, 2^28 values, 8 ranks: 0.606 -> 0.509 ms, 4.9 -> 5.9
// TB/s, the time of plain sums; a row body 1540 -> 630 ns per SIMD): every decoded term is a multiple of g = 2^-9 2^(bmin - 127) of at
// most 448 * 2^(bmax - 127), so for bmax - bmin <= 23 and up to 16 ranks
// Sum2's errors add up to at most 135 u 448 2^(bmax - 127) <= 2^24 g: its
// correction is exact and its result the exact sum rounded; and the
// binary64 sum is exact too (22 + 23 bits).  Above byte 240 a partial sum
// could leave binary32's range.
__device__ __forceinline__ bool mx_exact(uint32_t bmin, uint32_t bmax) {
  return bmax <= 240u && bmax - bmin <= 23u;
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
    const auto dec = [&](uint32_t w, int r, float(&d)[4]) {
      mx_dec4(w, e8m0_operand(b_in[r]), d);
    };
    bool sum2 = COMP;  // the binary32 Sum2 itself
    if constexpr (kSumF64<COMP, P>) {
      uint32_t bmin = b_in[0], bmax = b_in[0];
#pragma unroll
      for (int r = 1; r < P; ++r) {
        bmin = min(bmin, b_in[r]);
        bmax = max(bmax, b_in[r]);
      }
      bool exact = mx_exact(bmin, bmax);
      if (__ballot(!exact) != 0) {
        // all-zero blocks carry byte 0: their scale does not count
        bmin = 255u;
        bmax = 0u;
#pragma unroll
        for (int r = 0; r < P; ++r) {
          const bool zero = ((raw[r].x | raw[r].y | raw[r].z | raw[r].w) &
                             0x7f7f7f7fu) == 0u;
          bmin = min(bmin, zero ? 255u : b_in[r]);
          bmax = max(bmax, zero ? 0u : b_in[r]);
        }
        exact = bmin == 255u && bmax == 0u ? true : mx_exact(bmin, bmax);
      }
      sum2 = __ballot(!exact) != 0;
    }
    float y[16];
    float amax = 0.0f;
    if (kSumF64<COMP, P> && !sum2) {
      // binary64 running sums (exact here), rounded once; + 0 turns -0 into
      // Sum2's +0
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        double D[4];
#pragma unroll
        for (int r = 0; r < P; ++r) {
          float d[4];
          dec(Word32::get(raw[r], k), r, d);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            D[j] = r == 0 ? (double)d[j] : D[j] + (double)d[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) y[4 * k + j] = (float)D[j] + 0.0f;
        // one word at a time: the other words' terms would only hold
        // registers
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float v[4];
        sum_word<COMP, kSumF64<COMP, P>>(raw, k, dec, v);
#pragma unroll
        for (int j = 0; j < 4; ++j) y[4 * k + j] = v[j];
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
