// Exact dot products of bf16 rows on the int8 matrix cores, for the scorers.
//
// The scorers need q . k to far better than fp32 (the selection compares
// scores position by position), and the float64 matrix cores give 78 TFLOP/s
// where the int8 ones give 5 Pop/s.  A bf16 element has 8 significant bits, so
// a row scaled by a power of two is, in practice, a row of integers: with the
// row's largest exponent E,
//   x_i = X_i 2^(E-29),  |X_i| < 2^30,  exact for |x_i| >= 2^(E-22) (or 0),
// and X_i = d0 2^24 + d1 2^16 + d2 2^8 + d3 with balanced digits d0..d3 in
// [-128, 127].  Products of digit planes are int8 matrix products, exact in
// int32: with |d0| <= 64, S_s = sum_{i+j=s} d_i . d'_j over up to 128 elements
// is at most 2^19, 2^21, 2^22, 6 2^20, 3 2^21 for s = 0 .. 4.  The 13 plane
// pairs with i + j <= 4 are computed (the other three multiply d2 d3', d3 d2',
// d3 d3': nonzero only where both elements are under 2^-6 of their rows'
// largest and one under 2^-14).  What is left out is bounded for the data at
// hand: `b` (below) collects 2^15 |d3|_1 (the omitted pairs) and
// 2^30 |X - x 2^(29-E)|_1 (elements below 2^-22 of the largest, truncated), and
// a tile whose bound passes kMaxErr in the exponent of the softmax (base 2), or
// that holds an infinity or a NaN, is computed with float64 products instead.
// So a logit is the exact product (without d3 digits and truncation: nearly
// always) or within 2^-26 of it, the rounding to fp32 of its own exponential's
// argument.  (At 2^-28 the 0.6% of a normal prompt's tiles that hold an element
// under 2^-22 of its row's largest took float64 products, six times the work.)
#pragma once

#include "common.h"

namespace tb {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(4))) double f64x4;

constexpr int kDigits = 4;
constexpr int kSums = 5;                     // digit sums i + j = 0 .. 4
constexpr float kMaxErr = 0x1p-26f;          // largest tolerated error of a base-2 exponent
constexpr float kFarErr = 0x1p-24f;          // a bound past this one is the data's, not one tile's
constexpr int kF64Run = 8;                   // tiles that then take float64 products unseen
// Counted as an error of 2^13 product units, so that a tile of digits has
// |t| < 2^28: its |X . X'| <= 2^67 is 2^54 times this share of the bound.
constexpr float kBase = 0x1p13f;

// Largest |x| of 8 bf16 as a 15-bit pattern (ordered like the magnitude).
__device__ __forceinline__ uint32_t absmax8(const uint4& v) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  constexpr uint32_t kM = 0x7fff7fffu;
  const u16x2 a = __builtin_elementwise_max(__builtin_bit_cast(u16x2, v.x & kM),
                                            __builtin_bit_cast(u16x2, v.y & kM));
  const u16x2 b = __builtin_elementwise_max(__builtin_bit_cast(u16x2, v.z & kM),
                                            __builtin_bit_cast(u16x2, v.w & kM));
  const u16x2 m = __builtin_elementwise_max(a, b);
  return max(static_cast<uint32_t>(m[0]), static_cast<uint32_t>(m[1]));
}

// The scale 2^(29-E) and the unit 2^(E-29) of a row whose largest magnitude
// has the pattern m (E >= -97, so that both are normal fp32 numbers).
struct RowScale {
  float scale, unit;
  bool finite;
};
__device__ __forceinline__ RowScale row_scale(uint32_t m) {
  const uint32_t eb = max(m >> 7, 30u);                     // biased exponent
  return {__uint_as_float((283u - eb) << 23), __uint_as_float((eb - 29u) << 23), eb < 255u};
}

// Digit planes of 8 elements (plane p: byte i = digit p of element i); n3
// collects |d3|, and resid (RESID) |x scale - X|.
template <bool RESID>
__device__ __forceinline__ void digits8(const uint4& v, float scale, uint2 (&p)[kDigits],
                                        float& resid, uint32_t& n3) {
  float x[8];
  Elem<bf16_t>::widen(v, x);
  uint32_t y[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float t = x[i] * scale;
    const int X = static_cast<int>(t);
    if (RESID) resid += fabsf(t - static_cast<float>(X));
    y[i] = static_cast<uint32_t>(X) + 0x00808080u;          // bytes 0-2 offset by 128
  }
  uint32_t w[kDigits][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {                             // 4 x 4 byte transposes
    const uint32_t lo01 = __builtin_amdgcn_perm(y[4 * h + 1], y[4 * h], 0x05010400u);
    const uint32_t hi01 = __builtin_amdgcn_perm(y[4 * h + 1], y[4 * h], 0x07030602u);
    const uint32_t lo23 = __builtin_amdgcn_perm(y[4 * h + 3], y[4 * h + 2], 0x05010400u);
    const uint32_t hi23 = __builtin_amdgcn_perm(y[4 * h + 3], y[4 * h + 2], 0x07030602u);
    const uint32_t u3 = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
    n3 = __builtin_amdgcn_sad_u8(u3, 0x80808080u, n3);
    w[3][h] = u3 ^ 0x80808080u;
    w[2][h] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u) ^ 0x80808080u;
    w[1][h] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u) ^ 0x80808080u;
    w[0][h] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
  }
#pragma unroll
  for (int k = 0; k < kDigits; ++k) p[k] = make_uint2(w[k][0], w[k][1]);
}

// Smallest nonzero |x| of 8 bf16, minus one, as a 15-bit pattern (0xffff if all
// are zero).
__device__ __forceinline__ uint32_t absmin8(const uint4& v) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  u16x2 m = {0xffff, 0xffff};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    m = __builtin_elementwise_min(m, __builtin_bit_cast(u16x2, w[i] & 0x7fff7fffu) - u16x2{1, 1});
  return min(static_cast<uint32_t>(m[0]), static_cast<uint32_t>(m[1]));
}

// The bound's share of a row, in product units (the partner is below 2^30).
__device__ __forceinline__ float digit_bound(float resid, uint32_t n3) {
  return fmaf(resid, 0x1p30f, static_cast<float>(n3) * 0x1.02p15f);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return __builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xF, 0xF, true);
}

// The value of lanes l ^ 16 (l ^ 32): one result of the self-swap is the
// lane's own value, the other its partner's, so a commutative f(x, y) of both
// results is the pair's.
template <typename F>
__device__ __forceinline__ uint32_t pair16(uint32_t x, F f) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return f(r[0], r[1]);
}
template <typename F>
__device__ __forceinline__ uint32_t pair32(uint32_t x, F f) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return f(r[0], r[1]);
}
// over the four lane groups l, l ^ 16, l ^ 32, l ^ 48
template <typename F>
__device__ __forceinline__ uint32_t group_all(uint32_t x, F f) { return pair32(pair16(x, f), f); }
// over the whole wave
template <typename F>
__device__ __forceinline__ uint32_t wave_all(uint32_t x, F f) {
  x = f(x, dpp_u32<kDppQuadXor1>(x));
  x = f(x, dpp_u32<kDppQuadXor2>(x));
  x = f(x, dpp_u32<kDppRowHalfMirror>(x));
  x = f(x, dpp_u32<kDppRowMirror>(x));
  return group_all(x, f);
}
struct UMax { __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return max(a, b); } };
struct IMax {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const {
    return static_cast<uint32_t>(max(static_cast<int>(a), static_cast<int>(b)));
  }
};
struct FAdd {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const {
    return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
  }
};
// NaN-propagating maximum: a bound that is not a number must stay one
struct FMax {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const {
    return __float_as_uint(__builtin_elementwise_maximum(__uint_as_float(a), __uint_as_float(b)));
  }
};

// f over the four lane groups of a float64, the same result in each (through two
// 32-bit swaps): f(x, x of lane l ^ 16), then l ^ 32.
template <typename F>
__device__ __forceinline__ double group_f64(double x, F f) {
  auto swap = [f](double v, bool by32) {
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = static_cast<uint32_t>(u), hi = static_cast<uint32_t>(u >> 32);
    uint32_t l0, l1, h0, h1;
    if (by32) {
      const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
      l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
    } else {
      const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
      const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
      l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
    }
    return f(__longlong_as_double((static_cast<uint64_t>(h0) << 32) | l0),
             __longlong_as_double((static_cast<uint64_t>(h1) << 32) | l1));
  };
  return swap(swap(x, false), true);
}
__device__ __forceinline__ double group_sum_f64(double x) {
  return group_f64(x, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double group_max_f64(double x) {
  return group_f64(x, [](double a, double b) { return fmax(a, b); });
}

// 2^t as fp32 for a float64 t: t = n + f with n = round(t) exact and
// |f| <= 1/2, so only f is rounded to fp32 (relative effect on 2^f below
// 3e-8); 2^f comes from the hardware base-2 exponential (about 1 ulp) and the
// scaling by 2^n is exact (results under the smallest fp32 subnormal are 0).
__device__ __forceinline__ float exp2_split(double t) {
  const double n = rint(t);
  return ldexpf(__builtin_amdgcn_exp2f(static_cast<float>(t - n)), static_cast<int>(n));
}
// the same for |t| < 2^31, with n as the low word of t + 1.5 2^52
__device__ __forceinline__ float exp2_short(double t) {
  const double y = t + 0x1.8p52;
  return ldexpf(__builtin_amdgcn_exp2f(static_cast<float>(t - (y - 0x1.8p52))),
                static_cast<int>(static_cast<uint32_t>(__double_as_longlong(y))));
}
// the same for any t: 2^-inf = 0, and n stays within int
__device__ __forceinline__ float exp2_clamped(double t) {
  const double n = rint(fmax(t, -300.0));
  return ldexpf(__builtin_amdgcn_exp2f(static_cast<float>(t - n)), static_cast<int>(fmin(n, 300.0)));
}

// ------------------------------------------------------ stationary operand
// The wave's 32 stationary rows (two 16-row column tiles) as digit planes in
// registers: lane (q4, r16) holds row r16 of tile c, d = 64 ks + 16 q4 .. +15
// of every plane.  coef[c] is the row's unit; U and V bound the wave's rows
// (largest unit; largest unit * (kBase + b)).
template <int D>
struct Stationary {
  static constexpr int KS = D / 64;          // 64-deep steps of the int8 product
  i32x4 dig[2][KS][kDigits];
  float unit[2];
  float U, V;

  // src[c]: this lane's row of tile c (any valid row for padding)
  __device__ __forceinline__ void load(const uint16_t* const (&src)[2], int q4) {
    U = 0.f;
    V = 0.f;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      uint4 raw[KS][2];
      uint32_t m = 0u;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          raw[ks][h] = ldg16(src[c] + 64 * ks + 16 * q4 + 8 * h);
          m = max(m, absmax8(raw[ks][h]));
        }
      const RowScale rs = row_scale(group_all(m, UMax()));
      float resid = 0.f;
      uint32_t n3 = 0u;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        uint2 lo[kDigits], hi[kDigits];
        digits8<true>(raw[ks][0], rs.scale, lo, resid, n3);
        digits8<true>(raw[ks][1], rs.scale, hi, resid, n3);
#pragma unroll
        for (int k = 0; k < kDigits; ++k)
          dig[c][ks][k] = i32x4{static_cast<int>(lo[k].x), static_cast<int>(lo[k].y),
                                static_cast<int>(hi[k].x), static_cast<int>(hi[k].y)};
      }
      const float b = __uint_as_float(group_all(__float_as_uint(digit_bound(resid, n3)), FAdd()));
      unit[c] = rs.unit;
      const float v = rs.finite ? rs.unit * (kBase + b) : INFINITY;
      U = fmaxf(U, rs.unit);
      V = __builtin_elementwise_maximum(V, v);
    }
    U = __uint_as_float(wave_all(__float_as_uint(U), FMax()));
    V = __uint_as_float(wave_all(__float_as_uint(V), FMax()));
  }
};

// ------------------------------------------------------- streamed operand
// A tile of 64 streamed rows: digit planes in LDS, [plane][row][D bytes],
// 16-byte chunk ch of row r at ch ^ swz(r) (16 rows at one chunk then cover
// all banks), plus per staging group (the rows one wave stages together)
// its unit and unit * b.
template <int D>
struct StreamTile {
  static constexpr int LPR = D / 8;          // lanes per row (8 elements each)
  static constexpr int RPG = 64 / LPR;       // rows per group
  static constexpr int NG = 64 / RPG;        // groups per tile (16 or 8)
  alignas(16) uint8_t dig[kDigits][64 * D];  // read 16 bytes at a time
  float2 grp[NG];

  static __device__ __forceinline__ int swz(int r) { return D == 128 ? (r >> 1) & 7 : (r >> 2) & 3; }

  // One wave converts and stores group gi, of which this lane holds 8
  // elements.  Straight-line code (it is scheduled among matrix products);
  // a nonzero result in any lane says that the group has a bound, which
  // put_bound then stores.
  __device__ __forceinline__ uint32_t put(int gi, int lane, const uint4& raw) {
    const uint32_t m = wave_all(absmax8(raw), UMax());
    const RowScale rs = row_scale(m);
    float unused = 0.f;
    uint32_t n3 = 0u;
    uint2 p[kDigits];
    digits8<false>(raw, rs.scale, p, unused, n3);
    const int r = gi * RPG + lane / LPR, c8 = lane % LPR;
    const int off = r * D + (((c8 >> 1) ^ swz(r)) << 4) + (c8 & 1) * 8;
#pragma unroll
    for (int k = 0; k < kDigits; ++k) *reinterpret_cast<uint2*>(&dig[k][off]) = p[k];
    grp[gi] = make_float2(rs.unit, 0.f);                    // all lanes, one value
    // truncated elements are below 2^(E-22)
    const uint32_t lost = absmin8(raw) < ((max(m >> 7, 30u) - 22u) << 7) - 1u ? 1u : 0u;
    return n3 | lost | (rs.finite ? 0u : 1u);
  }
  // the group's total bounds each of its rows
  __device__ __forceinline__ void put_bound(int gi, int lane, const uint4& raw) {
    const RowScale rs = row_scale(wave_all(absmax8(raw), UMax()));
    float resid = 0.f;
    uint32_t n3 = 0u;
    uint2 p[kDigits];
    digits8<true>(raw, rs.scale, p, resid, n3);
    const float b = __uint_as_float(wave_all(__float_as_uint(digit_bound(resid, n3)), FAdd()));
    if (lane == 0) grp[gi].y = rs.finite ? rs.unit * b : INFINITY;
  }
  // operand of rows 16 kt + r16, d = 64 ks + 16 q4 .. +15, plane k
  __device__ __forceinline__ i32x4 get(int kt, int ks, int k, int q4, int r16) const {
    return *reinterpret_cast<const i32x4*>(
        &dig[k][(16 * kt + r16) * D + (((4 * ks + q4) ^ swz(r16)) << 4)]);
  }
  // the group holding rows 16 kt + 4 q4 .. +3
  static __device__ __forceinline__ int group_of(int kt, int q4) { return (16 * kt + 4 * q4) / RPG; }
  // wave-uniform: every product of the tile with the rows (U, V) stays within
  // `most` of the exponent (false for anything that is not a number)
  __device__ __forceinline__ bool within(float U, float V, float c, float most, int lane) const {
    const float2 g = grp[lane % NG];
    return __builtin_amdgcn_ballot_w64(!((V * g.x + U * g.y) * c <= most)) == 0;
  }
};

// Staging of streamed tiles by the WAVES waves of a block: wave w converts
// groups w MP .. w MP + MP - 1.  4 or 8 waves: two LDS buffers (one barrier a
// tile) and rows fetched a tile ahead, into registers; 1 or 2 waves: one
// buffer, the other blocks of the CU fill the gaps.
//
// The block decides together (U and V over all its rows, so every wave finds the
// same) whether a tile's digits will do.  Keys with a channel far above the rest
// fail in every tile; so a tile far past the bound sends the next ones to
// float64 products too, without staging, looking or barriers: the waves then run
// on their own.
template <int D, int WAVES>
struct Stager {
  using Tile = StreamTile<D>;
  static constexpr int MP = Tile::NG > WAVES ? Tile::NG / WAVES : 1;   // groups per wave
  static constexpr bool kTwo = WAVES >= 4;
  static constexpr int kBuffers = kTwo ? 2 : 1;
  static constexpr int kWin = MP < 4 ? MP : 4;                         // groups held in registers
  const uint16_t* src;                       // row 0
  int n_rows, n_tiles, wave, lane;
  float U, V, c;                             // of the block's stationary rows (share)
  uint4 raw[kWin];

  __device__ __forceinline__ bool stages() const { return wave * MP < Tile::NG; }   // wave-uniform
  // this lane's 8 elements of group u; rows past the end: the last row, tiles
  // past the end: the last tile (a wave-uniform base and a 32-bit lane offset)
  __device__ __forceinline__ uint4 fetch(int tile, int u) const {
    const int k0 = min(tile, n_tiles - 1) * 64;
    const int r = min((wave * MP + u) * Tile::RPG + lane / Tile::LPR, n_rows - 1 - k0);
    const uint32_t off = (r * D + 8 * (lane % Tile::LPR)) * 2;
    return ldg16(reinterpret_cast<const char*>(src + static_cast<size_t>(k0) * D) + off);
  }
  __device__ __forceinline__ void start(int tile) {
    if (kTwo && stages()) {
#pragma unroll
      for (int u = 0; u < kWin; ++u) raw[u] = fetch(tile, u);
    }
  }
  // the bound's factors over the block's waves; every wave, once
  __device__ __forceinline__ void share(float2 (&uv)[WAVES], float u, float v, float scale) {
    if (lane == 0) uv[wave] = make_float2(u, v);
    __syncthreads();
    U = V = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      U = fmaxf(U, uv[w].x);
      V = __builtin_elementwise_maximum(V, uv[w].y);
    }
    U = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(U)));   // scalar registers
    V = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(V)));
    c = scale;
  }
  // Stage a tile and look at it: its digits, or nullptr where they will not do.
  // The tiles from there to `end` are then for float64 products, and every wave
  // calls resume(end) behind them.  All waves of the block call these for the
  // same tiles, so they meet the same barriers.
  __device__ __forceinline__ const Tile* look(Tile* buf, int tile, int first, int last, int& end) {
    const Tile& st = stage(buf, tile, first);
    if (st.within(U, V, c, kMaxErr, lane)) return &st;
    end = st.within(U, V, c, kFarErr, lane) ? tile + 1 : min(tile + kF64Run, last);
    return nullptr;
  }
  __device__ __forceinline__ void resume(int end) {
    start(end);
    __syncthreads();                         // every wave has looked at the tile that failed
  }
  // Stage a tile and wait for it.
  __device__ __forceinline__ Tile& stage(Tile* buf, int tile, int first) {
    Tile& st = buf[kTwo ? (tile - first) & 1 : 0];
    if (!kTwo && tile > first) __syncthreads();             // the previous tile has been read
    if (stages()) {
      uint32_t flags = 0u;
#pragma unroll
      for (int u0 = 0; u0 < MP; u0 += kWin) {
        if (!kTwo) {
#pragma unroll
          for (int u = 0; u < kWin; ++u) raw[u] = fetch(tile, u0 + u);
        }
#pragma unroll
        for (int u = 0; u < kWin; ++u) flags |= st.put(wave * MP + u0 + u, lane, raw[u]);
      }
      if (__builtin_amdgcn_ballot_w64(flags != 0u)) {       // rare: the groups get their bounds
        if constexpr (MP == kWin) {
#pragma unroll
          for (int u = 0; u < MP; ++u) st.put_bound(wave * MP + u, lane, raw[u]);
        } else {
          for (int u = 0; u < MP; ++u) st.put_bound(wave * MP + u, lane, fetch(tile, u));
        }
      }
      if (kTwo) start(tile + 1);
    }
    __syncthreads();
    return st;
  }
};

// The 13 digit products of 16 streamed rows (operands A of StreamTile::get)
// with column tile c: lane (q4, r16) gets S_s of streamed rows 4 q4 + i (item
// i), stationary row r16 of the tile.
template <int D>
__device__ __forceinline__ void digit_products(const i32x4 (&A)[Stationary<D>::KS][kDigits],
                                               const Stationary<D>& sx, int c, i32x4 (&S)[kSums]) {
#pragma unroll
  for (int s = 0; s < kSums; ++s) S[s] = i32x4{0, 0, 0, 0};
#pragma unroll
  for (int ks = 0; ks < Stationary<D>::KS; ++ks)
#pragma unroll
    for (int j = 0; j < kDigits; ++j)
#pragma unroll
      for (int i = 0; i < kDigits; ++i)
        if (i + j < kSums)
          S[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[ks][i], sx.dig[c][ks][j], S[i + j], 0, 0, 0);
}

// The products of a whole tile, software-pipelined: step s = 2 kt + c issues
// the products of step s + 1 and hands the sums of step s to use(kt, c, S).
// `use` must not branch: each step is one scheduling region in which products
// and vector instructions alternate, so the int8 matrix cores run under the
// float64 recombination and the exponentials of the step before (unscheduled,
// the two came in blocks and did not overlap).
template <int D, typename F>
__device__ __forceinline__ void pipelined_products(const StreamTile<D>& st, const Stationary<D>& sx,
                                                   int q4, int r16, F use) {
  constexpr int KS = Stationary<D>::KS;
  constexpr int kValu = D == 128 ? 3 : 6;    // vector instructions per product
  i32x4 A[KS][kDigits], S[2][kSums];
  auto load = [&](int kt) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int k = 0; k < kDigits; ++k) A[ks][k] = st.get(kt, ks, k, q4, r16);
  };
  load(0);
  digit_products<D>(A, sx, 0, S[0]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    if (s < 7) {
      if (s & 1) load((s + 1) >> 1);
      digit_products<D>(A, sx, (s + 1) & 1, S[(s + 1) & 1]);
    }
    use(s >> 1, s & 1, S[s & 1]);
    if (s < 7) {
      if (s & 1) __builtin_amdgcn_sched_group_barrier(0x100, KS * kDigits, 0);   // LDS reads first
#pragma unroll
      for (int k = 0; k < 13 * KS; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);                         // one product,
        __builtin_amdgcn_sched_group_barrier(0x2, kValu, 0);                     // some vector work
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The same without overlap, for a few tiles whose longer `use` would not leave
// registers for it.
template <int D, typename F>
__device__ __forceinline__ void stepwise_products(const StreamTile<D>& st, const Stationary<D>& sx,
                                                  int q4, int r16, F use) {
  constexpr int KS = Stationary<D>::KS;
#pragma unroll 1
  for (int kt = 0; kt < 4; ++kt) {
    i32x4 A[KS][kDigits], S[kSums];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int k = 0; k < kDigits; ++k) A[ks][k] = st.get(kt, ks, k, q4, r16);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      digit_products<D>(A, sx, c, S);
      use(kt, c, S);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// The dot product behind item i of the sums, in units of 2^16 times the rows'
// units: hi 2^24 + mid 2^8 + S4 with hi = S0 2^8 + S1 and mid = S2 2^8 + S3,
// all within int32, and every step in float64 exact.  (A conversion runs at
// half rate; integers placed in a float64's low word by bit operations cost the
// same and hold constants in registers: three of them 2-5% of an H2O call.)
__device__ __forceinline__ double digit_value(const i32x4 (&S)[kSums], int i) {
  const int hi = (S[0][i] << 8) + S[1][i], mid = (S[2][i] << 8) + S[3][i];
  return fma(static_cast<double>(hi), 0x1p24, fma(static_cast<double>(mid), 0x1p8, static_cast<double>(S[4][i])));
}

// float64 products of whole tiles with the wave's rows, straight from memory, for
// tiles that the digits cannot hold: `src` has the streamed rows (those past the
// end: the last one), `col` are the lane's two stationary rows.  The float64
// 16x16x4 product returns row l/16 + 4 v in item v, so the streamed row behind
// MFMA row p is 16 kt + 4 (p % 4) + p / 4, and item i of t[c][kt] is streamed
// row 16 kt + 4 q4 + i with the row of column tile c, as in the digit sums.  d
// runs in 16-wide chunks, of which a lane reads 4 consecutive elements (d =
// 16 ch + 4 q4 + step) of either operand, a chunk ahead, across tiles too: the
// first chunk of the next tile comes from HBM, and a wait for it issued behind
// the caller's stores would wait for those.  The whole tile's logits stay in
// registers (64), so nothing is computed twice.
template <int D>
struct F64Tiles {
  const uint16_t* src;
  int n_rows;
  const uint16_t* col[2];                    // + 4 q4
  int q4, sub;                               // sub: the lane's streamed row within 16
  double scale;
  uint2 next[6];

  __device__ __forceinline__ void fetch(int tile, int ch) {
    const int base = min(tile * 64, n_rows - 1);
    const uint16_t* rows = src + static_cast<size_t>(base) * D;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
      next[kt] = *reinterpret_cast<const uint2*>(rows + min(16 * kt + sub, n_rows - 1 - base) * D + 4 * q4 + 16 * ch);
#pragma unroll
    for (int c = 0; c < 2; ++c) next[4 + c] = *reinterpret_cast<const uint2*>(col[c] + 16 * ch);
  }
  __device__ __forceinline__ F64Tiles(const uint16_t* s, int n, const uint16_t* const (&rows)[2], int q4_, int r16,
                                      double scale_, int tile)
      : src(s), n_rows(n), col{rows[0] + 4 * q4_, rows[1] + 4 * q4_}, q4(q4_), sub(4 * (r16 & 3) + (r16 >> 2)),
        scale(scale_) {
    fetch(tile, 0);
  }
  // the tile's logits in base-2 units; tiles come in order
  __device__ __forceinline__ void products(int tile, f64x4 (&t)[2][4]) {
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) t[0][kt] = t[1][kt] = f64x4{0.0, 0.0, 0.0, 0.0};
    auto widen = [](const uint2& v, int s) { // element s of 4
      const uint32_t w = s < 2 ? v.x : v.y;
      return static_cast<double>(__uint_as_float(s & 1 ? w & 0xffff0000u : w << 16));
    };
#pragma unroll 1
    for (int ch = 0; ch < D / 16; ++ch) {
      uint2 v[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) v[k] = next[k];
      const bool end = ch == D / 16 - 1;
      fetch(end ? tile + 1 : tile, end ? 0 : ch + 1);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const double b0 = widen(v[4], s), b1 = widen(v[5], s);
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
          const double x = widen(v[kt], s);
          t[0][kt] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b0, t[0][kt], 0, 0, 0);
          t[1][kt] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b1, t[1][kt], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      t[0][kt] *= scale;
      t[1][kt] *= scale;
    }
  }
};

}  // namespace tb
