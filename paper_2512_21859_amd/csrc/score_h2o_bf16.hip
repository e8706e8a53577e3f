// H2O scoring for bf16 inputs (score_h2o.hip has the definition and the fp32
// kernels): the two causal passes on the int8 matrix cores (exact_dot.h).
//
//   rows: block = WAVES waves of 32 consecutive queries of one query head, in
//     registers as digits; the key tiles up to the diagonal stream through LDS.
//     Every row keeps an integer base-2 reference and its sum of 2^(t - ref);
//     a tile whose largest logit passes the reference by 2^60 is redone.  The
//     log-sum-exp goes to row_M, the reference to row_Z.
//   cols: block = WAVES waves of 32 consecutive keys; the query tiles from the
//     diagonal on stream through LDS, with these.
//     Streamed rows are the MFMA rows, so a lane's 16 logits of a tile belong
//     to one key: it adds 2^(t - lse) to that key's float64 sum and the lanes
//     meet only at the end.  Per-head column masses; the caller's merge adds
//     the heads.
//
// Both are bound by vector instructions (about 19 per logit, and 100 per 512
// streamed elements converted); the products run under them.  L = 4096, 28 query
// heads on 4 KV heads, d = 128, traced: 457 + 442 us against 1423 + 1349 with
// float64 products.  Tiles that the digits cannot hold take those (F64Tiles).

#include <type_traits>

#include "exact_dot.h"
#include "kernels.h"

namespace tb {
namespace {

constexpr int kT = 64;                       // streamed rows per tile
constexpr int kNone = -(1 << 29);            // n of a masked logit
// kinds of passes over a tile: every logit counts; up to the diagonal; the first
// query tile, whose rows see one tile only.  With few keys the rounding of a
// row's largest term does not average out, so there the reference is the row's
// largest logit itself and the sum is not rounded on the way; and the column
// pass adds the very terms that the row pass summed, over their sum.  (Against
// 2^(t - lse) throughout, error of the scores from float64: 2 tokens 2.55 ->
// 2.29e-8, 300 tokens 2.543 -> 2.536e-8; 2.27 and 2.539e-8 with float64 products
// and a reference for each tile.)
enum { kPlain, kMasked, kFirst };
// a reference stands while the tile's largest n is at most kHigh above it, and
// that of the row's first tile with a logit over -inf at least kLow (the row's
// largest term then keeps its fp32 precision, and everything under 2^-102 of it
// vanishes)
constexpr int kLow = -24, kHigh = 60;

// Block order (one-dimensional grid): workgroup i runs on XCD i % 8, and XCD x
// takes the units x, x + 8, ... of (rank, batch, KV head), heaviest ranks
// first, the G query heads of a unit in G consecutive slots of it, so the
// blocks that stream one KV head's keys share that XCD's L2.
__device__ __forceinline__ void h2o_unit(const H2oArgs& a, int& rank, int& h, int& b) {
  const int G = a.Hq / a.Hkv;
  const int wg = static_cast<int>(blockIdx.x);
  const int slot = wg >> 3, unit = (slot / G) * 8 + (wg & 7);
  const int g = unit % a.Hkv, rb = unit / a.Hkv;
  b = rb % a.B;
  rank = rb / a.B;
  h = g * G + slot % G;
}

template <int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2)))
void h2o_rows_i8_kernel(H2oArgs a) {
  using Tile = StreamTile<D>;
  constexpr int kRows = 32 * WAVES;
  int rank, h, b;
  h2o_unit(a, rank, h, b);
  if (b >= a.B || rank >= a.n_ranks) return;                // padding of the last XCD round
  const int L = a.L[b], nt = (L + kT - 1) / kT;
  const int qb = (L + kRows - 1) / kRows - 1 - rank;        // latest rows first
  if (qb < 0) return;                                       // shorter sequence of the batch
  const int g = h / (a.Hq / a.Hkv);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q4 = lane >> 4, r16 = lane & 15;
  const uint16_t* qh = static_cast<const uint16_t*>(a.q) + (static_cast<size_t>(b) * a.Hq + h) * a.Lmax * D;
  const uint16_t* kg = static_cast<const uint16_t*>(a.k) + (static_cast<size_t>(b) * a.Hkv + g) * a.Lmax * D;
  const int row0 = qb * kRows + 32 * wave;
  const int t_hi = (min(L, (qb + 1) * kRows) + kT - 1) / kT;               // tiles of the block
  const int w_hi = row0 < L ? (min(L, row0 + 32) + kT - 1) / kT : 0;       // of this wave

  __shared__ Tile s_tile[Stager<D, WAVES>::kBuffers];
  Stager<D, WAVES> keys{kg, L, nt, wave, lane};
  keys.start(0);
  Stationary<D> sx;
  const uint16_t* col[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) col[c] = qh + static_cast<size_t>(min(row0 + 16 * c + r16, L - 1)) * D;
  sx.load(col, q4);
  const double cd = a.scale * 1.4426950408889634;
  __shared__ float2 s_uv[WAVES];
  keys.share(s_uv, sx.U, sx.V, static_cast<float>(cd));
  const double cu[2] = {static_cast<double>(sx.unit[0]) * (cd * 0x1p16),
                        static_cast<double>(sx.unit[1]) * (cd * 0x1p16)};

  double ref[2] = {0.0, 0.0}, z[2] = {0.0, 0.0};            // this lane's share of the sum
  bool seen[2] = {false, false};                            // the row has had a logit over -inf
  for (int tile = 0, end; tile < t_hi;) {
    const Tile* st = keys.look(s_tile, tile, 0, t_hi, end);
    if (st && tile >= w_hi) {                               // wave-uniform
      ++tile;
      continue;
    }
    const int kbase = tile * kT;
    const bool edge = kbase + kT - 1 > row0;
    // take the tile's largest n (or logit) per row into the references; false
    // where a row's reference moved and the tile has to be redone
    const bool one = w_hi == 1;
    auto settle = [&](const double (&top)[2]) {
      bool moved = false;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double to = one ? top[c] : rint(top[c]), over = to - ref[c];
        if (fabs(top[c]) < INFINITY && (over > kHigh || (!seen[c] && over < kLow) || (one && over != 0.0))) {
          z[c] = ldexp(z[c], static_cast<int>(fmax(-over, -4000.0)));
          ref[c] = to;
          moved = true;
        }
        seen[c] = seen[c] || top[c] > -INFINITY;
      }
      return __builtin_amdgcn_ballot_w64(moved) == 0;
    };
    if (st) {
      auto pass = [&](auto kind) -> bool {
        asm volatile("" ::: "memory");       // no operand is read ahead of the pass
        constexpr int kKind = decltype(kind)::value;
        int top[2] = {kNone, kNone}, iref[2];
        double tops[2] = {-INFINITY, -INFINITY}, zt[2] = {0.0, 0.0}, cref[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          cref[c] = fmin(fmax(ref[c], -0x1p30), 0x1p30);
          iref[c] = static_cast<int>(cref[c]);
        }
        auto use = [&](int kt, int c, const i32x4 (&S)[kSums]) {
          const double f = st->grp[Tile::group_of(kt, q4)].x * cu[c];
          if constexpr (kKind == kFirst) {   // any reference, terms summed as they are
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const double t = digit_value(S, i) * f;
              const bool ok = kbase + 16 * kt + 4 * q4 + i <= row0 + 16 * c + r16;
              tops[c] = ok ? fmax(tops[c], t) : tops[c];
              zt[c] += static_cast<double>(ok ? exp2_short(t - cref[c]) : 0.f);
            }
          } else {
            float e[4];
            int n[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const double v = digit_value(S, i);
              const double y = fma(v, f, 0x1.8p52);         // round(t) in the low word
              n[i] = static_cast<int>(static_cast<uint32_t>(__double_as_longlong(y)));
              e[i] = ldexpf(__builtin_amdgcn_exp2f(static_cast<float>(fma(v, f, 0x1.8p52 - y))), n[i] - iref[c]);
              if constexpr (kKind == kMasked) {
                const bool ok = kbase + 16 * kt + 4 * q4 + i <= row0 + 16 * c + r16;
                n[i] = ok ? n[i] : kNone;
                e[i] = ok ? e[i] : 0.f;
              }
            }
            top[c] = max(max(top[c], max(n[0], n[1])), max(n[2], n[3]));
            zt[c] += static_cast<double>((e[0] + e[1]) + (e[2] + e[3]));
          }
          asm volatile("" : "+v"(zt[c]));    // summed here, not sunk behind the check of the references
        };
        if constexpr (kKind == kFirst) stepwise_products<D>(*st, sx, q4, r16, use);
        else                           pipelined_products<D>(*st, sx, q4, r16, use);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          if constexpr (kKind == kFirst) {
            tops[c] = group_max_f64(tops[c]);
          } else {
            const int t = static_cast<int>(group_all(static_cast<uint32_t>(top[c]), IMax()));
            tops[c] = t == kNone ? -INFINITY : static_cast<double>(t);
          }
        }
        const bool ok = settle(tops);
        if (ok) {
#pragma unroll
          for (int c = 0; c < 2; ++c) z[c] += zt[c];
        }
        return ok;
      };
      if (one) {
        while (!pass(std::integral_constant<int, kFirst>())) {}              // twice at most
      } else {
        bool done = !edge && pass(std::integral_constant<int, kPlain>());
        while (!done) done = pass(std::integral_constant<int, kMasked>());   // twice at most
      }
      ++tile;
      continue;
    }
    if (tile < w_hi) {
      F64Tiles<D> f64(kg, L, col, q4, r16, cd, tile);
      for (int u = tile; u < min(end, w_hi); ++u) {
        f64x4 t[2][4];
        f64.products(u, t);
        const int first = u * kT + 4 * q4 - (row0 + r16);   // the lane's first key from its rows' diagonal
        double tops[2] = {-INFINITY, -INFINITY};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
          for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              tops[c] = first + 16 * kt + i <= 16 * c ? fmax(tops[c], t[c][kt][i]) : tops[c];
          tops[c] = group_max_f64(tops[c]);
        }
        settle(tops);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          double zt = 0.0;
#pragma unroll
          for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              zt += static_cast<double>(first + 16 * kt + i <= 16 * c ? exp2_clamped(t[c][kt][i] - ref[c]) : 0.f);
          if (tops[c] > -INFINITY) z[c] += zt;   // a tile without a logit over -inf adds nothing
        }
      }
    }
    tile = end;
    keys.resume(end);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const double Z = group_sum_f64(z[c]);
    const int row = row0 + 16 * c + r16;
    if (q4 == 0 && row < L) {
      const size_t o = (static_cast<size_t>(b) * a.Hq + h) * a.Lmax + row;
      a.row_M[o] = ref[c] + log2(Z);
      a.row_Z[o] = ref[c];
    }
  }
}

template <int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2)))
void h2o_cols_i8_kernel(H2oArgs a) {
  using Tile = StreamTile<D>;
  constexpr int kKeys = 32 * WAVES;
  int kb, h, b;
  h2o_unit(a, kb, h, b);                                    // first keys first: the most queries
  if (b >= a.B || kb >= a.n_ranks) return;
  const int L = a.L[b], nt = (L + kT - 1) / kT;
  if (kb * kKeys >= L) return;
  const int g = h / (a.Hq / a.Hkv);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q4 = lane >> 4, r16 = lane & 15;
  const size_t hrow = (static_cast<size_t>(b) * a.Hq + h) * a.Lmax;
  const uint16_t* qh = static_cast<const uint16_t*>(a.q) + hrow * D;
  const uint16_t* kg = static_cast<const uint16_t*>(a.k) + (static_cast<size_t>(b) * a.Hkv + g) * a.Lmax * D;
  const int key0 = kb * kKeys + 32 * wave;
  const int t_lo = kb * kKeys / kT, w_lo = key0 < L ? key0 / kT : nt;      // first tiles

  __shared__ Tile s_tile[Stager<D, WAVES>::kBuffers];
  // log-sum-exps of a tile's rows, for the digit path, at most kLseMax (a logit
  // there is under 2^28, so the term is 0, and its exponent stays within int:
  // another key may take a row's log-sum-exp past 2^31)
  constexpr double kLseMax = 0x1p30;
  static_assert(Stager<D, WAVES>::kTwo, "a tile's values are written while the one before is read");
  __shared__ double s_lse[2][kT];
  __shared__ double s_ref[kT], s_inv[kT];                   // of the first tile's rows: reference, 2^(ref - lse)
  Stager<D, WAVES> rows{qh, L, nt, wave, lane};
  rows.start(t_lo);
  Stationary<D> sx;
  const uint16_t* col[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) col[c] = kg + static_cast<size_t>(min(key0 + 16 * c + r16, L - 1)) * D;
  sx.load(col, q4);
  const double cd = a.scale * 1.4426950408889634;
  __shared__ float2 s_uv[WAVES];
  rows.share(s_uv, sx.U, sx.V, static_cast<float>(cd));
  const double cu[2] = {static_cast<double>(sx.unit[0]) * (cd * 0x1p16),
                        static_cast<double>(sx.unit[1]) * (cd * 0x1p16)};

  // log-sum-exp of row tid of a tile, fetched a tile ahead; rows past the
  // prompt: so large that their terms vanish
  auto fetch_lse = [&](int tile) {
    const int row = tile * kT + tid;
    return tid < kT && row < L ? a.row_M[hrow + row] : kLseMax;
  };
  double lse = fetch_lse(t_lo), sum[2] = {0.0, 0.0};
  if (kb == 0 && tid < kT) {
    const double ref = tid < L ? fmin(a.row_Z[hrow + tid], kLseMax) : kLseMax;
    s_ref[tid] = ref;
    s_inv[tid] = exp2(ref - lse);
  }
  for (int tile = t_lo, end; tile < nt;) {
    const int buf = (tile - t_lo) & 1;
    if (tid < kT) s_lse[buf][tid] = lse > kLseMax ? kLseMax : lse;           // NaN stays
    lse = fetch_lse(tile + 1);
    const Tile* st = rows.look(s_tile, tile, t_lo, nt, end);                 // its barrier covers the rows' values too
    const int rbase = tile * kT;
    const bool edge = rbase < key0 + 31;                    // some rows come before the keys
    if (st && tile < w_lo) {                                // wave-uniform
      ++tile;
      continue;
    }
    if (st) {
      auto pass = [&](auto kind) {
        constexpr int kKind = decltype(kind)::value;
        auto use = [&](int kt, int c, const i32x4 (&S)[kSums]) {
          const double f = st->grp[Tile::group_of(kt, q4)].x * cu[c];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = 16 * kt + 4 * q4 + i;
            const float p = exp2_short(fma(digit_value(S, i), f, kKind == kFirst ? -s_ref[r] : -s_lse[buf][r]));
            double x = kKind == kFirst ? static_cast<double>(p) * s_inv[r] : static_cast<double>(p);
            if constexpr (kKind != kPlain) x = rbase + r >= key0 + 16 * c + r16 ? x : 0.0;
            sum[c] += x;
          }
        };
        if constexpr (kKind == kFirst) stepwise_products<D>(*st, sx, q4, r16, use);
        else                           pipelined_products<D>(*st, sx, q4, r16, use);
      };
      if (tile == 0) pass(std::integral_constant<int, kFirst>());
      else if (edge) pass(std::integral_constant<int, kMasked>());
      else           pass(std::integral_constant<int, kPlain>());
      ++tile;
      continue;
    }
    const int lo = max(tile, w_lo);
    if (lo < end) {
      F64Tiles<D> f64(qh, L, col, q4, r16, cd, lo);
      for (int u = lo; u < end; ++u) {
        f64x4 t[2][4];
        f64.products(u, t);
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = u * kT + 16 * kt + 4 * q4 + i;
            const double o = a.row_M[hrow + min(r, L - 1)];
#pragma unroll
            for (int c = 0; c < 2; ++c)
              if (r < L && r >= key0 + 16 * c + r16) sum[c] += static_cast<double>(exp2_clamped(t[c][kt][i] - o));
          }
      }
    }
    tile = end;
    lse = fetch_lse(end);
    rows.resume(end);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const double s = group_sum_f64(sum[c]);
    const int key = key0 + 16 * c + r16;
    if (q4 == 0 && key < L) a.col_part[hrow + key] = s;
  }
}

template <int D, int WAVES>
hipError_t launch_w(H2oArgs a, int lmax, hipStream_t st) {
  a.n_ranks = (lmax + 32 * WAVES - 1) / (32 * WAVES);
  const int units = a.n_ranks * a.B * a.Hkv;                // (rank, batch, KV head)
  const dim3 grid(((units + 7) / 8) * 8 * (a.Hq / a.Hkv));
  h2o_rows_i8_kernel<D, WAVES><<<grid, 64 * WAVES, 0, st>>>(a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  h2o_cols_i8_kernel<D, WAVES><<<grid, 64 * WAVES, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_h2o_passes_bf16(const H2oArgs& a, int d, hipStream_t st) {
  int lmax = 0;
  long long blocks = 0;                      // of 256 rows
  for (int b = 0; b < a.B; ++b) {
    lmax = max(lmax, a.L[b]);
    blocks += static_cast<long long>((a.L[b] + 255) / 256) * a.Hq;
  }
  // 8 waves share one staging and fill a CU; under one round of such blocks
  // half of them a block spreads the rows over twice the CUs
  if (blocks >= 256) return d == 128 ? launch_w<128, 8>(a, lmax, st) : launch_w<64, 8>(a, lmax, st);
  return d == 128 ? launch_w<128, 4>(a, lmax, st) : launch_w<64, 4>(a, lmax, st);
}

}  // namespace tb
