// K1 of the observation-window scoring for bf16 inputs: the softmax numerators
// of every (window row, key) pair, on the int8 matrix cores (exact_dot.h).
//
// Block = 1, 2, 4 or 8 waves of 32 window rows of one KV head (chunks of 256
// rows past that) over a run of consecutive 64-key tiles.  A wave converts its
// rows to digit planes once and keeps them in registers; each tile's keys are
// read from HBM once per block (one tile ahead, into registers), converted by
// all waves, those without rows included, and shared through LDS.
// Per 16-key step a wave computes 13 digit products for each of its two 16-row
// column tiles, recombines them to the logit (base-2 units) in float64, splits
// it as t = n + f and takes 2^f in fp32.  Keys are the MFMA rows, so a lane
// holds 16 keys of one window row.  e is 2^(t - ref) with an integer reference
// (only the exponent shifts), taken from the tile before, so e is stored step
// by step and no logit waits in registers for the tile's maximum; a tile that
// the reference does not fit is redone.  Stores e (fp32, float4 of 4
// consecutive keys, laid out [tile][16-key step][row][16]) and per (tile, row)
// the reference in logit units (-inf where the row sees no key of the tile, or
// none over -inf: the tile then counts nowhere) and the sum.
// A tile that the digits cannot hold takes float64 products (F64Tiles), its own
// largest logit as the reference.

#include <type_traits>

#include "exact_dot.h"
#include "kernels.h"

namespace tb {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4n;
constexpr int kT = kScoreTile;
constexpr int kNone = -(1 << 29);            // n of a masked logit
// A tile's reference is the row's largest n of the tile before; it stands
// while the tile's own largest n lies kRefLow .. kRefLow + kRefSpan above it
// (e between 2^-102 of the largest and 2^60 keeps its fp32 precision).
constexpr int kRefLow = -24, kRefSpan = 84;

template <int D, int WAVES, bool STREAM>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2)))
void score_tiles_i8_kernel(ScoreArgs a) {
  using Tile = StreamTile<D>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q4 = lane >> 4, r16 = lane & 15;
  // block -> (sequence, KV head, row chunk, run of tiles)
  int b = 0;
  while (b + 1 < a.B && static_cast<int>(blockIdx.x) >= a.blk_off[b + 1]) ++b;
  const int L = a.L[b], nt = (L + kT - 1) / kT;
  const int runs = (nt + a.run - 1) / a.run;
  const int idx = static_cast<int>(blockIdx.x) - a.blk_off[b];
  const int unit = idx / runs;
  const int t_lo = (idx % runs) * a.run, t_hi = min(t_lo + a.run, nt);
  const int g = unit / a.row_chunks, row0 = (unit % a.row_chunks) * kScoreRows + 32 * wave;
  const int G = a.Hq / a.Hkv, R = a.R, w = a.w;
  const size_t bg = static_cast<size_t>(b) * a.Hkv + g;
  const uint16_t* kg = static_cast<const uint16_t*>(a.k) + bg * a.Lmax * D;
  const bool active = row0 < R;              // wave-uniform

  __shared__ Tile s_tile[Stager<D, WAVES>::kBuffers];
  Stager<D, WAVES> keys{kg, L, nt, wave, lane};
  keys.start(t_lo);

  Stationary<D> sx;
  int row[2];                                // padding rows repeat row R - 1
  const uint16_t* col[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    row[c] = min(row0 + 16 * c + r16, R - 1);
    col[c] = static_cast<const uint16_t*>(a.q_win) +
             ((static_cast<size_t>(b) * a.Hq + g * G + row[c] / w) * w + row[c] % w) * D;
  }
  sx.load(col, q4);
  const double cd = a.scale * 1.4426950408889634;           // exp(x) = 2^(x log2 e)
  const double cu[2] = {static_cast<double>(sx.unit[0]) * (cd * 0x1p16),
                        static_cast<double>(sx.unit[1]) * (cd * 0x1p16)};
  __shared__ float2 s_uv[WAVES];
  keys.share(s_uv, sx.U, sx.V, static_cast<float>(cd));

  if (!active) {                             // waves without rows only stage
    for (int tile = t_lo, end; tile < t_hi;) {
      if (keys.look(s_tile, tile, t_lo, t_hi, end)) {
        ++tile;
      } else {
        tile = end;
        keys.resume(end);
      }
    }
    return;
  }

  // Every lane stores, the same count on every path: the four lane groups hold
  // the same sum, and padding rows are copies of row R - 1.  So a wait for the
  // keys fetched before the stores need not wait for the stores.
  auto store_e = [&](int tile, int c, int kt, const float (&e)[4]) {
    const f32x4n x = {e[0], e[1], e[2], e[3]};
    const size_t te = (bg * a.n_tiles + tile) * R;
    uint32_t off = (row[c] * 16 + 4 * q4) * 4;
    asm volatile("" : "+v"(off));            // added here, not once per step ahead of the loop
    f32x4n* p = reinterpret_cast<f32x4n*>(
        reinterpret_cast<char*>(a.e + (te * 4 + static_cast<size_t>(kt) * R) * 16) + off);
    if constexpr (STREAM) __builtin_nontemporal_store(x, p);
    else                  *p = x;
    return static_cast<double>((e[0] + e[1]) + (e[2] + e[3]));
  };
  auto store_stats = [&](int tile, const double (&m)[2], const double (&z)[2]) {
    const size_t te = (bg * a.n_tiles + tile) * R;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      uint32_t mo = row[c] * 8;
      asm volatile("" : "+v"(mo));
      *reinterpret_cast<double*>(reinterpret_cast<char*>(a.tile_m + te) + mo) = m[c];
      *reinterpret_cast<double*>(reinterpret_cast<char*>(a.tile_z + te) + mo) = group_sum_f64(z[c]);
    }
  };
  // last key of a tile that the lane's rows see, from the lane's first key on
  auto limits = [&](int tile, int (&lim)[2]) {
    const int kbase = tile * kT;
    const bool edge = kbase + kT > L - w;                   // some rows do not see all 64 keys
#pragma unroll
    for (int c = 0; c < 2; ++c) lim[c] = edge ? min(L - 1, L - w + row[c] % w) - kbase - 4 * q4 : 63;
    return edge;
  };

  int ref[2] = {0, 0};                       // of this lane's rows, base-2 units
  for (int tile = t_lo, end; tile < t_hi;) {
    const Tile* st = keys.look(s_tile, tile, t_lo, t_hi, end);
    int lim[2];
    if (st) {
      const bool edge = limits(tile, lim);
      double m[2], z[2] = {0.0, 0.0};
      // false: a reference did not fit, and has been set
      auto pass = [&](auto masked) -> bool {
        asm volatile("" ::: "memory");       // no operand is read ahead of the pass
        int top[2] = {kNone, kNone};
        z[0] = z[1] = 0.0;
        pipelined_products<D>(*st, sx, q4, r16, [&](int kt, int c, const i32x4 (&S)[kSums]) {
          const double f = st->grp[Tile::group_of(kt, q4)].x * cu[c];
          float e[4];
          int n[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double v = digit_value(S, i);
            // the sum with 1.5 2^52 holds round(t), t = v f, in its low word
            // (|t| < 2^28 here)
            const double y = fma(v, f, 0x1.8p52);
            n[i] = static_cast<int>(static_cast<uint32_t>(__double_as_longlong(y)));
            e[i] = ldexpf(__builtin_amdgcn_exp2f(static_cast<float>(fma(v, f, 0x1.8p52 - y))), n[i] - ref[c]);
          }
          if constexpr (decltype(masked)::value) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const bool ok = 16 * kt + i <= lim[c];
              n[i] = ok ? n[i] : kNone;
              e[i] = ok ? e[i] : 0.f;
            }
          }
          top[c] = max(max(top[c], max(n[0], n[1])), max(n[2], n[3]));
          z[c] += store_e(tile, c, kt, e);
        });
        bool bad = false;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int t = static_cast<int>(group_all(static_cast<uint32_t>(top[c]), IMax()));
          const int over = t == kNone ? 0 : t - ref[c];
          m[c] = t == kNone ? -INFINITY : static_cast<double>(ref[c]) * 0.69314718055994530942;
          ref[c] += over;                    // the next tile's reference
          bad = bad || over > kRefLow + kRefSpan || over < kRefLow;
        }
        return __builtin_amdgcn_ballot_w64(bad) == 0;
      };
      // the masked pass serves the last tiles and (twice at most) a reference
      // that does not fit
      bool done = !edge && pass(std::false_type());
      while (!done) done = pass(std::true_type());
      store_stats(tile, m, z);
      ++tile;
      continue;
    }
    // float64 products; the reference is the tile's own largest logit
    F64Tiles<D> f64(kg, L, col, q4, r16, cd, tile);
    for (; tile < end; ++tile) {
      limits(tile, lim);
      f64x4 t[2][4];
      f64.products(tile, t);
      double m[2], z[2] = {0.0, 0.0};
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        double top = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) top = 16 * kt + i <= lim[c] ? fmax(top, t[c][kt][i]) : top;
        top = group_max_f64(top);
        m[c] = top * 0.69314718055994530942;
        const double r = top == -INFINITY ? 0.0 : top;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
          float e[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) e[i] = 16 * kt + i <= lim[c] ? exp2_clamped(t[c][kt][i] - r) : 0.f;
          z[c] += store_e(tile, c, kt, e);
        }
      }
      store_stats(tile, m, z);
    }
    keys.resume(end);
  }
}

template <int D, int WAVES>
void launch_w(const ScoreArgs& a, int blocks, hipStream_t st) {
  if (a.stream_e) score_tiles_i8_kernel<D, WAVES, true><<<blocks, 64 * WAVES, 0, st>>>(a);
  else            score_tiles_i8_kernel<D, WAVES, false><<<blocks, 64 * WAVES, 0, st>>>(a);
}

template <int D>
hipError_t launch_d(const ScoreArgs& a, int blocks, int waves, hipStream_t st) {
  switch (waves) {
    case 8:  launch_w<D, 8>(a, blocks, st); break;
    case 4:  launch_w<D, 4>(a, blocks, st); break;
    case 2:  launch_w<D, 2>(a, blocks, st); break;
    default: launch_w<D, 1>(a, blocks, st); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_score_tiles_bf16(const ScoreArgs& args, int d, hipStream_t st) {
  ScoreArgs a = args;
  int waves = 1;
  while (waves < 8 && 32 * waves < a.R) waves *= 2;
  // Two waves per SIMD fit a CU (registers), so 8 / waves blocks, up to 4
  // (LDS: 64 KB for 4 or 8 waves, 32 KB below).  One round of blocks over the
  // chip, each taking a run of tiles as long as that needs, since a block
  // first converts its rows.
  const int per_cu = waves >= 2 ? 8 / waves : 4;
  long long total = 0;
  for (int b = 0; b < a.B; ++b) total += (a.L[b] + kT - 1) / kT;
  total *= static_cast<long long>(a.Hkv) * a.row_chunks;
  a.run = static_cast<int32_t>((total + 256 * per_cu - 1) / (256 * per_cu));
  int blocks = 0;
  for (int b = 0; b < a.B; ++b) {
    a.blk_off[b] = blocks;
    const int nt = (a.L[b] + kT - 1) / kT;
    blocks += (nt + a.run - 1) / a.run * a.Hkv * a.row_chunks;
  }
  return d == 128 ? launch_d<128>(a, blocks, waves, st) : launch_d<64>(a, blocks, waves, st);
}

}  // namespace tb
