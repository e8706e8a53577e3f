// Observation-window scoring: softmax of the last w queries against all
// prompt keys, summed per KV head over the G*w window rows, then max-pooled.
//
// Precision.  The selection that follows is compared position by position, so
// scores are kept to ~1e-7 relative: dot products of the (exact) bf16/fp32
// inputs are accumulated in float64, exponent arguments are reduced in float64,
// and sums are float64.  The per-logit exponentials (fp32, within ~1.5e-7
// relative) and the raw scores (fp32 rounding, 6e-8) are the only
// single-precision values; pooling is a max, so it is exact.
//
// Four kernels, all with fixed-order reductions (no atomics):
//   K1 score_tiles: the softmax numerators e = exp(s - m) (fp32) of every
//      (window row, key) with a reference m per (row, 64-key tile), and
//      z = sum e.  bf16: exact digit products on the int8 matrix cores
//      (score_tiles_bf16.hip; traced, L = 131072, 8 KV heads, 256 rows: 434 us
//      against 1288 with float64 products, L = 8192, 4 KV heads, 224 rows: 24
//      against 47).  fp32 (below): block = (64-key tile, <= 256 window rows) of
//      one KV head, 512 threads; wave w owns 32 rows x the 64 keys (waves
//      whose rows are all padding skip the products).  With 4, 6 or 7 row
//      pairs and enough blocks, a block instead takes 8 consecutive units (32
//      rows x one tile, numbered tile-major) over at most two tiles, so no
//      wave idles.  Window queries (as fp32) and keys (as float64, converted
//      once since every wave reads them) are staged in LDS in 32-wide d
//      chunks, the next chunk's global loads in flight while the current one
//      is multiplied; the products run on the float64 matrix cores
//      (v_mfma_f64_16x16x4_f64, 2 x 4 tiles of 16 x 16 per wave).  Each row's
//      64 logits sit in one 16-lane DPP row, so the causal mask, m (the row's
//      largest dot product rounded to fp32) and z need no LDS.
//   K2 row_stats: each window row's global max M and normaliser Z from its
//      tiles' (m, z).
//   K3 score_accum: block = 64 prefix columns; A[j] = sum_r e[r][j] *
//      exp(m[r][tile] - M[r]) / Z[r] in float64 (four row groups, four
//      independent accumulators each, combined in a fixed order); raw A as fp32.
//   K4 pool: max of the raw scores over |j - j'| <= pool/2 within the prefix
//      (or their mean with zeros outside the prefix and divisor pool, summed in
//      float64, for the average-pool variant).
//
// The per-logit exponential is the one place fp64 arithmetic is avoided: K1's
// epilogue reduces the argument in fp64 (exactly) and evaluates 2^f for
// |f| <= 1/2 in fp32.

#include "exact_dot.h"
#include "kernels.h"

namespace tb {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4n;

constexpr int kThreads = 256;
constexpr int kT = kScoreTile;     // keys per tile (64)
constexpr int kRows = kScoreRows;  // rows per block (256)
constexpr int kDC = 32;            // d chunk staged in LDS

__device__ __forceinline__ void load8(const float* p, float* out) {
  Elem<float>::widen(ldg16(p), out);
  Elem<float>::widen(ldg16(p + 4), out + 4);
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t u = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u & 0xffffffffu), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double((static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) |
                              static_cast<uint32_t>(lo));
}
// Sum over the 16 lanes of a DPP row; every lane gets the result, in a fixed
// order (deterministic).
__device__ __forceinline__ double row16_sum_f64(double x) {
  x += dpp_f64<kDppQuadXor1>(x);
  x += dpp_f64<kDppQuadXor2>(x);
  x += dpp_f64<kDppRowHalfMirror>(x);
  x += dpp_f64<kDppRowMirror>(x);
  return x;
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row16_max_f32(float x) {
  x = fmaxf(x, dpp_f32<kDppQuadXor1>(x));
  x = fmaxf(x, dpp_f32<kDppQuadXor2>(x));
  x = fmaxf(x, dpp_f32<kDppRowHalfMirror>(x));
  x = fmaxf(x, dpp_f32<kDppRowMirror>(x));
  return x;
}

constexpr int kTilesThreads = 512;
constexpr int kWaveRows = 32;      // window rows per wave in score_tiles

// Work unit of a wave: 32 window rows x one 64-key tile.  NS = 1: block =
// (tile, 256-row chunk), wave w takes rows 32 w .. 32 w + 31 (waves past R
// idle).  NS = 2 (R <= 256 with P = ceil(R / 32) row pairs, P in {4, 6, 7}):
// the units are numbered tile-major, u = P t + p, and block j takes units
// 8 j .. 8 j + 7, so every wave has one and the block's units span at most two
// tiles, whose keys it stages together.  With one idle wave per block (R =
// 224) the busiest SIMD of a CU carries as many waves as at R = 256 and the
// block barriers pace every block by it; packing gives each block 8 busy waves.
template <int D, int NS>
__global__ __launch_bounds__(kTilesThreads, 2) void score_tiles_kernel(ScoreArgs a) {
  const int g = blockIdx.y, b = blockIdx.z;
  const int L = a.L[b];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int t0, tile, pair, row0;                       // block's first tile; this wave's unit
  if constexpr (NS == 1) {
    t0 = tile = blockIdx.x / a.row_chunks;
    row0 = (blockIdx.x % a.row_chunks) * kRows;
    pair = wave;
  } else {
    const int P = a.pack_pairs;
    const int u = static_cast<int>(blockIdx.x) * 8 + wave;
    t0 = static_cast<int>(blockIdx.x) * 8 / P;
    tile = u / P;
    pair = u % P;
    row0 = 0;
  }
  if (t0 * kT >= L) return;                       // block-uniform
  const int kbase = tile * kT;
  const int G = a.Hq / a.Hkv, R = a.R, w = a.w;
  const int q4 = lane >> 4, r16 = lane & 15;
  // wave-uniform: the unit has real rows and real keys
  const bool active = row0 + kWaveRows * pair < R && kbase < L;

  __shared__ float qs[kRows][kDC + 1];             // +1: conflict-free column reads
  // Keys staged as float64 (every wave reads them).  Two doubles of padding per
  // 16 rows spread the staging's 8 rows x 4 positions of a half wave over all
  // banks (the rows are permuted, see krow).  Without it, 4-way conflicts:
  // L = 65536, 224 rows, 4 KV heads, traced, 323 -> 301 us.
  __shared__ double s_keys[NS * kT * (kDC + 1) + NS * kT / 8];
  auto ks = [&](int r) { return &s_keys[r * (kDC + 1) + (r >> 4) * 2]; };
  __shared__ int s_lim[kRows];                     // last key a row sees (-1: padding)
  if (tid < kRows) {
    const int r = row0 + tid;
    s_lim[tid] = r < R ? min(L - 1, L - w + r % w) : -1;
  }

  // Staging: two threads per window row (16 elements each) and four threads
  // per key (8 elements each; the first 256 threads when NS = 1).
  const int qrow = tid >> 1, qoff = (tid & 1) * 16;
  const bool qvalid = row0 + qrow < R;
  const float* qsrc = nullptr;
  if (qvalid) {
    const int r = row0 + qrow, h = g * G + r / w, i = r % w;
    qsrc = static_cast<const float*>(a.q_win) + ((static_cast<size_t>(b) * a.Hq + h) * w + i) * D + qoff;
  }
  const int kk = (tid & (NS * 256 - 1)) >> 2, kdp = (tid & 3) * 8;
  // key kk of a tile sits in LDS row 16 (kk % 4) + kk / 4, so the product's
  // column r16 of step kt is key 4 r16 + kt: a lane's 4 keys are consecutive
  const int krow = (kk & ~63) | ((kk & 3) << 4) | ((kk & 63) >> 2);
  const bool kvalid = tid < NS * 256 && t0 * kT + kk < L;
  const float* ksrc = static_cast<const float*>(a.k) +
                  ((static_cast<size_t>(b) * a.Hkv + g) * a.Lmax + t0 * kT + kk) * D + kdp;
  float qv[16], kv[8];
  auto fetch = [&](int dc) {
    if (qvalid) {
      load8(qsrc + dc, qv);
      load8(qsrc + dc + 8, qv + 8);
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) qv[e] = 0.f;
    }
    if (kvalid) {
      load8(ksrc + dc, kv);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) kv[e] = 0.f;
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int e = 0; e < 16; ++e) qs[qrow][qoff + e] = qv[e];
    if (tid < NS * 256) {
#pragma unroll
      for (int e = 0; e < 8; ++e) ks(krow)[kdp + e] = static_cast<double>(kv[e]);
    }
  };

  f64x4 acc[2][4];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) acc[rt][kt] = f64x4{0.0, 0.0, 0.0, 0.0};

  fetch(0);
  stage();
  __syncthreads();
#pragma unroll 1
  for (int dc = 0; dc < D; dc += kDC) {
    const bool more = dc + kDC < D;
    if (more) fetch(dc + kDC);                     // in flight during the products
    if (active) {
#pragma unroll
      for (int k4 = 0; k4 < kDC / 4; ++k4) {
        const int dd = 4 * k4 + q4;                // this lane's k index
        double av[2], bv[4];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
          av[rt] = static_cast<double>(qs[kWaveRows * pair + 16 * rt + r16][dd]);
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) bv[kt] = ks((tile - t0) * kT + 16 * kt + r16)[dd];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
          for (int kt = 0; kt < 4; ++kt)
            acc[rt][kt] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[rt], bv[kt], acc[rt][kt], 0, 0, 0);
      }
    }
    __syncthreads();
    if (more) {
      stage();
      __syncthreads();
    }
  }
  if (!active) return;

  // acc[rt][kt][v] = q(row 16 rt + q4 + 4 v) . k(key 4 r16 + kt) of this wave
  // (the float64 16x16x4 product returns rows interleaved: item v of lane l is
  // row l/16 + 4v, column l%16).
  const size_t bg = static_cast<size_t>(b) * a.Hkv + g;
  float* ebase = a.e + (bg * a.n_tiles + tile) * static_cast<size_t>(R) * kT;
  const double c = a.scale * 1.4426950408889634;  // exp(x) = 2^(x log2 e)
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int rl = kWaveRows * pair + 16 * rt + q4 + 4 * v;
      const int lim = s_lim[rl];
      bool ok[4];
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        ok[kt] = kbase + 4 * r16 + kt <= lim;
        mx = fmaxf(mx, ok[kt] ? static_cast<float>(acc[rt][kt][v]) : -INFINITY);
      }
      // reference: the row's largest dot product rounded to fp32 (exact as a
      // double); e and m below use the same value, so any nearby one is as good
      const double md = row16_max_f32(mx);
      const double mdc = md * c;
      float ev[4], zs = 0.f;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        ev[kt] = ok[kt] ? exp2_split(fma(acc[rt][kt][v], c, -mdc)) : 0.f;
        zs += ev[kt];
      }
      const double z = row16_sum_f64(static_cast<double>(zs));
      const int rg = row0 + rl;
      if (rg < R) {
        float* dst = ebase + (static_cast<size_t>(r16 >> 2) * R + rg) * 16 + 4 * (r16 & 3);
        if (a.stream_e) __builtin_nontemporal_store(f32x4n{ev[0], ev[1], ev[2], ev[3]},
                                                    reinterpret_cast<f32x4n*>(dst));
        else            *reinterpret_cast<float4*>(dst) = make_float4(ev[0], ev[1], ev[2], ev[3]);
        if (r16 == 0) {
          const size_t o = (bg * a.n_tiles + tile) * R + rg;
          a.tile_m[o] = md * a.scale;       // -inf when the whole row-tile is masked
          a.tile_z[o] = z;
        }
      }
    }
  }
}

// Global max and normaliser of ROWS rows per block over their tiles: thread
// (phase, row) merges the row's tiles phase, phase + 64, ..., eight at a time,
// then the phases are merged.
constexpr int kStatPhases = 64;
template <int ROWS>
__global__ __launch_bounds__(ROWS * kStatPhases) void row_stats_kernel(ScoreArgs a) {
  const int g = blockIdx.y, b = blockIdx.z;
  const int rr = threadIdx.x % ROWS, ph = threadIdx.x / ROWS;
  const int r = blockIdx.x * ROWS + rr;
  const int nt = (a.L[b] + kT - 1) / kT;
  const size_t bg = static_cast<size_t>(b) * a.Hkv + g;
  const size_t o = bg * a.n_tiles * a.R + min(r, a.R - 1);
  constexpr int kWaves = ROWS * kStatPhases / 64;
  __shared__ double s_m[kWaves][ROWS], s_z[kWaves][ROWS];
  constexpr int kAhead = 8;
  double M = -INFINITY, Z = 0.0;
  for (int t0 = ph; t0 < nt; t0 += kStatPhases * kAhead) {
    double mv[kAhead], zv[kAhead], top = M;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int t = t0 + kStatPhases * k;
      const size_t p = o + static_cast<size_t>(min(t, nt - 1)) * a.R;
      mv[k] = a.tile_m[p];
      zv[k] = a.tile_z[p];
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (t0 + kStatPhases * k >= nt) mv[k] = -INFINITY;
      top = fmax(top, mv[k]);
    }
    if (M != -INFINITY) Z *= exp(M - top);
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
      if (mv[k] != -INFINITY) Z += zv[k] * exp(mv[k] - top);
    M = top;
  }
  const double own = M;
#pragma unroll
  for (int off = ROWS; off < 64; off <<= 1) M = fmax(M, __shfl_xor(M, off));
  if ((threadIdx.x & 63) < ROWS) s_m[threadIdx.x >> 6][rr] = M;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kWaves; ++k) M = fmax(M, s_m[k][rr]);
  Z = own == -INFINITY ? 0.0 : Z * exp(own - M);
#pragma unroll
  for (int off = ROWS; off < 64; off <<= 1) Z += __shfl_xor(Z, off);
  if ((threadIdx.x & 63) < ROWS) s_z[threadIdx.x >> 6][rr] = Z;
  __syncthreads();
  if (ph == 0 && r < a.R) {
    Z = s_z[0][rr];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) Z += s_z[k][rr];
    a.row_M[bg * a.R + r] = M;
    a.row_Z[bg * a.R + r] = Z;
  }
}

// Column sums of one 64-column tile: thread (rg, col), rows r = rg + 4k.
__global__ __launch_bounds__(kThreads) void score_accum_kernel(ScoreArgs a) {
  const int ct = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int L = a.L[b], pref = L - a.w;
  const int j0 = ct * kT;
  if (j0 >= pref) return;
  const int R = a.R;
  const size_t bg = static_cast<size_t>(b) * a.Hkv + g;
  const int tid = threadIdx.x;

  __shared__ double coef[1024];
  __shared__ double part[16][kT];

  for (int r = tid; r < R; r += kThreads) {
    const double m = a.tile_m[(bg * a.n_tiles + ct) * R + r];
    const double M = a.row_M[bg * R + r], Z = a.row_Z[bg * R + r];
    coef[r] = (m != -INFINITY && Z > 0.0) ? exp(m - M) / Z : 0.0;
  }
  __syncthreads();
  // Thread (q, rs) reads the float4 of columns 4 q .. 4 q + 3 from rows rs,
  // rs + 16, ..., eight loads in flight, and keeps four float64 column sums;
  // the 16 row phases are then added in order.
  // (Sixteen loads in flight, issued before the coefficients, measured slower.)
  const int q = tid & 15, rs = tid >> 4;
  const float* et = a.e + (bg * a.n_tiles + ct) * static_cast<size_t>(R) * kT +
                    static_cast<size_t>(q >> 2) * R * 16 + 4 * (q & 3);
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  constexpr int kBatch = 8;
  for (int rb = rs; rb < R; rb += 16 * kBatch) {
    float4 v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int r = rb + 16 * u;
      v[u] = r < R ? *reinterpret_cast<const float4*>(et + static_cast<size_t>(r) * 16)
                   : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int r = rb + 16 * u;
      const double c = r < R ? coef[r] : 0.0;
      s0 = fma(static_cast<double>(v[u].x), c, s0);
      s1 = fma(static_cast<double>(v[u].y), c, s1);
      s2 = fma(static_cast<double>(v[u].z), c, s2);
      s3 = fma(static_cast<double>(v[u].w), c, s3);
    }
  }
  part[rs][4 * q] = s0;
  part[rs][4 * q + 1] = s1;
  part[rs][4 * q + 2] = s2;
  part[rs][4 * q + 3] = s3;
  __syncthreads();
  if (tid < kT) {
    const int j = j0 + tid;
    if (j < pref) {
      double A = part[0][tid];
#pragma unroll
      for (int k = 1; k < 16; ++k) A += part[k][tid];
      a.raw[bg * a.Lmax + j] = static_cast<float>(A);
    }
  }
}

__global__ __launch_bounds__(kThreads) void pool_kernel(ScoreArgs a) {
  const int g = blockIdx.y, b = blockIdx.z;
  const int j = blockIdx.x * kThreads + threadIdx.x;
  const int pref = a.L[b] - a.w;
  if (j >= pref) return;
  const int hp = a.pool / 2;
  const size_t bg = static_cast<size_t>(b) * a.Hkv + g;
  const float* raw = a.raw + bg * a.Lmax;
  const int lo = max(j - hp, 0), hi = min(j + hp, pref - 1);
  if (a.pool_avg) {
    // positions outside the prefix count as zeros; the divisor is always pool
    double sum = 0.0;
    for (int jn = lo; jn <= hi; ++jn) sum += raw[jn];
    a.scores[bg * a.Lmax + j] = static_cast<float>(sum / a.pool);
  } else {
    float mx = raw[j];
    for (int jn = lo; jn <= hi; ++jn) mx = fmaxf(mx, raw[jn]);
    a.scores[bg * a.Lmax + j] = mx;
  }
}

hipError_t launch_tiles_f32(const ScoreArgs& args, int d, hipStream_t st) {
  ScoreArgs a = args;
  // Packed blocks (P = 4, 6 or 7 row pairs: waves would idle, and every run of
  // 8 units spans at most two tiles) when packing lowers the blocks per CU and
  // still leaves two per CU (two resident blocks overlap each other's barriers
  // and staging).  Measured, d = 128, one scoring call, packed against not
  // (us): P = 7, 4 KV heads: L = 32768 174 / 187 (8 -> 7 blocks per CU),
  // 36864 198 / 210, 65536 352 / 369, but 8192 64.0 / 62.5, 16384 107 / 105,
  // 24576 157 / 153, 28672 175 / 169 (blocks per CU unchanged); P = 6:
  // 16384 85.0 / 99.7, 32768 152 / 184, 8192 60.1 / 59.2 (2 -> 2); P = 4:
  // 16384 60.9 / 66.6, 32768 107 / 117, 8192 43.9 / 40.8 (one block per CU).
  constexpr long long kCUs = 256;
  const int P = (a.R + kWaveRows - 1) / kWaveRows;
  const long long units = static_cast<long long>(a.Hkv) * a.B;
  const long long plain = static_cast<long long>(a.n_tiles) * units;
  const long long packed = (static_cast<long long>(P) * a.n_tiles + 7) / 8 * units;
  const bool pack = a.row_chunks == 1 && (P == 4 || P == 6 || P == 7) && packed >= 2 * kCUs &&
                    (packed + kCUs - 1) / kCUs < (plain + kCUs - 1) / kCUs;
  a.pack_pairs = pack ? P : 0;
  if (pack) {
    const dim3 g1((P * a.n_tiles + 7) / 8, a.Hkv, a.B);
    if (d == 128) score_tiles_kernel<128, 2><<<g1, kTilesThreads, 0, st>>>(a);
    else          score_tiles_kernel<64, 2><<<g1, kTilesThreads, 0, st>>>(a);
  } else {
    const dim3 g1(a.n_tiles * a.row_chunks, a.Hkv, a.B);
    if (d == 128) score_tiles_kernel<128, 1><<<g1, kTilesThreads, 0, st>>>(a);
    else          score_tiles_kernel<64, 1><<<g1, kTilesThreads, 0, st>>>(a);
  }
  return hipGetLastError();
}

}  // namespace

size_t score_ws_bytes(int B, int Lmax, int Hkv, int R) {
  const size_t n_tiles = (static_cast<size_t>(Lmax) + kT - 1) / kT;
  const size_t units = static_cast<size_t>(B) * Hkv;
  auto up = [](size_t x) { return (x + 255) & ~size_t(255); };
  size_t bytes = up(units * n_tiles * R * kT * sizeof(float));       // e
  bytes += 2 * up(units * n_tiles * R * sizeof(double));             // tile m, z
  bytes += 2 * up(units * R * sizeof(double));                       // row M, Z
  bytes += up(units * Lmax * sizeof(float));                         // raw scores
  return bytes;
}

hipError_t launch_score(const ScoreArgs& args, int d, bool bf16, hipStream_t st) {
  // Exponentials larger than the 256 MB last-level cache cannot stay there for
  // K3 anyway: write them with streaming stores (at L = 131072, 8 KV heads,
  // 1.07 GB: K3 reads them back in 199 us instead of 223, K1 unchanged);
  // smaller ones are written normally so that K3 finds them cached
  // (streaming them cost ~2 us per call at L = 8192).
  ScoreArgs a = args;
  const double e_bytes = 4.0 * kT * a.R * a.n_tiles * a.Hkv * a.B;
  a.stream_e = e_bytes > 256.0 * (1 << 20);
  hipError_t err = bf16 ? launch_score_tiles_bf16(a, d, st) : launch_tiles_f32(a, d, st);
  if (err != hipSuccess) return err;
  // 8 rows a block keep more CUs busy; past the L2 the half lines they read are
  // fetched twice, and 16 rows (whole lines) win.  Traced, 8 / 16 rows: L = 8192,
  // 4 KV heads of 224 rows 3.9 / 4.8 us, 32768 6.5 / 8.4, 65536 8.2 / 11.2,
  // 131072, 8 heads of 256 rows (67 MB) 24.6 / 21.7.
  const double stat_bytes = 16.0 * a.R * a.n_tiles * a.Hkv * a.B;
  if (stat_bytes <= 32.0 * (1 << 20))
    row_stats_kernel<8><<<dim3((a.R + 7) / 8, a.Hkv, a.B), 8 * kStatPhases, 0, st>>>(a);
  else
    row_stats_kernel<16><<<dim3((a.R + 15) / 16, a.Hkv, a.B), 16 * kStatPhases, 0, st>>>(a);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  const dim3 g3((a.Lmax + kT - 1) / kT, a.Hkv, a.B);
  score_accum_kernel<<<g3, kThreads, 0, st>>>(a);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  const dim3 g4((a.Lmax + kThreads - 1) / kThreads, a.Hkv, a.B);
  pool_kernel<<<g4, kThreads, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace tb
