// Host-side rules of the dispatch: plain arithmetic on sizes and weights,
// without HIP, so that they can be compiled and checked on any host.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>

namespace xc {

// The softmax scale 1 / sqrt(d) in log2 units; bf16 models fold it into the
// stored queries.
inline float softmax_scale(int D) { return 1.4426950408889634f / sqrtf((float)D); }

// Upper bound of |q . k| / sqrt(d) in log2 units from the RMSNorm gains: a
// normalised head vector has norm at most sqrt(d), so |q . k| <= d max_i
// |gq_i gk_i|; a rotation mixes the dimensions of a pair, so the maximum then
// is taken per pair.  2% cover the rounding of q and k to bf16 (2^-8 each).
// Infinity where a gain is not finite.
inline float qk_score_bound(const float* gq, const float* gk, int D, bool rope) {
  const int step = rope ? 2 : 1;
  float most = 0.f;
  for (int i = 0; i + step <= D; i += step) {
    float a = 0.f, b = 0.f;
    for (int j = i; j < i + step; ++j) {
      if (!std::isfinite(gq[j]) || !std::isfinite(gk[j])) return INFINITY;
      a = std::max(a, std::fabs(gq[j]));
      b = std::max(b, std::fabs(gk[j]));
    }
    most = std::max(most, a * b);
  }
  return 1.02f * (float)D * softmax_scale(D) * most;
}

// Upper bound of an affine map's outputs |w_r . h + b_r| over its rows r:
// `norm` the largest 2-norm of a row, `bias` the largest |b_r|.  Rows with a
// non-finite element make it infinite or NaN, which no rule accepts.
struct RowBound {
  double norm = 0, bias = 0;
};

// Largest |v| of a self-attention: v = Wv h + bv with h = LN(x) (1 + scale) +
// shift, |LN(x)|_2 <= sqrt(C); the modulations are rows of W_ada SiLU(c) +
// b_ada with |c_k| <= cond_max (at least 1, the timestep embedding), Dc
// entries.  1% per factor covers the bf16 roundings.
inline double self_value_bound(const RowBound& mod, const RowBound& v, int C, int Dc, double cond_max) {
  const double m = 1.01 * (mod.norm * std::sqrt((double)Dc) * cond_max + mod.bias);
  return 1.01 * (v.norm * 1.01 * std::sqrt((double)C) * (1 + 2 * m) + v.bias);
}

// ... and of a cross-attention over condition tokens with |cond| <= cond_max.
inline double cross_value_bound(const RowBound& v, int C, double cond_max) {
  return 1.01 * (v.norm * 1.01 * std::sqrt((double)C) * cond_max + v.bias);
}

// Attention without a running maximum (attn_bounded_kernel): probabilities are
// 2^s, |s| <= score_bound (log2 units), values at most value_bound, and
// numerator and denominator carry the same relative errors as with a maximum
// subtracted as long as neither leaves the range of a float.
// * score_bound <= 64: sums of probabilities do not.  Gains of 1 give 16.6 (d =
//   128), gain products over 3.8 pass 64.
// * the sum over Lk keys of 2^s |v| stays below 2^120, so no partial sum
//   overflows where the running maximum (p <= 2^8) would not;
// * the smallest products that matter, 2^-s |v| 2^-24, stay above 2^-126 for
//   values down to 2^-10 of their bound (4 - 200 times what models store).
// Ordinary models are far from both (|v| of 2^10, 48384 keys: 2^42 at a bound
// of 16.6).  False for a bound that is NaN or infinite.
inline bool attention_bounded(float score_bound, double value_bound, long long Lk) {
  const double values = std::log2(value_bound);
  return score_bound <= 64.0f && score_bound + std::log2((double)Lk) + values <= 120.0 && score_bound - values <= 92.0;
}

// Whether the kernel without a running maximum (four waves of 64 queries) is the
// faster one for L queries over Lk keys, `items` (head, 256-query) items on
// `cus` CUs; otherwise the running-maximum kernel (eight waves of 32) serves
// them.  Up to 128 queries leave half of the 64-query waves idle, and a wave's
// tile is a longer chain; two key tiles are the running-maximum kernel's
// shortest loop, unless two workgroups of 64 head dims share a CU.  us without
// / with a running maximum:
//   33 queries, 8 heads of 64: 128 keys 8.7 / 8.1, 448 keys 12.6 / 10.9, 1024 keys 12.4 / 11.9
//   128 queries, 8 heads of 128: 64 keys 10.5 / 10.5, 128 keys 12.3 / 11.7, 1024 keys 16.9 / 15.9
//   160 queries, 8 heads of 64: 64 keys 8.2 / 8.8, 192 keys 10.6 / 10.4, 448 keys 13.9 / 13.9
//   9522 queries, 15 heads of 128: 64 keys 37.2 / 37.7, 128 keys 45.9 / 43.8, 192 keys 50.4 / 53.5, 256 keys
//     54.5 / 53.1, 384 keys 63.7 / 62.6, 512 keys 72.4 / 72.2, 2048 keys 178 / 189
//   3245 queries, 16 heads of 64 (208 items): 128 keys 12.4 / 11.9, 256 keys 14.2 / 13.9, 384 keys 16.2 / 16.1
//   7020 queries, 16 heads of 64 (448 items): 128 keys 17.0 / 20.2, 256 keys 21.7 / 24.6
inline bool attention_wide_waves(int L, long long Lk, int D, long long items, int cus) {
  const long long tiles = (Lk + 63) / 64;
  if (L <= 128) return false;
  return tiles != 2 || (D == 64 && items > cus);
}

// Key splits of the bf16 attention (at most `most`) for `items` (head, 256-query)
// items of `tiles` key tiles on `slots` resident workgroups.  Estimated time in
// key-tile steps (1.2 us at 128 head dims, 0.8 at 64): rounds * (tiles per unit +
// 4 for the unit's prologue and epilogue) + 1.5 + 5 S items / slots for the
// merge, over S <= 16 with at least 2 tiles each.  Up to 7 tiles stay whole: a
// split gains at most 1.3 us there and a skipped block would pay 1.8 for the
// merge's launch.  us with 1 / 2 / 3 / 4 / 5 / 8 splits:
//   128 dims, 24 items: 7 tiles 21.1 / 20.9 / 20.1 / 19.5 / 20.4 / -, 8 tiles 22.1 / 21.1 / 20.2 / 19.5 / 20.2 / 19.1
//   128 dims, 64 items: 8 tiles 23.1 / 22.2 / 22.3 / 23.5 / 31 / 34, 12 tiles 27.2 / 24.9 / 24.0 / 24.9 / 36 / 38
//   128 dims, 112 items: 8 tiles 25.2 / 27.1 / 38, 12 tiles 30.7 / 30.2 / 42, 16 tiles 36.6 / 33.5 / 47
//   64 dims, 24 items: 8 tiles 15.7 / 15.6 / 15.3 / 15.2 / 15.6 / 16.0, 16 tiles 22.1 / 18.8 / 17.7 / 16.9 / 17.3 / 17.7,
//     48 tiles - / 31.7 / 26.2 / 23.9 / 22.6 / 21.6 (10: 21.8, 12: 27.1)
inline int attention_split_count(long long items, long long tiles, long long slots, long long most) {
  int best = 1;
  double best_cost = 1e300;
  for (int s = 1; s <= 16 && (s == 1 || (tiles >= 8 && tiles / s >= 2 && s <= most)); ++s) {
    const long long rounds = (items * s + slots - 1) / slots;
    const double cost = (double)rounds * ((double)tiles / s + 4.0) + (s > 1 ? 1.5 + 5.0 * s * items / slots : 0.0);
    if (cost < best_cost - 1e-9) {
      best_cost = cost;
      best = s;
    }
  }
  return best;
}

// Tile of a bf16 M x N x K product on `cus` CUs.  Times are estimated in
// microseconds as rounds * (fixed + K / 64 * stage); fixed holds the launch, the
// first stage's latency and the epilogue, the QKV product's longer one has
// constants of its own.  Fitted to launches of every tile over 470 models of 200
// to 16000 tokens, hidden 128 to 2560 and MLP 128 to 10240, with and without
// rotation: 0.3% (QKV) and 0.7% (others) over the fastest tile on average, no
// product over 1.5% slower than on the 32-deep two-workgroup kernel that these
// tiles replaced.  Small tiles run one workgroup per CU with a deep ring or two
// with a shallow one; a shallow 64 x 128 tile with its CU to itself takes its own
// line.
//   768 x 512 x 2048: 64 x 64 13.2 us, 64 x 128 15.5, 128 x 128 deep 20.9
//   3240 x 1024 x 4096: 64 x 128 43.6, 128 x 128 deep 40.6, 192 x 128 57.9
//   8370 x 1024 x 256: 128 x 128 17.5, 192 x 128 15.0, 256 x 256 17.8
//   7020 x 1536 x 6144: 128 x 128 deep 168, 192 x 128 140, 192 x 256 131, 256 x 256 156
//   12096 x 2048 x 8192: 192 x 128 379, 192 x 256 360, 256 x 256 410
//   QKV 13260 x 384 x 128: 64 x 128 13.7, 128 x 128 11.4, 192 x 128 deep 13.7, 192 x 128 13.0
//   QKV 14100 x 768 x 256, rotated: 64 x 128 27.6, 192 x 128 24.8, 256 x 256 30.4, 192 x 256 26.1
//   QKV 5820 x 4992 x 1664, rotated: 128 x 128 135, 192 x 128 deep 155, 192 x 128 129
//   QKV 7020 x 4608 x 1536: 192 x 128 114, 256 x 256 102, 192 x 256 113
struct GemmTile {
  int id, bm, bn, per_cu;
  double fixed, stage, qkv_fixed, qkv_stage;
};
enum TileId { kT64x64, kT64x128, kT128x128deep, kT128x128, kT192x128deep, kT192x128, kT256x256, kT192x256 };
constexpr GemmTile kGemmTiles[] = {
    {kT64x64, 64, 64, 1, 6.5, 0.24, 0, 0},
    {kT64x128, 64, 128, 1, 6.0, 0.31, 6.0, 0.31},
    {kT64x128, 64, 128, 2, 7.5, 0.58, 6.75, 0.60},
    {kT128x128deep, 128, 128, 1, 8.5, 0.48, 9.5, 0.48},
    {kT128x128, 128, 128, 2, 9.5, 0.93, 9.75, 1.10},
    {kT192x128deep, 192, 128, 1, 11.25, 0.69, 14.0, 0.87},
    {kT192x128, 192, 128, 2, 12.0, 1.34, 12.25, 1.38},
    {kT256x256, 256, 256, 1, 12.0, 1.50, 12.0, 1.62},
    {kT192x256, 192, 256, 1, 14.0, 1.20, 14.0, 1.26},
};

// C: columns of each of q, k, v for the QKV epilogue (0: another epilogue)
inline int pick_tile(int M, int N, int K, int C, int cus) {
  int best = kT64x128;
  double best_us = 1e300;
  for (const GemmTile& t : kGemmTiles) {
    if (N % t.bn != 0) continue;
    // a QKV tile lies in one of q, k, v, its waves hold 64 columns
    if (C != 0 && (C % t.bn != 0 || t.id == kT64x64)) continue;
    const long long tiles = (long long)((M + t.bm - 1) / t.bm) * (N / t.bn), slots = (long long)cus * t.per_cu;
    const double fixed = C != 0 ? t.qkv_fixed : t.fixed, stage = C != 0 ? t.qkv_stage : t.stage;
    const double us = (double)((tiles + slots - 1) / slots) * (fixed + K / 64 * stage);
    if (us < best_us) {
      best_us = us;
      best = t.id;
    }
  }
  return best;
}

// Tile (16, 32 or the staged 64 square) of a float32 M x N x K product with
// 16-byte rows on `cus` CUs.  Every tile re-reads its operands, so the tiles grow
// with the product; a long K makes the 16-square ones re-read more.  us with 16 /
// 32 / 64 by the number of 16-square tiles (256 CUs):
//   K = 1024: 256 9.3 / 15.2 / 145, 512 12.4 / 15.0 / 140, 704 17.0 / 15.4 / 141, 832 19.7 / 15.7 / 119, 1104
//     23.3 / 25.6 / 140, 2048 34.0 / 26.6 / 141
//   K = 256: 512 6.8 / 8.2 / 39, 704 7.7 / 8.2 / 41, 1104 9.6 / 10.1 / 42, 1536 10.1 / 9.5 / 41, 2048 12.6 / 10.4 / 42
//   K = 128: 1056 7.1 / 7.9 / 22, 1408 8.8 / 8.9 / 22, 2048 9.6 / 8.7 / 23
//   8448 x K 1024: 121 / 93 / 145, 12288 x 1536: 261 / 202 / 262, 16384 x 1024: 232 / 180 / 192, 18432 x 768: 196 /
//     151 / 145, 24576 x 1024: 343 / 255 / 221
inline int gemm_f32_tile(int M, int N, int K, int cus) {
  const long long t16 = (long long)((M + 15) / 16) * ((N + 15) / 16);
  return t16 <= (K >= 512 ? 2 : 6) * (long long)cus ? 16 : t16 <= 64ll * cus ? 32 : 64;
}

// Waves of a float32 attention workgroup (one query of one head): no more than
// the keys have 64-key chunks, the others would only cost the launch (3000
// queries, 8 heads of 32, 20 keys: four waves 54.2 us, one 27.1; 4096 queries, 2
// heads of 32, 65 keys: four 28.9, two 26.6; 200 queries, 800 keys: one 104, four 33).
inline int attention_f32_waves(long long Lk) { return Lk <= 64 ? 1 : Lk <= 128 ? 2 : 4; }

// Rows of W_ada per wave in adaln_flat_kernel, 8 or 32, for `rows` rows of
// `chunks` 16-byte chunks.  32 amortise a wave's fixed work but need many rows
// to fill the chip, and 32 lanes then sum rows that lie `chunks` words apart in
// LDS: multiples of 8 meet in few banks, and long rows leave few workgroups a
// CU.  HIP events, us with 8 / 32 rows per wave:
//   33 chunks (272 bf16): 49152 rows 10.3 / 11.1, 61440 11.6 / 11.7, 73728 13.5 / 12.8, 98304 15.5 / 13.9
//   18 chunks (72 float): 49152 rows 7.8 / 8.3, 61440 8.6 / 8.6, 98304 12.0 / 9.8, 368640 30.3 / 24.2
//   147456 rows: 24 chunks 16.9 / 14.8, 30 19.6 / 16.9, 32 21.7 / 26.7, 40 20.1 / 21.2, 42 21.3 / 20.9,
//     50 24.9 / 23.6, 56 26.4 / 29.2, 64 36.6 / 51.3, 128 65.9 / 103
inline int adaln_wave_rows(long long rows, int chunks) {
  const bool spread = chunks <= 24 || (chunks <= 50 && chunks % 8 != 0);
  return rows >= 60 * 1024 && spread ? 32 : 8;
}

}  // namespace xc
