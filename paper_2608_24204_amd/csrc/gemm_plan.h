// Which kernel runs a product C[M, N] = A[M, K] x W[N, K]^T of nt activation terms, in
// which shape and in how many K ranges.  Host code alone (no HIP), so that a test can
// evaluate the rules.
#pragma once
#include <algorithm>
#include <cstddef>

namespace wici {

enum GemvEpi { GEMV_STORE = 0, GEMV_RESID = 1, GEMV_SWIGLU = 2, GEMV_ARGMAX = 3, GEMV_QKV = 4 };

// Weight storage (the values of the C ABI's wici_dtype).  A W_Q8 matrix [N, K]
// is N*K code bytes (q + 128, row-major) followed, at the next 256-byte
// boundary, by N*K/32 half-precision block scales (row-major, one per 32
// consecutive weights of a row); the weight is (code - 128) * scale.
enum WType { W_F32 = 0, W_BF16 = 1, W_Q8 = 2 };

constexpr int kBK = 32;   // K per step (one v_mfma_f32_16x16x32_bf16 depth)

// ---- tiles
// Tiles of the bf16 product (four wavefronts each): 128 x 256 (64 x 128 a wavefront:
// half the activation fragment reads per product), 128 x 128, and 64 x 128 (64 x 32 a
// wavefront, three stages, for few rows).
//   Two activation terms, random operands, fp32 output, 128 x 256: 8B gate/up at 1024
// rows 395 us (1218 TFLOP/s), down in four K ranges 205, gate/up at 2048 rows 751
// (1281); with fragments read just before their products, and 64-bit addresses in
// vector registers, the same blocks took 425, 228 and 791.  256 x 256 blocks (eight
// wavefronts, one workgroup per CU, three stages) measured the same (390, 204, 764),
// 256 x 128 445, 237 and 839, 256 x 256 on four wavefronts of 128 x 128 562, 264 and
// 1118; raised wavefront priority around the products 1-4% slower.
enum TileShape { TILE_128x256 = 0, TILE_128x128 = 1, TILE_64x128 = 2 };
constexpr int kTileShapes = 3;

// Per shape and 1, 2 or 3 activation terms: workgroups that fit on a CU (by LDS, 64 bytes
// a row, term and stage, and by registers); the time of a K step, us, with 1, 2, ... of
// them on the CU (a lone one waits out its loads; more fill in until the matrix cores are
// busy); and the time a MB takes to reach an XCD's L2.  Fitted to the products of
// profiles/tile_times.csv (4761: 1B, 8B, 32B and smaller shapes, 65 to 4096 rows, 1
// to 8 K ranges): 8% rms.  The two wavefront layouts of 64 x 128 are rows of their own.
struct Tile {
  int bm, bn;
  bool by_columns;  // an XCD owns column tiles (otherwise a run of tiles, row by row)
  int fit[3];
  float step[3][4], fetch[3];
};
inline const Tile& tile_of(int shape, bool swiglu) {
  static const Tile T[kTileShapes + 1] = {
      {128, 256, true, {2, 2, 2}, {{.62f, 1.04f}, {.82f, 1.37f}, {1.05f, 2.13f}}, {.64f, .56f, .65f}},
      {128, 128, false, {4, 3, 2}, {{.43f, .60f, .88f, 1.25f}, {.55f, .89f, 1.40f}, {.67f, 1.24f}},
       {.28f, .29f, .41f}},
      {64, 128, true, {4, 3, 2}, {{.30f, .45f, .70f, .89f}, {.32f, .65f, .96f}, {.37f, .80f}},
       {.25f, .17f, .30f}},
      {64, 128, true, {4, 3, 2}, {{.26f, .44f, .71f, .82f}, {.33f, .64f, .95f}, {.38f, .84f}},
       {.63f, .19f, .19f}}};
  return T[shape == TILE_64x128 && swiglu ? kTileShapes : shape];
}

// Time of a product of M x N x K in nsplit K ranges, us: on the XCD with most workgroups
// (32 CUs; tiles that do not divide into eight leave some XCDs less), rounds of resident
// ones times K steps, plus the rows and columns that it reads through its L2, plus the
// partials written.
inline float tile_time(int shape, bool swiglu, int nt, int M, int N, int K, int nsplit) {
  const Tile& t = tile_of(shape, swiglu);
  const int fit = t.fit[nt - 1], places = 32 * fit;
  const int rows = (M + t.bm - 1) / t.bm, cols = (N + t.bn - 1) / t.bn;
  const int own = t.by_columns ? (cols + 7) / 8 * rows : (rows * cols + 7) / 8;  // a range's
  const int n = own * nsplit, rest = n % places;
  const float* step = t.step[nt - 1];
  float per_step = (float)(n / places) * step[fit - 1];
  if (rest) {
    const int k = (rest + 31) / 32;
    const float lo = step[k > 1 ? k - 2 : 0], f = (float)(rest - 32 * (k - 1)) / 32.f;
    per_step += lo + (step[k - 1] - lo) * (0.5f + 0.5f * f);
  }
  // tiles at work together, and what they read
  const int now = std::min(places, own), line = t.by_columns ? rows : cols;
  const int lines = (now + line - 1) / line, across = std::min(line, now);
  const int r = t.by_columns ? across : lines, c = t.by_columns ? lines : across;
  const float mb = (float)(r * t.bm * nt + c * t.bn) * 64e-6f * (float)(K / kBK) *
                   std::max(1.f, (float)own / (float)places);
  float us = 3.3f + per_step * (float)K / (float)(kBK * nsplit) + mb * t.fetch[nt - 1];
  if (nsplit > 1) us += (float)nsplit * M * N * 0.5e-6f;
  return us;
}

// The fastest tile for a split count.
inline int tile_shape(int nt, int M, int N, int K, int nsplit, bool swiglu) {
  int best = 0;
  for (int s = 1; s < kTileShapes; ++s)
    if (tile_time(s, swiglu, nt, M, N, K, nsplit) < tile_time(best, swiglu, nt, M, N, K, nsplit))
      best = s;
  return best;
}

// K ranges of a tiled product whose partials another kernel adds, each at least 256 deep:
// as many (at most four) as still leave at most two blocks per CU (512).  bf16 weights: or
// up to eight, if the time with the partials' reading is at least 8% below that count's;
// or fewer for a fifth, since longer fp32 sums are less exact (1B with an fp32 cache, logits
// from 64 bits 3.0e-6; QKV and O at 512 rows in one and two ranges instead of four 4.1e-6).
// Over the measured products of more than 128 rows count and tile then cost 4.2% more than
// the best ones on average, the worst choice 39% (1B down, one term, 4096 rows): 32B O at
// 333 rows 51.9 us, 74.3 on the wider tile; 32B down at 1024 rows 552 in eight ranges, 707
// in three, at 2048 rows 1035 in four, 1197 in two.
inline int tile_split_count(int wt, int nt, int M, int N, int K, int max_split) {
  if (nt < 1 || M <= 32 || (wt != W_BF16 && wt != W_Q8)) return 1;
  auto fits = [&](int n) { return K % (2 * kBK * n) == 0 && K / n >= 256; };
  const int bn = wt == W_BF16 && M >= 1024 ? 256 : 128;
  const int tiles = ((M + 127) / 128) * ((N + bn - 1) / bn);
  int n = std::max(1, std::min({max_split, 4, 512 / std::max(tiles, 1)}));
  while (n > 1 && !fits(n)) --n;
  if (wt == W_Q8) return n;
  auto time = [&](int s) {
    return tile_time(tile_shape(nt, M, N, K, s, false), false, nt, M, N, K, s) +
           (s > 1 ? (float)s * M * N * 0.7e-6f : 0.f);
  };
  const float usual = time(n);
  int best = n;
  for (int s = 1; s <= std::min(max_split, 8); ++s)
    if (s != n && (s == 1 || fits(s)) && time(s) < (s < n ? 0.8f : 0.92f) * usual &&
        time(s) < time(best))
      best = s;
  return best;
}

// ---- few rows
constexpr int kRowsKC = 128;       // K ranges are multiples of this (whole slices)
constexpr int kRowsSyncLine = 64;  // ints per tile: counter at 0, XCD records from 32
constexpr int kRowsMaxTiles = 512;  // tiles that can be split
// Rows the kernel takes (8-bit weights: at 64 rows it is level with the tiles on the
// narrow products, 32B O 34.0 and 35.0 us, 8B QKV 29.5 and 31.4).
constexpr int kRowsMaxBf16 = 128, kRowsMaxQ8 = 64;
constexpr int kGemmRowsSyncInts = kRowsMaxTiles * kRowsSyncLine;

inline bool gemm_rows_takes(int wt, int nt, int M, int K) {
  return nt >= 1 && nt <= 3 && M >= 1 && K % kRowsKC == 0 &&
         ((wt == W_BF16 && M <= kRowsMaxBf16) || (wt == W_Q8 && M <= kRowsMaxQ8));
}

// Splits along K for the few-rows kernel: the fewest (up to `most`) that give at
// least 192 workgroups of bn weight rows with whole 128-deep slices, as far as the
// partials (tm 16-row tiles) fit `part_floats` and the tiles the sync lines.
// (Measured at 16 rows on the 8B shapes, bf16: QKV 2 splits 12.6 us, 4 13.3; O 4
// splits 9.9 us, 8 10.3; down 4 splits 24.8 us, 7 27.3; at 48 rows QKV 2 splits
// 19.1 us, 8 20.0: more, shorter workgroups pay more in pipeline fill and in the
// sum.)
inline int gemm_rows_splits(int tm, int bn, int N, int K, size_t part_floats, int most) {
  const int T = (N + bn - 1) / bn;
  if (T > kRowsMaxTiles) return 1;
  int best = 1;
  for (int s = 2; s <= most && T * best < 192; ++s) {
    if (K % (s * kRowsKC)) continue;
    if ((size_t)T * s * bn * 16 * tm > part_floats) break;
    best = s;
  }
  return best;
}

// 16-row tiles, 64-row column tiles per workgroup and K ranges of the few-rows kernel;
// part_floats is kAddedOutside where another kernel adds the ranges.
constexpr size_t kAddedOutside = ~(size_t)0;
struct RowsPlan {
  int tm, wn, nsplit;
};

inline RowsPlan rows_plan(int wt, int epi, int M, int N, int K, size_t part_floats, int most) {
  const bool q8 = wt == W_Q8;
  const int tm = M <= 64 ? (M + 15) / 16 : M <= 96 ? 6 : 8;
  auto plan = [&](int wn) {
    return RowsPlan{tm, wn, gemm_rows_splits(tm, 64 * wn, N, K, part_floats, most)};
  };
  if (tm > 4) return plan(2);
  // 128 weight rows per workgroup (each activation fragment read for twice the
  // columns) where that alone still gives 192 workgroups: 8B gate/up, bf16, 43.2 ->
  // 40.2 us at 16 rows, 49.2 -> 42.7 at 32, 55.5 -> 47.4 at 48, 62.3 -> 55.1 at 64;
  // Q8 43.8 -> 39.6 at 32 and 78 -> 66 at 64, but 31.8 -> 33.3 at 8 and 47.8 -> 49.5
  // at 48.  Narrower products keep 64 (O at 48 rows 15.6 against 17.9 us).
  if (epi != GEMV_RESID && N >= 192 * 128 && !(q8 && (tm == 1 || tm == 3))) return plan(2);
  // Also, from 17 rows of bf16 weights, where the K ranges that give 192 workgroups are
  // still 1024 deep: QKV 19.4 -> 16.4 us at 32 rows, 23.1 -> 20.0 at 48, 27.1 -> 23.2 at
  // 64, down 27.4 -> 26.6, 33.1 -> 29.0 and 37.3 -> 32.8 (at 16 rows 25.2 against 25.3; O,
  // whose ranges would be 512 deep, 16.5 -> 22.0 at 48).
  if (!q8 && tm > 1 && most > 1) {
    const RowsPlan p = plan(2);
    if ((long)((N + 127) / 128) * p.nsplit >= 192 && K / p.nsplit >= 1024) return p;
  }
  return plan(1);
}

// Whether the few-row kernel beats the tiles where another kernel adds K ranges, at most
// `most`.  Up to 64 rows always: product plus the row norm that adds, us, few-row kernel
// and tiles, 8B O 14.7 and 16.3 at 48 rows, 16.2 and 16.8 at 64; down 32.2 and 35.5, 34.6
// and 37.8; QKV 16.5 and 17.9, but 20.3 and 19.3; 1B down 16.0 and 19.4 at 64 rows, 32B
// 84.1 and 80.2.  More rows leave one workgroup per CU, so only where the launch fills
// most of one round of them (96 rows: 8B down 42.0 and 52.8, O 20.5 and 20.6, QKV 26.5
// and 28.2, gate/up 78.0 and 90.0, 32B down 104 and 116; but 1B down, 128 workgroups, 23.9
// and 20.2, and 32B gate/up, 432, 178 and 163), past 96 rows in whole products (128 rows:
// 8B gate/up 90.1 and 97.4; O in eight ranges 24.9 and 21.5, QKV in four 34.6 and 31.3).
inline bool gemm_rows_best(int wt, int nt, int M, int N, int K, int most) {
  if (!gemm_rows_takes(wt, nt, M, K)) return false;
  if (M <= 64) return true;
  const RowsPlan p = rows_plan(wt, GEMV_STORE, M, N, K, kAddedOutside, M <= 96 ? most : 1);
  const int wgs = (N + 64 * p.wn - 1) / (64 * p.wn) * p.nsplit;
  return wgs >= 192 && wgs <= 256;
}

// Whether it does where only the launch itself can add K ranges; the other choice is a
// tiled product in one range (up to 64 rows 8B QKV 18.9 and 52.9 us at 48, gate/up 47.4
// and 58.6; LM head 239 and 246, but 286 and 264 at 64).  Past 64 rows again not in more than one round (LM head of
// 128256 at 80 rows 348 and 309 us, at 128 477 and 341; 32B gate/up 175 and 160, 233 and
// 179; 8B gate/up, one round, 74.3 and 87.9, 86.5 and 97.4), nor in K ranges where the
// tiles, two to each of its 128 weight rows then, fill the chip (1B gate/up 30.4 and
// 28.5, 37.6 and 28.6; but 8B QKV, 96 tiles, 28.8 and 51.7, 40.3 and 55.4).
inline bool gemm_rows_merge_best(int wt, int nt, int M, int N, int K) {
  if (!gemm_rows_takes(wt, nt, M, K)) return false;
  const int wgs = (N + 127) / 128;
  return M <= 64 || wgs < 128 || (wgs >= 192 && wgs <= 256);
}

// K ranges of a product whose partials another kernel adds, at most max_split (1: do not
// split): of the few-row kernel where that is the best one, of the tiles otherwise.
inline int gemm_split_count(int wt, int nt, int M, int N, int K, int max_split) {
  return gemm_rows_best(wt, nt, M, N, K, max_split)
             ? rows_plan(wt, GEMV_STORE, M, N, K, kAddedOutside, max_split).nsplit
             : tile_split_count(wt, nt, M, N, K, max_split);
}

}  // namespace wici
