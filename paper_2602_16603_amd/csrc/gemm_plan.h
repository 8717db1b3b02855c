// Which tile a GEMM runs on.  Plain C++17 with no GPU dependency: the rules can be built and checked on the CPU.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace fp {

constexpr int kBK = 64;                            // k-tile of the large tiles, and the unit of K ranges

constexpr uint32_t kOffOutOfRange = 0x80000000u;   // a byte offset no buffer descriptor here covers

// Row tile of a grouped launch whose experts receive `mean_rows` rows on average: the smallest that holds nearly every
// expert in one tile (a second one reads the expert's weights again), up to 128 rows of the ring kernel; from about 100
// rows on the matrix pipes bound the launch and the 256-row tile, which multiplies only the rows it has in steps of 32, is ahead.  The
// counts spread by about the root of their mean, hence the lines below 64 and 128.  experts_up + experts_down (with the combine), us,
// on tiles of 32, 64, 128 and 256 rows, [hidden, ffn, experts, top_k]:
//   rows per expert   [2048 768 128 8]      [4096 1536 64 8]      [4096 14336 8 2]        [2048 1408 64 6]
//   16                200  201              380  386              428  428                182  185
//   22                215  209              421  395              427  432                201  189
//   44                     230  244  247         425  458  468         452   576   651         205  224  229
//   52                     256  256  260         472  468  476         464   587   659         234  223  227
//   86                          280  281              503  504               613   700              250  250
//   92                          284  284              509  510               628   703              249  253
//   100                         325  290              521  521               640   709              257  260
//   110                         334  295              616  528               660   718              307  266
//   130                         398  315              790  553              1020   738              380  275
// (Tiles that are left out are slower by more.  At the line of 96 rows some of the narrow experts have a second 128-row tile already, 325
// against 288 us, and on the widest ones the 128-row tile stays 9 to 11 % ahead up to 110.)
// The smaller tiles reach an expert's gate and up rows through one 32-bit offset, as the dense fused kernel does
// ([2 ffn][hidden] below 2 GiB); the 256-row tile has a base for each.
inline int moe_tile_rows(int64_t mean_rows, int64_t ffn, int64_t hidden) {
  if ((ffn + 256) * hidden * 2 >= (int64_t)kOffOutOfRange) return 256;
  return mean_rows <= 18 ? 32 : mean_rows <= 48 ? 64 : mean_rows <= 96 ? 128 : 256;
}

// Shares of a W panel in the large tile's L2 warm-up, for as many row tiles as walk the panel together (at most eight): with
// eight shares among two to seven the rest of the lines was never asked for (all five heights of the tile, 2-7 row tiles: 4 to 15 %
// faster with four or two shares; more row tiles: 0 to 5 %).  One row tile shares its lines with nobody, and asking for them
// ahead only crowds out the others: 256 x 27648 x 5120 SwiGLU 168 us with two shares, 158 with eight, 153 with none; 129 to 256 rows of
// 160 column tiles and more 0 to 10 % faster than with eight, 1 % slower at most.
constexpr int warm_shares(int row_tiles) { return row_tiles >= 8 ? 8 : row_tiles >= 4 ? 4 : row_tiles >= 2 ? 2 : 0; }

// Whether the large tile on three stages (128 and 160 rows) asks for the L2 warm-up as well.  Three stages hide most of what
// sharers wait for each other, and the extra requests then cost 1 to 6 %; but where K is an odd number of times a power of two
// from 512 on they gain more than that on average, with SwiGLU up to 7 times.  1259 problems of 257 to 3000 rows, 44 K from 320
// to 28672, cold weights; time with the warm-up over time without it, mean per K (powers of two times the factor):
//   factor        bf16 and residual                       SwiGLU
//   1             1.011 to 1.051                          1.021 to 1.078
//   3  (x 512 up) 0.952 0.956 0.970 0.978, 24576 1.010    0.987 1.008 1.019 1.019, 24576 1.025
//   5             0.936 0.923 0.953, 20480 1.033          0.971 0.952 1.003, 20480 1.019
//   7             1.000 1.008 0.994 0.945                 1.010 1.015 1.019 0.967
//   9 to 15       0.983 to 1.003                          1.019 to 1.049
//   27, 37        1.014 1.018 1.060                       1.064 1.074 1.077
//   x 256         0.987 to 1.019                          1.001 to 1.041
//   less          0.971 to 1.034                          1.004 to 1.040
// Single problems differ from these means by up to 10 %: which lines crowd one another depends on all three sizes.  So the large
// factors stay in for bf16 and residual: 18944 would gain 6 % without, but 5120 columns of 27648, nine row counts from 1885 to
// 3846, lose 2 % on average and up to 5.
constexpr bool warm_three_stages(int k, bool swiglu) {
  const int power = k & -k;
  return power >= 512 && k > power && (!swiglu || k < 8 * power);
}

// Column tiles of 256 from which on a launch of one row tile is not cut over K and does not take the 128-column tile.
constexpr int64_t kWideTiles = 160;

// Whether a problem runs on the few-rows (ring) kernel: up to kFewRows rows, and up to twice as many where the large kernel's
// tile on 96 or 128 rows is not ahead.  That is where the latter is slower, us, few-rows kernel / large kernel, cold weights:
//  - kWideTiles column tiles and more, where it is 256 columns wide: 65 x 49152 x 5120 110 / 137, 65 x 128256 x 5120 244 / 288,
//    128 x 57344 x 5120 6 % ahead.  Not so for a short K in one round of its tiles, whose prologues and stores it has fewer of
//    (K of 256 to 1088: the large kernel 1 % behind to 75 % ahead).  558 problems of 65 to 128 rows on 41000 to 180000 columns: none
//    slower than on the few-rows kernel alone, 1.03 times its speed; what is left on the table is K of 8192 (up to 22 %), of
//    1536 to 2112 in one round (up to 22 %) and two whole rounds of short K (up to 40 %), beside losses close by.
//  - fused gate_up projections of that width, which are asked about apart (32B shape, 70 / 128 rows: 120 / 129, 140 / 149).
//  - a long K: 128 x 5120 x 24576 66 / 71; 16448 to 17664 are up to 9 % faster on the large kernel, 20480 is even.
// The others are faster there: 8B shape, 70 / 128 rows, cold, us, gate_up 54 / 55.5 -> 51 / 54, qkv 19 / 22.5 -> 16 / 19.5, o
// 15.5 / 18.5 -> 14.5 / 17.5, down 29 / 34 -> 28.5 / 33.5; 300 drawn projections of 65 to 128 rows 8 % on average.
constexpr int kFewRows = 64;
inline bool few_rows(int64_t m, int64_t n, int64_t k) {
  if (m <= kFewRows || m > 2 * kFewRows) return m <= kFewRows;
  const int64_t tiles = (n + 255) / 256;
  return tiles >= kWideTiles ? tiles > 256 || k > 1152 : k > 16384;
}

// Tile width and number of K ranges for a problem.  Enough 256-column tiles to occupy the chip, or
// more than two row tiles (then the MFMAs bound the launch and the wide tile's operand reuse
// counts: measured at 768 tokens and up): the 256-column tile.  Otherwise the 128-column tile.
// Either is cut over K only as far as it takes to reach about one workgroup per CU, and never
// below 8 k-tiles (512 columns) per range.
struct W4Shape {
  int nj;       // W blocks per wave tile: 8 (256-column tile) or 4 (128-column tile)
  int splits;   // 1 = no split
};
inline W4Shape w4_shape(int64_t m, int64_t n, int64_t k) {
  const int64_t tiles_m = (m + 255) / 256;
  const int64_t wide = tiles_m * ((n + 255) / 256);
  if (wide >= kWideTiles) return {8, 1};
  const bool narrow = tiles_m <= 2;
  const int64_t tiles = std::max<int64_t>(1, narrow ? tiles_m * ((n + 127) / 128) : wide);
  int s = (int)std::max<int64_t>(1, std::min<int64_t>(16, 256 / tiles));
  while (s > 1 && (k / kBK) / s < 8) --s;
  return {narrow ? 4 : 8, s};
}

// Tile and number of K ranges launch_gemm uses with that much workspace (splits 1 = uncut; 0 = the
// problem does not run on the fast kernel at all).
inline W4Shape w4_plan(int dtype, int64_t m, int64_t n, int64_t k, size_t workspace_bytes) {
  if (dtype != 1 || k % kBK != 0 || n % 8 != 0 || n > (1 << 21) || k > (1 << 21)) return {8, 0};
  // (the size limits keep the fast kernel's 32-bit buffer offsets below kOffOutOfRange)
  W4Shape p = w4_shape(m, n, k);
  if (p.splits > 1 && (size_t)p.splits * m * n * sizeof(float) > workspace_bytes) p.splits = 1;
  const int64_t tiles = ((m + 255) / 256) * ((n + 32 * p.nj - 1) / (32 * p.nj));
  if (tiles * p.splits < 96) p.splits = 0;
  return p;
}

// What a problem that w4_plan cuts over K runs as.  Three or four row tiles and a short K: the 128-column
// tile in fewer ranges (possibly one: nothing is cut then), if that occupies the chip -- fewer partial sums
// against more operand reads per MFMA, which a long K would pay for too often.  With the reduction, us:
// 777 x 6144 x 4096 54 -> 45, 777 x 4096 x 4096 44 -> 40, 590 x 5120 x 2048 30 -> 24, but x 14336 110 -> 115; 600 x 6144 x
// 4096 has 144 tiles and stays (47.7, 49).  Of 80 drawn problems of 513 to 1024 rows and K up to 6144 none was more than 3 %
// slower than without this rule.  Residual projections stay cut (their tail rides on the reduction).
inline W4Shape w4_cut(int64_t m, int64_t n, int64_t k, bool residual, W4Shape p) {
  const int64_t tiles_m = (m + 255) / 256, tiles = tiles_m * ((n + 127) / 128);
  if (p.nj != 8 || tiles_m > 4 || k > 6144 || tiles > 256) return p;
  const int s = (int)std::min<int64_t>(p.splits, 256 / tiles);
  return tiles * s >= 184 && s >= (residual ? 2 : 1) ? W4Shape{4, s} : p;
}

// Tile of the fused gate_up projection: 128 FFN columns when that occupies the chip or the
// request has more than two row tiles, else 64.
inline int swiglu_nj(int64_t m, int64_t f) {
  const int64_t tiles_m = (m + 255) / 256;
  return tiles_m <= 2 && tiles_m * ((f + 127) / 128) < 160 ? 4 : 8;
}

// Whether the fused gate_up projection (f outputs, W of 2 f rows) runs on the large and the few-rows tiles: the others' W
// offsets are 32 bits wide and reach both halves of the [gate | up] panel.
inline bool swiglu_fusable(int64_t m, int64_t f, int64_t k) {
  if (k % kBK != 0 || f % 8 != 0 || m <= 0) return false;
  if ((f + 256) * k * 2 >= (int64_t)kOffOutOfRange) return false;
  const int cols = swiglu_nj(m, f) * 16;
  return ((m + 255) / 256) * ((f + cols - 1) / cols) >= 96;
}

// Whether it runs on the few-rows kernel (which wants 16-byte aligned operands): where its own tile would be 256 columns wide, up
// to 128 rows (few_rows has the figures).
inline bool swiglu_few_rows(int64_t m, int64_t f) { return m <= kFewRows || (m <= 2 * kFewRows && swiglu_nj(m, f) == 8); }

// A launch of one or two row tiles on the 128-column or the few-rows tile reads every line of W for one or two workgroups only,
// and workgroups in step ask for the same 128 or 256 bytes of every row.  Where rows lie a power of two or three of them apart those
// fall on few HBM channels, on fewer or more of them with where the allocation lies; so the columns' starts in K are spread evenly
// over it, in groups of 128 columns.  Returns the number of such groups, 0: all start at the beginning.  A projection fused with SiLU*up
// and the plain one of the same matrix have to add up their products in the same order whatever kernel takes them: the start
// depends on the column modulo half the columns (gate and up of one output start alike) and nothing else, and
// where either form could be on a tile that does not start elsewhere (kWideTiles, few_rows of a long K) neither does.  So a row's
// bits are the same in all calls that have these starts, and differ from those of a larger call in the order of the sums.
// us, cold, five allocations each, gate_up of [14336 outputs 4096]: 50 rows 52.5 (45..57) -> 43.0 (42.7..43.4), 256 rows 69.3 -> 63.1;
// [14336 6144] 50 rows 82.3 -> 65.6, 200 rows 102.6 -> 89.1; [8192 2048] 23.7 -> 23.6, 31.8 -> 30.7; [18944 3584] 73.7 -> 73.4,
// 98.9 -> 98.1.  Other spreads are worse or no better: 8 or 16 starts in turn 44 to 68, a random one 46.6.
inline int start_groups(int64_t m, int64_t n, int64_t k) {
  const bool narrow = m <= 512 && (m + 255) / 256 * ((n + 255) / 256) < kWideTiles;
  return narrow && n % 256 == 0 && k % 128 == 0 && k >= 2048 && k <= 16384 ? (int)(n / 256) : 0;
}

// The starts an uncut bf16 projection runs with (of n columns of W, gate and up ones together if fused): its tile is `nj` W
// blocks per wave wide, or the few-rows kernel's, which starts elsewhere on 32 and 64 rows only.
inline int uncut_starts(int64_t m, int64_t n, int64_t k, int nj, bool few) {
  return few ? (m <= kFewRows ? start_groups(m, n, k) : 0) : nj == 4 ? start_groups(m, n, k) : 0;
}

// The k at which a workgroup whose columns begin at `col` starts.
constexpr int k_start(int col, int k, int groups) { return groups ? (col / 128 % groups) * (k / 128) / groups * 128 : 0; }

// Rows of the large tile (256 columns; SwiGLU 128 outputs; K % 64 == 0, not cut).  A CU works off its tiles one after the other;
// a launch of a few rounds loses what its last round leaves empty and the padding of its last row tile, a smaller tile
// reads W more often.  The rule is an estimate in ns fitted to 700 problems on all five heights (257-9000 rows, the dense
// shapes' projections and drawn ones, cold weights): a round costs a fixed part and a part per k, a partly filled one at
// least 0.66 of that.  On 239 other problems (with the warm-up rule above) its choice is 0.04 % slower than the best of the five and
// 10.1 % faster than 256 rows on average, more than 1 % slower than the best on 2, by 4.7 % at most (1217 x 13816 x 9024 SwiGLU, 524
// us on 192 rows, 500 on 224), and nowhere more than 0.8 % slower than 256 rows.  us, 256 rows against the choice: 600 x 14336 x
// 4096 SwiGLU 139 -> 121 (160 rows), 1300 x 6144 x 4096 73 -> 57 (160), 3001 x 27648 x 5120 SwiGLU 1255 -> 1204 (224), 3000 x 14336
// x 4096 SwiGLU 514 -> 492 (192).
enum class LargeEpilogue { kBf16, kSwiGLU, kResidual };

inline double large_tile_ns(int rows, int64_t m, int64_t tiles_n, int64_t k, LargeEpilogue epilogue) {
  const double per_k = rows == 128 ? 12.66 : rows == 160 ? 14.56 : rows == 192 ? 16.51 : rows == 224 ? 18.02 : 20.76;
  const double fixed = epilogue == LargeEpilogue::kResidual ? 20880 : epilogue == LargeEpilogue::kSwiGLU ? 8370 : 6890;
  const int64_t tiles = (m + rows - 1) / rows * tiles_n, left = tiles % 256;
  return (tiles / 256 + (left ? 0.66 + 0.34 * left / 256.0 : 0.0)) * (fixed * rows / 256.0 + per_k * (double)k);
}

inline int large_tile_rows(int64_t m, int64_t tiles_n, int64_t k, LargeEpilogue epilogue) {
  int best = 256;
  double best_ns = 0.98 * large_tile_ns(256, m, tiles_n, k, epilogue);   // (the estimate's error: a tie stays with the large one)
  for (int rows : {224, 192, 160, 128}) {
    const double ns = large_tile_ns(rows, m, tiles_n, k, epilogue);
    if (ns < best_ns && (m + rows - 1) / rows * tiles_n <= INT32_MAX) { best_ns = ns; best = rows; }
  }
  return best;
}

// Problems with too few 256x256 tiles to occupy the chip, and odd K.  A CU works off its tiles one after the other, so a
// tile size costs rounds = ceil(tiles / 256) times what a tile costs: a fixed part (prologue, epilogue, for a residual
// also its read) and a part per k.  Small tiles keep more CUs busy, large ones read their operands less often; which wins
// turns on how the rounds come out, so the rule is the estimate itself, in ns, fitted to 510 problems of 16 to 8192 rows,
// 256 to 8192 columns and K with cold weights: its choice is 0.7 % slower than the best of the five (all five measured),
// in 5 of the 510 slower than 128x128 register-staged tiles alone, by up to 13 %.  (The fewest outputs on the busiest CU,
// the rule before, chose many small tiles for wide problems of short K: 725 x 7104 x 256 31.6 us, now 15.2; 1168 x 2648 x
// 1312 38 -> 21; and the large tile for odd K from 96 tiles on, where 128x128 ones still fit two to a CU: 2012 x 2840 x
// 2552 64 -> 51.)
enum class GemmTile { kRing32, kRing64, kRing128, kAny128, kLarge };   // 32x64, 64x64, 128x128; register-staged 128x128; 256x256

inline int64_t tile_rounds(int64_t m, int64_t n, int64_t bm, int64_t bn) {
  return (((m + bm - 1) / bm) * ((n + bn - 1) / bn) + 255) / 256;
}

inline double small_problem_ns(GemmTile tile, int64_t m, int64_t n, int64_t k, bool residual) {
  const double kd = (double)k;
  switch (tile) {
    case GemmTile::kRing32: return 2100 + tile_rounds(m, n, 32, 64) * ((residual ? 2500 : 2200) + 2.3 * kd);
    case GemmTile::kRing64: return 1000 + tile_rounds(m, n, 64, 64) * ((residual ? 4300 : 3500) + 3.9 * kd);
    case GemmTile::kRing128: return -1400 + tile_rounds(m, n, 128, 128) * ((residual ? 9900 : 6800) + 9.1 * kd);
    case GemmTile::kAny128: {                      // two workgroups share a CU: a pair takes 1.35 times as long as one
      const int64_t r = tile_rounds(m, n, 128, 128);
      return ((r / 2) * 1.35 + r % 2) * ((residual ? 13800 : 4200) + 13.8 * kd);
    }
    default: return 900 + tile_rounds(m, n, 256, 256) * ((residual ? 17100 : 8600) + 21.5 * kd);
  }
}

// The tile for 16-byte aligned operands.  The large one takes K that is not a multiple of 64 here (kBK), from the number of
// tiles on that makes it worth a look; the ring kernel's and the large tile's 32-bit offsets bound their sizes.
inline GemmTile small_problem_tile(int64_t m, int64_t n, int64_t k, bool residual) {
  GemmTile best = GemmTile::kAny128;
  double best_ns = small_problem_ns(best, m, n, k, residual);
  auto consider = [&](GemmTile tile) {
    const double ns = small_problem_ns(tile, m, n, k, residual);
    if (ns < best_ns) { best_ns = ns; best = tile; }
  };
  if (k <= (1 << 21) && ((m + 31) / 32) * ((n + 63) / 64) <= INT32_MAX) {
    consider(GemmTile::kRing32);
    consider(GemmTile::kRing64);
    consider(GemmTile::kRing128);
  }
  const int64_t large = ((m + 255) / 256) * ((n + 255) / 256);
  if (k % kBK != 0 && n <= (1 << 21) && k <= (1 << 21) && large >= 96 && large <= INT32_MAX) consider(GemmTile::kLarge);
  return best;
}

// The gate_up projection of such a problem with SiLU(gate)*up in the ring kernel's epilogue: rows per tile (64 of the f
// outputs each), or 0 where the projection on its own tile and a silu_mul launch (4 us) are ahead, as they are for many
// rows of few k (867 rows, 4704 outputs of 1144: 50 + 5 us against 56).  Fitted to 200 problems; 0.4 % from the best.
inline int swiglu_tile_rows(int64_t m, int64_t f, int64_t k) {
  const double kd = (double)k;
  const double ns[3] = {3800 + tile_rounds(m, f, 32, 64) * (600 + 5.6 * kd), 800 + tile_rounds(m, f, 64, 64) * (3900 + 7.5 * kd),
                        -400 + tile_rounds(m, f, 128, 64) * (5800 + 11.0 * kd)};
  const int i = ns[0] <= ns[1] && ns[0] <= ns[2] ? 0 : ns[1] <= ns[2] ? 1 : 2;
  const GemmTile plain = small_problem_tile(m, 2 * f, k, false);
  const bool ring = plain != GemmTile::kAny128 && plain != GemmTile::kLarge;   // (the same tiles, and a launch more)
  return ring || ns[i] <= small_problem_ns(plain, m, 2 * f, k, false) + 4000 ? 32 << i : 0;
}

// Rows of the fp32 tile (64 columns; 128 rows: 128 columns).  128 rows where the busiest of 256 CUs then has no more outputs
// than with 64 or 32, padding included; else an estimate in ns.  The tiles of a CU share its matrix pipes, and small ones hide
// each other's latencies, so it has a part per tile of the busiest CU and one per tile on average; fitted to 250 problems of
// 1 to 1024 rows (the 8B shape's projections, the tiny shape's, drawn ones) on the kernel as it was before its reads went between the
// MFMAs.  On the present one its choice is 0.1 % slower than the best of the six on 90 other problems, 3.2 % at most (37 x 5560 x
// 648, 10.0 against 9.7 us).  us on 16, 32, 48, 64, 80 and 128 rows: 300 x 4096 x 4096 101, 103, 100, 128, 91, 247; 300 x 4096 x
// 14336 376, 368, 360, 438, 328, 843; 300 x 28672 x 4096 698, 612, 621, 562, 576, 771; 67 x 6144 x 4096 50, 73, 57, 73, 91, 256.
inline double f32_tile_ns(int rows, int64_t m, int64_t n, int64_t k, bool residual) {
  struct Cost { int rows; double launch, tile, residual, busiest_k, average_k; };
  constexpr Cost costs[] = {{16, 4200, 0, 242, 5.06, 0.21}, {32, 3210, 265, 289, 6.38, 2.94}, {48, 2877, 554, 450, 8.63, 4.90},
                            {64, 2286, 1107, 573, 12.74, 4.58}, {80, 1553, 2063, 412, 14.98, 7.22}};
  const int64_t tiles = (m + rows - 1) / rows * ((n + 63) / 64);
  const double busiest = (double)((tiles + 255) / 256), average = tiles > 256 ? tiles / 256.0 : 1.0;
  for (const Cost& c : costs)
    if (c.rows == rows)
      return c.launch + busiest * (c.tile + (residual ? c.residual : 0)) + (double)k * (c.busiest_k * busiest + c.average_k * average);
  return 0;
}

inline int f32_tile_rows(int64_t m, int64_t n, int64_t k, bool residual) {
  auto outputs = [&](int64_t bm, int64_t bn) { return (((m + bm - 1) / bm) * ((n + bn - 1) / bn) + 255) / 256 * bm * bn; };
  const int64_t large = outputs(128, 128);
  if (large <= outputs(64, 64) && large <= outputs(32, 64)) return 128;
  int best = 80;
  double best_ns = f32_tile_ns(80, m, n, k, residual);
  for (int rows : {64, 48, 32, 16}) {
    const double ns = f32_tile_ns(rows, m, n, k, residual);
    if (ns < best_ns && (m + rows - 1) / rows * ((n + 63) / 64) <= INT32_MAX) { best_ns = ns; best = rows; }
  }
  return best;
}

}  // namespace fp
