// Which tile each grouped-GEMM launch runs on: rules on sizes only, host code without HIP.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>

namespace moe {

// token rows x weight rows (a SwiGLU tile's weight rows are half gate, half up)
enum Tile { TILE_64X128, TILE_128X256, TILE_256X128, TILE_256X256, TILE_320X256 };

// Expected tiles of `groups` row segments of about `rows` rows each.  The per-expert row counts of a
// routed batch scatter around their mean (standard deviation about its square root), so an expert
// whose mean is 256 rows takes 1.5 256-row m-tiles on average but one 320-row tile.
inline double expected_mtiles(int bm, double rows, int64_t groups) {
  if (groups <= 1 || rows <= 0) return std::ceil(rows / bm) * groups;
  const double sigma = std::sqrt(rows);
  double per_group = 0;
  const int jmax = (int)((rows + 8 * sigma) / bm) + 1;
  for (int j = 0; j <= jmax; ++j)                          // E[ceil(m / bm)] = sum_j P(m > j bm)
    per_group += 0.5 * std::erfc((j * bm - rows) / (sigma * std::sqrt(2.0)));
  return per_group * groups;
}
// rounds of a persistent grid of one workgroup per CU; an expected count a few hundredths of a round
// above a whole number (the normal tail of the row counts) is that whole number
inline double tile_rounds(double tiles, int cus) { return std::max(1.0, std::ceil(tiles / cus - 0.05)); }

enum FwdEpilogue { FWD_SWIGLU, FWD_BF16, FWD_SCATTER };
// A forward launch (also the backward's recomputed up-projection): `groups` row segments (1: dense rows)
// of about rows_hint rows (0: unknown), rows2 rows of the extra dense group, N outputs, reduction K.
struct FwdSizes {
  int cus;
  int N, K;
  int64_t groups, rows_hint, rows2;
};

// 256 x 256 tiles of the phase kernel: the best measured on the DeepSeek-V3, Mixtral and skewed
// workloads (largest reuse per byte copied into LDS; also whenever a large dense extra group shares
// the launch).  With few expected rows per group the launch is a
// weight stream over few m-tiles, spread over more workgroups by smaller tiles: 64 x 128 up to
// 128 rows per group (1.4-1.8x faster at 2-128 rows), 128 x 256 up to 512 (1.1-1.5x).
inline Tile fwd_tile(const FwdSizes& s, FwdEpilogue epi) {
  const Tile tier = s.rows_hint <= 0 || s.rows2 > 512 ? TILE_256X256
                    : s.rows_hint <= 128              ? TILE_64X128
                    : s.rows_hint <= 512              ? TILE_128X256
                                                      : TILE_256X256;
  if (tier == TILE_64X128 || s.rows_hint <= 0 || epi == FWD_SCATTER) return tier;
  // Tile shape from the expected tile count of each shape.  A persistent launch takes about ceil(tiles / CUs) rounds of
  // its slowest workgroup.  A round of each tile against one of 256 x 256, measured over whole rounds of full tiles (K =
  // 1024 to 7168, 1 to 7 rounds, both epilogues): 320 x 256 1.07-1.17 (priced 1.15), 256 x 128 0.53-0.63 (priced 0.6), 128 x 256
  // 0.71-0.94.  The last is priced 0.7, its cost when the 256 x 256 tile was 10-15% slower; the choices that follow
  // from it were checked at the sizes below.  DeepSeek-V3 shapes (256 rows per expert, shared expert of 8192 rows
  // in the launch) run both projections on 320-row tiles, Mixtral shapes (1024 rows per expert, 2.25 rounds of 256 x 256
  // down-projection tiles) their down-projection, while Mixtral's up-projection (15.75 rounds either way) and the skewed
  // workload stay on 256 x 256.  Up-projections on 320-row tiles against 128 x 256 ones: 32 experts of 290 rows, d = 6384, F =
  // 4104 1147 us and 1607; 64 of 227, d = 3184, F = 4688 1133 and 1352; 32 of 320, d = 6160, F = 600 236 and 269.
  auto mtiles = [&](int bm) {
    return expected_mtiles(bm, (double)s.rows_hint, s.groups) + std::ceil((double)s.rows2 / bm);
  };
  auto rounds = [&](double tiles) { return tile_rounds(tiles, s.cus); };
  const double tn128 = (double)((s.N + 127) / 128);        // 128-column output blocks
  // a 256-row weight tile yields 128 SwiGLU outputs
  const double tn = epi == FWD_SWIGLU ? tn128 : std::ceil(tn128 / 2);
  const double m128 = mtiles(128), m256 = mtiles(256), m320 = mtiles(320);
  // A launch whose 256-row tiles cover at most a quarter of the chip takes 64 x 128 ones, an eighth of
  // the work each and two workgroups per CU, so they still fit about one round.  One segment, us on 256 x 256 / 64 x 128, by
  // tiles of 256 x 256 (of 256 CUs), up-projection and down-projection:
  //   tiles                 16         32         64         96         128        256
  //   up, K = 2048          41/18      42/19      42/31      43/44      45/54      55/105
  //   up, K = 7168          121/45     122/49     122/104    126/130    135/177    175/351
  //   down, K = 1024        24/11      24/12      25/19      26/26      27/32      33/58
  if (tier == TILE_256X256 && s.rows2 == 0 && m256 * tn <= s.cus / 4.0) return TILE_64X128;
  // With a partial last K slice too: 32 experts of 256 rows, d = F = 2040: up-projection 174 us on 320-row tiles, 274 on
  // 128 x 256, down-projection 96 and 152; 8 experts of 569 rows, d = 6408, F = 6112: up 633 and 842 (256 x 256), down 355 and 408.
  const double c320 = 1.15 * rounds(m320 * tn);
  if (tier == TILE_128X256) return c320 < 0.7 * rounds(m128 * tn) ? TILE_320X256 : tier;
  const double c256 = rounds(m256 * tn);
  // bf16 epilogue: also 256 x 128 tiles
  const double c256x128 = epi == FWD_BF16 ? 0.6 * rounds(m256 * tn128) : 1e30;
  if (c320 < c256 && c320 <= c256x128) return TILE_320X256;
  return c256x128 < c256 ? TILE_256X128 : tier;
}

// Rows of the extra group's tiles in a launch on `tile`, 0 for that tile's own.  On 320-row tiles, a
// dense extra group (the shared expert) is tiled 256 rows high when that
// adds no round: its tiles then carry the 8 live token blocks the routed ones do (the routed
// experts' ~256 rows), instead of 10.  DeepSeek-V3 shapes: up-projection 928 -> 1024 tiles
// (4 rounds either way), down-projection 1624 -> 1792 (7 rounds either way).
inline int extra_group_rows(const FwdSizes& s, FwdEpilogue epi, Tile tile) {
  if (tile != TILE_320X256 || s.rows2 <= 256) return 0;
  const double cols = (double)(epi == FWD_SWIGLU ? (s.N + 127) / 128 : (s.N + 255) / 256);
  const double g320 = expected_mtiles(320, (double)s.rows_hint, s.groups);
  return tile_rounds((g320 + std::ceil(s.rows2 / 256.0)) * cols, s.cus) <=
                 tile_rounds((g320 + std::ceil(s.rows2 / 320.0)) * cols, s.cus)
             ? 256
             : 0;
}

// m-tiles per band of the forward's tile order, by tile height.  256 and 320 rows: 4 against 8 measured 2% faster on the
// up-projection of 4096 tokens x 8 experts of 14336 (1450 -> 1421 us); 256 x 128 tiles, six down-projections of 1 to 8
// segments of 2500 to 6900 rows: within 1%, one 4% faster (59.8 us, 62.3 with 8).  Smaller tiles run launches that stream
// weights, once per band: 8, so that a shared expert's few hundred rows are one band (a layer of 400 tokens, d = 7168, 32 of 256
// experts and a shared one of F = 2048: 591 us, 604 with 4).
constexpr int band_m(int bm) { return bm >= 256 ? 4 : 8; }

// The backward's row products (dA, dX): max_rows rows in all.
// Tile shapes (all on the MN-major weight operand, two ds_read_b64_tr_b16 per fragment):
// 256 x 256 over 2 x 4 waves, a wave holding 128 token rows x 64 weight columns, so a K-step
// reads four token fragments (ds_read_b128) and two weight fragments, against two and four
// with 4 x 2 waves -- the transpose reads are the dearer ones (DeepSeek-V3 routed dX 816 ->
// 634 us, shared dX 605 -> 481); 256 x 128 (4 x 2 waves); 320 x 256 (2 x 4 waves, 10 token
// blocks).  Chosen like the forward's tiles, from the expected tile count of each shape; a round of 320 x 256 against
// one of 256 x 256 measured 1.08-1.23 (priced 1.15), 256 x 128 0.55-0.65 (priced 0.6).  No 320-row tiles with a
// K tail: no instance of the kernel (its registers do not suffice).
inline Tile bwd_rows_tile(int cus, int64_t groups, int64_t rows_hint, int64_t max_rows, int N, int K) {
  if (rows_hint > 0 && rows_hint <= 128) return TILE_64X128;
  const double rows = rows_hint > 0 ? (double)rows_hint : (double)max_rows / groups;
  auto cost = [&](int bm, int bn) {
    return tile_rounds(expected_mtiles(bm, rows, groups) * ((N + bn - 1) / bn), cus);
  };
  const double c256 = cost(256, 256), c256x128 = 0.6 * cost(256, 128);
  const double c320 = K % 64 ? 1e30 : 1.15 * cost(320, 256);
  if (c320 < c256 && c320 <= c256x128) return TILE_320X256;
  return c256x128 < c256 ? TILE_256X128 : TILE_256X256;
}

// Weight gradients over segments of about rows_hint rows (0: unknown) into rows of `pitch` bf16 values: true = the
// ring kernel's 256 x 256 tiles, false = the phase kernel's.  A tile of one or two K slices is bound by its stores.  The
// ring kernel's waves write 256-byte row pieces, the phase kernel's 128-byte ones, which on rows that do not
// start on a 128-byte line are two part lines each.  dW2 + dW13, us, ring / phase (F = 1024; 96 experts, or 64 at
// 32, 40 and 144 rows):
//   rows                     16       32       40       51       100      144      180      256
//   d = 2560 (whole lines)   303/281  206/206  212/219  336/341  443/466  366/335  570/505  675/600
//   d = 2528                 312/332  215/227  224/233  360/369  470/502  371/347  584/551  703/638
//   d = 2552                 466/574  307/386  305/391  433/587  475/555  389/390  601/592  732/676
inline bool wgrad_on_ring(int64_t rows_hint, int64_t pitch) {
  return rows_hint > 0 && rows_hint <= 128 && (pitch % 64 != 0 || rows_hint > 32);
}

// Order of a weight gradient's tm x tn tiles.  bf16 results n-fastest: the tiles an XCD runs together store whole output rows
// (32 experts of 255 rows, d = 7168, F = 2048: dW13 785 us m-fastest, 739 in blocks of 4 x 8 tiles, 720
// n-fastest; the ring kernel, 96 experts of 51 rows, d = 2560, F = 1024: 239 and 215).  The router's float32 partials m-fastest, its
// few m-tiles on one panel of the tokens (E = 384, T = 4096, d = 7168: 54.2 us, n-fastest 56.4; E = 256, T = 8192: 62.5, 63.6).
struct TileMN {
  int m, n;
};
constexpr TileMN wgrad_order(int i, int tm, int tn, bool f32) {
  return f32 ? TileMN{i % tm, i / tm} : TileMN{i / tn, i % tn};
}

}  // namespace moe
