// Which tiling a launch of the bf16 linear layer takes (plain C++: the rule runs on the device, which alone knows the rows).
#pragma once

#ifdef __HIPCC__
#define LLMC_RULE __host__ __device__ constexpr
#else
#define LLMC_RULE constexpr
#endif

namespace llmc {

constexpr int kGemmBig = 0, kGemmMid = 1, kGemmLow = 2, kGemmTiny = 3, kGemmFew = 4, kGemmTilings = 5;
constexpr int kGemmTileRows[kGemmTilings] = {128, 128, 64, 64, 32};
constexpr int kGemmTileCols[kGemmTilings] = {192, 128, 128, 64, 64};
constexpr int kGemmGrid = 512;                         // two workgroups on each of 256 compute units

// Cost of `tiles` tiles of nk steps: whole rounds of 512 tiles, two to a compute unit, and what is left over, one to a compute
// unit if that many are enough.  A round is a tile's fixed part and its steps.
struct GemmCost { int both_fixed, both_step, alone_fixed, alone_step; };

LLMC_RULE int gemm_cost(int tiles, int nk, GemmCost c) {
  const int rest = tiles % kGemmGrid;
  return (tiles / kGemmGrid) * (c.both_fixed + nk * c.both_step) +
         (rest == 0 ? 0 : rest <= kGemmGrid / 2 ? c.alone_fixed + nk * c.alone_step : c.both_fixed + nk * c.both_step);
}

// up to this many rows (and one round of 64 x 128 tiles) a launch waits for its weights: constants of their own, and no ring
constexpr int kGemmFewRows = 1024;

struct GemmPick { int path, tiles; };

// M > 0 rows, N columns, nk steps of 64 columns of the operands; act, resid: an activation follows the product, a residual.
//
// The constants are fitted for the CHOICE, not for the time, to the four products of blocks 64 to 2048 wide (QKV, output
// projection, both feed-forward layers) at 64 to 32,768 rows, each of the five tilings forced in turn in one process with
// complete outputs (the same bits).  Of 616 products at 1280 rows and more the choice is 0.7 % slower than the fastest
// tiling in the mean, eight times more than 10 %, at most 15 %; one set of constants for all rows, fitted to widths of 256,
// 768 and 1024, was 2.4 % slower in the mean, 55 times more than 10 %, up to 37 %, because it took 64 x 64 tiles where
// 64 x 128 or the ring are faster: the four layers (us, before / now) of a block 128 wide at 24,576 rows 53.3 / 46.4, 256
// wide at 8192 47.6 / 42.5, 384 wide at 8192 76.2 / 69.8, 512 wide at 6144 87.8 / 80.8, 768 wide at 2048 66.7 / 63.9, at 4096
// 107.1 / 105.1 and at 8192 164.4 / 164.7.
// Up to 1024 rows the constants are those of before without the ring, which won nothing there; few instructions count as
// well, because such a launch runs through its code once, from a cold cache (128 rows of 768 29.2 / 29.1).
// At 768 columns and K = 3072, 128 x 192 / 128 x 128 / 64 x 128 / 64 x 64 / 32 x 64 tiles take (us, one run) 126 / 144 / 167 /
// 210 / 270 for 24,576 rows, 68 / 58 / 76 / 92 / 117 for 10,240, 49 / 53 / 59 / 71 / 94 for 8192, 43 / 38 / 36 / 36 / 48 for
// 4096, 42 / 37 / 20 / 24 / 25 for 2048, 43 / 37 / 18 / 13 / 17 for 788, 44 / 37 / 17 / 12 / 11 for 256.
LLMC_RULE GemmPick gemm_pick(int M, int N, int nk, bool act, bool resid) {
  const int n64 = (N + 63) / 64, n128 = (n64 + 1) / 2, m64 = (M + 63) / 64, m32 = (M + 31) / 32;
  const int low_tiles = m64 * n128, tiny_tiles = m64 * n64, few_tiles = m32 * n64;
  GemmPick best = {kGemmLow, low_tiles};
  int best_cost = 0;
  auto offer = [&](int path, int tiles, int cost) {
    if (cost < best_cost) {
      best_cost = cost;
      best = GemmPick{path, tiles};
    }
  };
  if (M <= kGemmFewRows && low_tiles <= kGemmGrid) {
    best_cost = gemm_cost(low_tiles, nk, {350, 66, 260, 39});
    offer(kGemmTiny, tiny_tiles, gemm_cost(tiny_tiles, nk, {100, 44, 150, 23}));
    offer(kGemmFew, few_tiles, gemm_cost(few_tiles, nk, {100, 30, 130, 19}));
    return best;
  }
  const int n192 = (n64 + 2) / 3, m128 = (M + 127) / 128, big_tiles = m128 * n192, mid_tiles = m128 * n128;
  const int a = act ? 50 : 0;                          // alone, nothing covers a large tile's epilogue
  // a long product with a residual follows one whose idle workgroups have read its weights: 128 x 192 tiles, one to a compute
  // unit, against 128 x 128 tiles, two to some (us): 8192 x 768, K = 3072 49.0 / 52.9, 6144 x 768 45.7 / 48.9, 5120 x 1024,
  // K = 4096 60.2 / 66.0, 4096 x 1280, K = 5120 87.2 / 88.8; of short ones 3072 x 1536, K = 1536 34.1 / 31.2, 2560 x 2048,
  // K = 2048 42.0 / 40.1
  const bool warm = resid && nk >= 40;
  const GemmCost big = {1021, 155, (warm ? 574 : 564) + a, warm ? 123 : 129}, mid = {663, 122, 386 + a, 77};
  const bool ring = nk >= 2;                           // the ring starts with two steps
  if (ring && big_tiles > 4 * kGemmGrid) {             // many rounds: by the columns that are computed for padding
    const bool narrow = n192 * (big.both_fixed + nk * big.both_step) > n128 * (mid.both_fixed + nk * mid.both_step);
    return narrow ? GemmPick{kGemmMid, mid_tiles} : GemmPick{kGemmBig, big_tiles};
  }
  best_cost = gemm_cost(low_tiles, nk, {380, 70, 233, 55});
  offer(kGemmTiny, tiny_tiles, gemm_cost(tiny_tiles, nk, {196, 60, 177, 12}));
  if (few_tiles <= kGemmGrid / 2) offer(kGemmFew, few_tiles, 6 + nk * 9);          // only one to a compute unit
  if (ring) {
    offer(kGemmBig, big_tiles, gemm_cost(big_tiles, nk, big));
    offer(kGemmMid, mid_tiles, gemm_cost(mid_tiles, nk, mid));
  }
  return best;
}

}  // namespace llmc
