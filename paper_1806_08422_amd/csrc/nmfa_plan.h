// Rules that choose a kernel's tile from the sizes of a run and the CUs of the device: plain functions of
// integers, so that they can be checked without a GPU.
#pragma once

namespace nmfa {

// Tile of the BF16 per-iteration kernel: rows x replicas of a workgroup. STEP_128 is 128 x 64 with BF16 J and
// 128 x 32 with FP8 or FP4 J; STEP_64X32_ALONE is 64 x 32 with the longer ring of one workgroup per CU.
enum StepTile : int { STEP_64X32_ALONE, STEP_64X32, STEP_128, STEP_256X64, STEP_256X128 };

struct StepPick {
  StepTile tile;
  double us;  // estimated time of the iteration
};

// jfmt: format of J (0 BF16, 1 FP8, 2 FP4). The cost of a tile size in us, fitted to measurements at N = 2100,
// 4100 and 8192, R = 64 .. 1024 (within 10 % of them but for a few at 2100): for every time the tiles fill the
// chip, or part of it, `once` + 2 us and a time per 128-k block, s1 while a CU has one workgroup and s2 with the
// two it can hold. 64 x 32 is the least serial time for a few tiles; 128 x 32 (BF16 J: 128 x 64) and 256 x 64
// read less per product; 256 x 128 is the best that fills the chip whole. Measured with 256 x 128 always
// and with this rule, us per iteration: FP4 J N = 2100, R = 64 39.0 -> 10.8, R = 1024 44 -> 30; N = 4100,
// R = 200 67 -> 19; N = 8192, R = 64 110 -> 27, R = 256 113 -> 47, R = 512 117 -> 84, R = 1024 142 (the
// next best, 256 x 64: 165); FP8 J N = 4100, R = 200 72 -> 21, R = 512 74 -> 51; BF16 J N = 2100,
// R = 300 45 -> 15, N = 8192, R = 64 118 -> 28, R = 256 122 -> 62, R = 512 127 -> 111, R = 1024 162 (the
// next best, 128 x 64: 245). With `once` counted once per launch, tiles that fill the chip more than once were
// taken where 256 x 128 is faster (that one, then the estimate's choice): FP4 J N = 2100, R = 2048 41 against 48,
// N = 2600, R = 4096 99 against 109; BF16 J N = 2000, R = 2048 43 against 48, N = 5500, R = 1536 182 against 215.
inline StepPick step_pick(int jfmt, int N, int R, int cus) {
  auto tiles = [&](int tm, int tr) { return (long)((N + tm - 1) / tm) * ((R + tr - 1) / tr); };
  auto cost = [&](int tm, int tr, int per_cu, double once, double s1, double s2) {
    const long n = tiles(tm, tr), full = n / (per_cu * cus), rest = n % (per_cu * cus);
    const double nb = (N + 127) / 128;
    return full * (once + 2 + s2 * nb) + (rest == 0 ? 0.0 : once + 2 + (rest <= cus ? s1 : s2) * nb);
  };
  StepPick p{STEP_64X32, 0.0};
  auto least = [&](StepTile tile, double us) {
    if (us < p.us) p = StepPick{tile, us};
  };
  if (jfmt == 0) {
    if (tiles(64, 32) <= cus)  // a workgroup per CU
      return StepPick{STEP_64X32_ALONE, cost(64, 32, 1, 3, 0.37, 0.37)};
    p.us = cost(64, 32, 2, 3, 0.58, 0.65);
    least(STEP_128, cost(128, 64, 1, 8, 0.88, 0.88));
    least(STEP_256X128, cost(256, 128, 1, 6, 2.3, 2.3));
  } else {
    const bool f4 = jfmt == 2;
    p.us = cost(64, 32, 2, 3, f4 ? 0.37 : 0.36, f4 ? 0.53 : 0.52);
    least(STEP_128, cost(128, 32, 2, f4 ? 4 : 5, f4 ? 0.39 : 0.5, f4 ? 0.7 : 0.85));
    least(STEP_256X64, cost(256, 64, 1, f4 ? 10 : 12, f4 ? 1.1 : 1.15, f4 ? 1.1 : 1.15));
    least(STEP_256X128, cost(256, 128, 1, 6, f4 ? 2.08 : 2.15, f4 ? 2.08 : 2.15));
  }
  return p;
}

// How the persistent small-N kernel shares its work among waves and lanes: `split` waves per 16-row tile, and
// 16 / ls replicas per workgroup, whose product holds each of them in ls columns.
struct SmallSplit {
  int split, ls;
};

// waves: row tiles of the instance (a wave each). FP64: while every wave of a workgroup can have a SIMD to
// itself, a tile's waves share its rows, each running the whole matrix product (the matrix cores are idle) and
// the libm epilogue of its rows only. us per iteration with 16 replicas per workgroup: N = 20, R = 256 2.6 with
// one wave per tile, 1.5 with two; N = 16 2.4 with one, 1.4 with two, 1.2 with four. Two waves on a SIMD gain
// nothing (N = 20, four waves per tile: 2.15; N = 33, two: 2.9 against 2.7), nor do several workgroups per CU (N
// = 20, R = 16384).
// While all its workgroups find a CU each, a workgroup takes 8 or (FP64) 4 replicas (ls = 2 or 4): the other
// columns of its product repeat them, and the lanes of the copies take over rows. us per iteration with ls =
// 1, 2, 4: FP64 N = 62, R = 1000 2.84, 1.72, 1.46, N = 100, R = 1000 5.67, 3.85, 3.41, N = 62, R = 2000 2.79,
// 1.79, 2.60, N = 20, R = 256 (two waves per tile) 1.15, 0.97; BF16 N = 173, R = 64 0.68, 0.60, 0.60, N = 256, R =
// 1024 0.92, 0.81, 0.85; FP32 N = 50, R = 1024 0.58, 0.49, 0.53. Two workgroups on a CU lose: BF16 N = 250, R =
// 4096 0.97, 1.63, FP32 N = 100, R = 4096 1.30, 2.19.
inline SmallSplit small_split(bool fp64, int waves, int R, int cus) {
  SmallSplit s{1, 1};
  if (fp64 && (R + 15) / 16 <= cus && waves <= 2) s.split = 4 / waves;
  if (fp64 && s.split == 1 && 4 * R <= 16 * cus) s.ls = 4;
  else if (2 * R <= 16 * cus) s.ls = 2;
  return s;
}

}  // namespace nmfa
