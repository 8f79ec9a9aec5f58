// Output tile and K split of a bf16 GEMM launch: host code without any
// dependency, so that tests can compile it by itself.
#pragma once

#include <stdint.h>

namespace acid {

constexpr int kGemmTile = 256, kGemmStep = 64;  // the largest tile's sides; K per step
constexpr int64_t kSplitMaxItems = 256;         // work items the split workspace holds

enum class Tile { k256, k256x128, k128, k64 };
// What a launch's epilogue does with the tile: fp32 stores, GELU, a
// read-modify-write of fp32 rows, or the Q | K | V split.
enum class Out { kPlain, kGelu, kUpdate, kHeads };
struct Form {
  Tile tile;
  int split;    // of a ring tile's K range, or of the 256 x 256 tail tiles'
  int64_t rem;  // k256 with split > 1: the tail tiles
};

// K split of the last round's tiles: when the tiles beyond whole rounds of
// the device's CUs would leave at least half of them idle, those `rem` tiles
// are split into S K ranges (S <= 8, S * rem within the CUs and the 256 work
// items the workspace holds, each range a multiple of 128).  Each range is at
// least 2048 long: a work item also fills the staging ring and writes its
// 256 KB of partial sums, which the reduction reads back, and with shorter
// ranges that costs more than the fuller round saves (measured: split into
// K ranges of 256-1024, the small configuration's GEMMs ran twice as long).
inline int choose_split(int64_t tiles, int K, int64_t cus, int64_t& rem) {
  rem = tiles % cus;
  if (rem == 0 || 2 * rem > cus) return 1;
  int S = (int)(cus / rem);
  if (S > 8) S = 8;
  while (S > 1 && (rem * S > kSplitMaxItems || K % (S * 128) != 0 || K / S < 2048)) --S;
  return S;
}

// The form with the least estimated time, in microseconds: once + rounds of
// the CUs x (a + b x K-steps of 64).  A round that is not full counts in part
// (it overlaps the one before); a depends on the epilogue, b on the share of the
// CUs at work and on the launch's length (the clock falls under the power cap);
// the rows of a ragged last row tile cost the Q | K | V split 15 us per 256
// (2-byte stores of V^T under a guard), an update 2.  The constants are those
// that lose least against the best form of each of 16843 measured launches:
// blocks' products in place, with and without a K split, and products with each
// epilogue; 16 to 119056 rows, N 128 to 25000, K 128 to 17000.  On 5615 others the
// choices take 0.7% more than the best form (over 10% more in 2%), and 0.2% of
// them over 5% more than 256 x 256 tiles alone.
// Microseconds, 256 x 256 / 256 x 128 / 128 x 128 / 64 x 64:
//    256 x  3072 x  1024:  25.5 /  20.2 /  14.4 /   9.0
//   1000 x  8960 x  1536:  41.2 /  51.2 /  58.7 /  60.6
//   1560 x  1536 x  1536:  35.9 /  24.3 /  18.4 /  21.3
//   1560 x  4608 x  1536:  36.2 /  30.3 /  36.6 /  44.3
//   4000 x 12288 x  3072: 251.0 / 295.7 / 357.0 / 473.9
//   8200 x  1536 x   128:  13.9 /  16.4 /  18.7 /  18.1
//  24000 x   640 x  3072: 122.5 /  85.1 / 103.2 / 142.5
//  60000 x  2176 x   128: 118.3 / 138.8 / 161.6 / 182.5
// 119056 x  8960 x   128:   824 /   949 /  1092 /  1357
//   2780 x  3456 x  1536:  59.1 /  51.4 /  43.4 /  47.6 (Q | K | V, 220 ragged rows)
// With a workspace the K range of a ring tile may be split too, where all
// items fit one round: 64 rows x 1536 x 8960 45.1 -> 18.3 us, 300 rows 40.7
// -> 26.4, 1000 rows 72.5 -> 43.7, 1560 rows 65.8 -> 59.0.  The second pass
// costs about 6 us and its bytes at 4 TB/s.  Every tile without a split gives
// the same bits.
inline Form choose_form(Out out, int64_t M, int N, int K, bool have_ws, int64_t cus) {
  // by epilogue: per round, and per 256 ragged rows
  static constexpr double kOut[4][4] = {
      {0, 0, 0, 0}, {1.0, 0.2, 0, 0}, {2.4, 1.2, 0.2, 0.05}, {3.3, 1.1, 0.55, 0.12}};
  static constexpr double kRagged[4] = {0, 0, 2, 15};
  // A smaller tile has to promise 8%: with less it is as often the slower one.
  constexpr double kMargin = 1.08;
  const int steps = K / kGemmStep, o = (int)out;
  const double tflop = 2e-12 * M * N * K, length = tflop < 0.38 ? tflop / 0.38 : 1;
  auto second_pass = [](int64_t items, int area) { return 6.0 + items * area * 1e-6; };
  Form f = {Tile::k256, 1, 0};
  double best = 0;
  // part: how much of a partly filled round overlaps the one before it; the time
  // of a K-step is b, + c with every CU at work, + d in a long launch
  auto consider = [&](Tile t, int tm, int tn, double once, double a, double b, double c, double d,
                      double part) {
    a += kOut[o][(int)t];
    const int64_t n = (M + tm - 1) / tm * ((N + tn - 1) / tn);
    const double x = (double)n / cus;
    const double rounds = (1 - part) * (double)((n + cus - 1) / cus) + part * (x > 1 ? x : 1);
    double whole = once + rounds * (a + (b + c * (x < 1 ? x : 1) + d * length) * steps) +
                   kRagged[o] * (double)(M % tm) / 256;
    if (t == Tile::k256) {
      if (have_ws) f.split = choose_split(n, K, cus, f.rem);
      if (f.split > 1)  // the last round takes a part of its K-steps
        whole += second_pass(f.rem * f.split, tm * tn) - b * (steps - steps / f.split);
      best = whole / kMargin;
      return;
    }
    if (whole < best) {
      best = whole;
      f = {t, 1, 0};
    }
    if (!have_ws) return;
    for (int sp = 2; sp <= 8; ++sp) {
      if (n * sp > cus || n * sp > kSplitMaxItems || steps / sp < 8) break;
      const double cost = once + a +
                          (b + c * (x * sp < 1 ? x * sp : 1) + d * length) * ((steps + sp - 1) / sp) +
                          second_pass(n * sp, tm * tn);
      if (cost < best) {
        best = cost;
        f = {t, sp, 0};
      }
    }
  };
  consider(Tile::k256, 256, 256, 1.5, 7.9, 1.16, 0.23, 0.09, 0.24);
  consider(Tile::k256x128, 256, 128, 0.8, 6.5, 0.59, 0.14, 0.23, 0.22);
  consider(Tile::k128, 128, 128, 2.3, 3.5, 0.355, 0.13, 0.05, 0.22);
  consider(Tile::k64, 64, 64, 3.7, 0.75, 0.213, 0, 0.01, 0.23);
  return f;
}

}  // namespace acid
