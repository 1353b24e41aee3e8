// Plans of the dense projections, host code only: which kernel of k_gemm.hip a product runs in, its block
// tile and its K split.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace rollpack {

constexpr int kGBK = 64;  // K elements of a step (k_gemm_tiled) or unit (k_gemm_deep, k_gemm_ring)
constexpr int kMaxSplitsAny = 64;

enum GemmKernel { kKNone, kKTiled, kKF32, kKDeep, kKRing };

struct GemmPlan {
  int kernel = kKNone;
  int splits = 1;
  int R = 0, D = 0;  // k_gemm_deep, k_gemm_ring: weight fragments per block; k_gemm_deep: register stages
  int bm = 256;      // k_gemm_tiled: activation rows per block tile
  int bn = 256;      // k_gemm_tiled: weight rows per block tile
  int n_first = 0;   // k_gemm_tiled: columns of the first launch; the rest run in bm2 x bn2 tiles
  int bm2 = 256, bn2 = 256;
};

// The (R, D) pairs of k_gemm_deep.
struct DeepCfg { int R, D; };
constexpr DeepCfg kDeepCfg[] = {
    {10, 2}, {8, 2}, {4, 4},
};

// Number of K splits that leaves no split empty, for a wish of `want`.
inline int even_splits(int n_units, int want) {
  if (want < 1) want = 1;
  if (want > n_units) want = n_units;
  const int per = (n_units + want - 1) / want;
  return (n_units + per - 1) / per;
}

// k_gemm_deep plan.  The blocks hold one CU each (their register use
// allows one wave per SIMD), so the time is set by the busiest CU: rounds of
// 256 blocks times the rows x K units of one block.  The K split is the
// largest that keeps all blocks in one round and every wave at >= 3 units, of
// those in [split_lo, split_hi] (equal ends: that split as it is);
// a small penalty for activation traffic (1 / R of the weight loads)
// breaks ties toward more weight rows per block.  Measured on the Qwen2.5
// 7B decode shapes, this picks the best swept configuration or one within
// a few percent of it.
inline GemmPlan plan_deep(int N, int K, bool silu, int split_lo, int split_hi) {
  const int KU = K / 64, units = N / 16;
  GemmPlan best{kKDeep, 1};
  double best_cost = 1e300;
  for (const DeepCfg& c : kDeepCfg) {
    const int per = silu ? c.R / 2 : c.R;
    const int nb = (units + per - 1) / per;
    int S = split_lo;
    if (split_lo < split_hi) {
      const int smax = std::max(1, std::min(std::min(16, split_hi), KU / 12));
      while (S < smax && nb * (S + 1) <= 256) ++S;
      S = even_splits(KU, S);
    }
    const int rounds = (nb * S + 255) / 256;
    const double cost = static_cast<double>(rounds) * c.R * 16 * ((KU + S - 1) / S) * (1.0 + 0.15 / c.R);
    if (cost < best_cost) {
      best_cost = cost;
      best = GemmPlan{kKDeep, S, c.R, c.D};
    }
  }
  return best;
}

// k_gemm_ring plan: fragments per block and K split, priced in us.  A launch takes what its fullest CU does
// (rounds of 256 blocks, whose rings fill a CU's LDS: the units of a wave with their fragments and
// activation tiles, the reduction) and what the weights take at the HBM rate, neither hiding quite behind the
// other (root of the squares), plus the fp32 partials and a little per plane of them.  Fitted to a sweep of all R and splits 1-16 at
// 1-64 rows of the 7B, 0.5B and 32B projections and heads: 0.5% from the fastest in the geometric mean, at
// most 5%.  Splits are those in [split_lo, split_hi] that leave none empty; equal ends: that split as it is.
inline GemmPlan plan_ring(int M, int N, int K, bool silu, int split_lo, int split_hi, bool* one_round = nullptr) {
  const int KU = K / 64, units = N / 16, mt = (M + 15) / 16;
  const double hbm = static_cast<double>(N) * K * (silu ? 4 : 2) / 7.2e6;
  GemmPlan best{kKRing, 1};
  double best_cost = 1e300;
  for (int R : {2, 4, 6, 8, 10}) {
    const int per = silu ? R / 2 : R;
    const int nb = (units + per - 1) / per;
    const int s_max = split_lo == split_hi ? split_hi : std::max(split_lo, std::min(std::min(16, split_hi), KU / 4));
    for (int S = split_lo; S <= s_max; ++S) {
      if (split_lo < split_hi && even_splits(KU, S) != S) continue;
      const int rounds = (nb * S + 255) / 256, wave_units = ((KU + S - 1) / S + 3) / 4;
      const double cu = rounds * (wave_units * 0.115 * (R + mt) + 0.068 * R * mt + 1.4);
      const double cost = std::sqrt(cu * cu + hbm * hbm) + (silu ? 0.0 : S * (static_cast<double>(M) * N * 2.5e-6 + 0.15));
      if (cost < best_cost) {
        best_cost = cost;
        best = GemmPlan{kKRing, S, R};
        if (one_round) *one_round = rounds == 1;
      }
    }
  }
  return best;
}

// k_gemm_tiled plan: the block tile (BM activation rows x BN weight rows) and
// the K split, each tile shape and split in [split_lo, split_hi] priced as
// rounds of 256 blocks (one per CU) x (a start and an end + K steps of a block
// x the tile's price per step), plus the fp32 partials the split writes and its
// consumer reads.  128 x 128 tiles run two blocks per CU, alone when the last
// round has no more than one block per CU.  Fitted to a sweep of single
// launches, all tile shapes and splits 1-16 at 70-9,216 rows of the 7B, 0.5B and 32B
// projections: the plans are 1.0% from the fastest in the geometric mean and at most 8%.
// The prices rank plans; they are not the times of launches in a step, at the clock that
// the chip holds there and with cold weights: 7B gate/up at 9,216 rows is priced at 1,313
// and takes 1,937 us, at 397 rows 97 and 128-132, 0.5B gate/up at 256 rows 8.8 and
// 13.4.  Partials and the second launch below are in us, so that beside them the
// products count 1.3-1.7 times too little.
// An unsplit product may run as two launches: the columns that fill whole rounds
// of 256 x 256 tiles, and the rest in the tile that is fastest for them, instead
// of a nearly empty last round (7B gate/up at 257-512 rows is 296 tiles on 256
// CUs: 128 against 154 us at 397 rows, 136 against 163 at 512; 0.5B gate/up at 2,000
// rows 42.6 against 49.1).
struct Tile { int bm, bn; double ends, step; };
constexpr Tile kTiles[] = {{256, 256, 1.5, 1.09}, {256, 128, 5.5, 0.654}, {128, 256, 5.5, 0.654}, {128, 128, 1.0, 0.955}};
constexpr double kSecondLaunchUs = 2.5;

// Weight rows of a tile panel are bn, of which a SiLU product makes bn / 2 outputs.
inline int panels(int n, int bn, bool silu) { return silu ? (2 * n + bn - 1) / bn : (n + bn - 1) / bn; }

inline double tile_cost(const Tile& c, int M, int N, bool silu, int splits, int steps) {
  const int items = panels(N, c.bn, silu) * ((M + c.bm - 1) / c.bm) * splits;
  if (c.bm != 128 || c.bn != 128) return (items + 255) / 256 * (c.ends + steps * c.step);
  const int rem = items % 512;
  double cost = (items / 512) * (c.ends + steps * c.step);
  if (rem) cost += c.ends + steps * (rem <= 256 ? 0.556 : c.step);
  return cost;
}

inline GemmPlan plan_tiled(int M, int N, int K, bool silu, int split_lo, int split_hi) {
  const int KB = K / kGBK;
  GemmPlan best{kKTiled, 1};
  double best_cost = 1e300;
  for (int sp = split_lo; sp <= split_hi; ++sp) {
    if (split_hi > split_lo && even_splits(KB, sp) != sp) continue;
    const int steps = (KB + sp - 1) / sp;
    const double part = silu ? 0.0 : sp * static_cast<double>(M) * N * 8 / 4.2e6;
    auto take = [&](double cost, int bm, int bn, int n_first, const Tile& rest) {
      if (cost + part >= best_cost) return;
      best_cost = cost + part;
      best = GemmPlan{kKTiled, sp, 0, 0, bm, bn, n_first, rest.bm, rest.bn};
    };
    for (const Tile& c : kTiles) take(tile_cost(c, M, N, silu, sp, steps), c.bm, c.bn, N, c);
    const Tile& big = kTiles[0];
    const int n_mb = (M + big.bm - 1) / big.bm, tiles = n_mb * panels(N, big.bn, silu);
    if (sp == 1 && tiles > 256) {
      const int n_first = 256 * (tiles / 256) / n_mb * (silu ? big.bn / 2 : big.bn);  // whole panels of whole rounds
      if (n_first > 0 && n_first < N)
        for (const Tile& c : kTiles)
          take(tile_cost(big, M, n_first, silu, 1, steps) + tile_cost(c, M, N - n_first, silu, 1, steps) + kSecondLaunchUs,
               big.bm, big.bn, n_first, c);
    }
  }
  return best;
}

// Kernel and split choice, from sweeps of the Qwen2.5 decode shapes on
// gfx950 (weights cycled through more than the 256 MB last-level cache so
// that none is reused between launches):
//  * 17-64 rows: the LDS-ring kernel throughout.  At 64 rows gate/up of the 7B
//    takes 47.6 against 61.9 us for the register ring, the 0.5B head 78.7
//    against 111 us, the 0.5B q/k/v and o 5.2 against 9.8 us for the streaming
//    kernels; at 17-32 rows the gains are 0-10% at 7B and 40% at 0.5B.
//  * with row-major weights the same kernels: four layers of the 0.5B take 151 us at
//    one row and 185 at 64 against 174 and 290 for the kernels before the ring, of
//    the 7B 489 and 586 against 520 and 780, two of the 32B 446 and 520 against 457
//    and 706; no row count from 1 to 64 is slower.
//  * up to 16 rows: the ring for products under 14M weights: alone and with
//    warm weights it ties with kernels that stream weights and activations
//    straight into registers, but within a step, whose weights come from HBM
//    every time, it keeps more of them in flight (the 0.5B model at 1-16 rows
//    0.91-0.99 ms a step against 1.02-1.04).  And the ring where one round of
//    blocks covers a product of 60M weights and more (7B gate/up 45.0 against
//    45.8 us, 32B down 44.1 against 46.2), or from nine rows of 25M and more (two
//    layers of the 32B model 405.9 against 409.1 us at 12 rows, 411.1 against
//    416.1 at 16; at one row 401.3 against 398.4).  Else the register ring, which
//    also runs several blocks per CU (the 0.5B head takes 44 against 52 us; 7B
//    q/k/v 8.7 against 9.4).  With a split that is not the planner's own (an
//    unsplit head) the register ring, of four fragments and more a block, can leave
//    most CUs idle: below 128 of its blocks the LDS ring's two fragments win (a
//    head of 4,864 x 5,120: 76 blocks, 17.4 against 13.3 us at one row, 20.4
//    against 14.9 at 16; of 8,320 x 3,584: 130 blocks, 14.7 against 15.2 and 16.6
//    against 16.4).
inline GemmPlan make_plan(int bf16, int M, int N, int K, bool silu, int split_lo, int split_hi) {
  if (!bf16) return {kKF32, 1};
  if (M > 64) {
    if (split_lo < split_hi) split_hi = std::max(split_lo, std::min(std::min(16, split_hi), K / kGBK / 2));
    return plan_tiled(M, N, K, silu, split_lo, split_hi);
  }
  const double work = static_cast<double>(N) * K * (silu ? 2 : 1);
  bool one_round = false;
  const GemmPlan ring = plan_ring(M, N, K, silu, split_lo, split_hi, &one_round);
  if (M > 16 || work < 1.4e7 || (one_round && work >= (M > 8 ? 2.5e7 : 6.0e7))) return ring;
  const GemmPlan deep = plan_deep(N, K, silu, split_lo, split_hi);
  const int per = silu ? deep.R / 2 : deep.R, blocks = (N / 16 + per - 1) / per * deep.splits;
  return split_lo == split_hi && !silu && blocks < 128 ? ring : deep;
}

// The plan of a shape for a split in [split_lo, split_hi] (SiLU products: 1), remembered per thread (16 sets of
// four, the oldest replaced): a decode step asks for the same few shapes in every layer, and pricing one takes
// 1-2 us of the host's time per launch.
inline GemmPlan plan_gemm(int bf16, int M, int N, int K, bool silu, int split_lo, int split_hi) {
  struct Entry { int bf16 = -1, M = 0, N = 0, K = 0, silu = 0, lo = 0, hi = 0; GemmPlan plan{}; };
  struct Set { Entry e[4]; unsigned next = 0; };
  thread_local Set memo[16];
  if (silu) split_lo = split_hi = 1;
  uint64_t h = (static_cast<uint64_t>(static_cast<uint32_t>(M)) << 32 | static_cast<uint32_t>(N)) * 0x9e3779b97f4a7c15ull;
  h = (h ^ static_cast<uint64_t>(static_cast<uint32_t>(K)) << 8 ^ static_cast<uint64_t>((split_hi * 64 + split_lo) * 2 + silu)) *
      0xd1342543de82ef95ull;
  Set& set = memo[h >> 60];
  for (const Entry& e : set.e)
    if (e.bf16 == bf16 && e.M == M && e.N == N && e.K == K && e.silu == silu && e.lo == split_lo && e.hi == split_hi)
      return e.plan;
  Entry& e = set.e[set.next++ & 3];
  e = Entry{bf16, M, N, K, silu, split_lo, split_hi, make_plan(bf16, M, N, K, silu, split_lo, split_hi)};
  return e.plan;
}

// The plan of a launch that has `splits` K splits: the planner's own where that is its choice, else the best for
// the split it has.  (The LM head is never split, and a small workspace caps the split: with the fragments per block of
// the planner's own split such a launch leaves CUs idle.  The 4,864 x 5,120 head at 45 rows takes 19.7 us against 25.9
// with the fragments of a plan for three splits, the 8,320 x 3,584 one 21.1 against 24.9.)
inline GemmPlan plan_launch(int bf16, int M, int N, int K, bool silu, int splits) {
  if (M <= 64) {
    const GemmPlan own = plan_gemm(bf16, M, N, K, silu, 1, kMaxSplitsAny);
    if (own.splits == splits) return own;
  }
  return plan_gemm(bf16, M, N, K, silu, splits, splits);
}

}  // namespace rollpack
