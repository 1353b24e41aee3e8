// Host-only checks of the KV page pool, the tail-batching planner, the GEMM plans and the decode attention
// items, built
// with g++ and AddressSanitizer/UndefinedBehaviorSanitizer by the CPU tests.
#include <cassert>
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <set>
#include <stdexcept>
#include <vector>

#include "decode_plan.hpp"
#include "gemm_plan.hpp"
#include "kv_pool.hpp"
#include "tail_batch.hpp"

using rollpack::PagePool;

static int failures = 0;
#define CHECK(c)                                                  \
  do {                                                            \
    if (!(c)) {                                                   \
      std::fprintf(stderr, "CHECK failed %s:%d: %s\n", __FILE__, __LINE__, #c); \
      ++failures;                                                 \
    }                                                             \
  } while (0)

static void test_pool_random() {
  std::mt19937 rng(7);
  PagePool pool(257);
  std::vector<std::vector<int32_t>> owned(20);
  for (int it = 0; it < 20000; ++it) {
    const int o = rng() % 20;
    if (rng() % 2) {
      const int64_t want = rng() % 40;
      const int64_t before = pool.free_pages();
      try {
        pool.take(want, o, owned[o]);
        CHECK(pool.free_pages() == before - want);
      } catch (const std::runtime_error&) {
        CHECK(want > before);
        CHECK(pool.free_pages() == before);  // no side effect on failure
      }
    } else {
      pool.give_back(owned[o], o);
      owned[o].clear();
    }
    // conservation and exclusive ownership
    int64_t held = 0;
    std::set<int32_t> seen;
    for (int k = 0; k < 20; ++k) {
      held += owned[k].size();
      for (int32_t p : owned[k]) {
        CHECK(seen.insert(p).second);
        CHECK(pool.owner_of(p) == k);
      }
    }
    CHECK(held + pool.free_pages() == pool.capacity());
    CHECK(pool.peak_used() >= pool.used_pages());
  }
  for (int k = 0; k < 20; ++k) pool.give_back(owned[k], k);
  CHECK(pool.free_pages() == pool.capacity());
}

static void test_pool_misuse() {
  PagePool pool(4);
  std::vector<int32_t> a, b;
  pool.take(2, 1, a);
  bool threw = false;
  try { pool.give_back(a, 2); } catch (const std::logic_error&) { threw = true; }
  CHECK(threw);
  CHECK(pool.free_pages() == 2);
  threw = false;
  try { pool.take(3, 2, b); } catch (const std::runtime_error&) { threw = true; }
  CHECK(threw && b.empty());
  CHECK(PagePool::pages_for(0, 64) == 0 && PagePool::pages_for(1, 64) == 1 && PagePool::pages_for(64, 64) == 1 &&
        PagePool::pages_for(65, 64) == 2);
}

static void test_plan_invariants() {
  std::mt19937 rng(11);
  for (int it = 0; it < 300; ++it) {
    const int P0 = 1 + rng() % 6, R0 = 1 + rng() % 4, n = rng() % 40;
    const double eta = 1.25;
    const int r_spec = static_cast<int>(std::ceil(eta * R0 - 1e-9));
    std::vector<int32_t> lens(static_cast<size_t>(n) * r_spec);
    for (auto& L : lens) L = 1 + rng() % 500;
    auto plan = rollpack::plan_tail_batching(n, r_spec, lens.data(), P0, R0, eta, eta);
    std::vector<int> accepted(n, 0);
    for (const auto& r : plan.rounds) {
      for (int32_t p : r.accepted) accepted[p]++;
      CHECK(r.run_steps.size() == r.launched.size() * r_spec);
      if (r.kind == 1) CHECK(r.accepted == r.launched);
      else CHECK(static_cast<int>(r.accepted.size()) == std::min<int>(P0, r.launched.size()));
    }
    for (int p = 0; p < n; ++p) {
      CHECK(accepted[p] == 1);
      int kept = 0;
      for (int r = 0; r < r_spec; ++r) kept += plan.kept[static_cast<size_t>(p) * r_spec + r];
      CHECK(kept == R0);
    }
  }
}

// A launch whose split is not the planner's own is planned for the split it has.
static void test_gemm_plan_for_the_launched_split() {
  using namespace rollpack;
  // an unsplit head: two fragments per block give 152 blocks where the plan for three splits would leave 76
  CHECK(plan_launch(1, 45, 4864, 5120, false, 1).R == 2);
  CHECK(plan_launch(1, 64, 8320, 3584, false, 1).R == 4);
  CHECK(plan_launch(1, 8, 4864, 5120, false, 1).kernel == kKRing && plan_launch(1, 8, 8320, 3584, false, 1).kernel == kKDeep);
  std::mt19937 rng(5);
  for (int it = 0; it < 4000; ++it) {
    const int M = 1 + rng() % 600, N = 128 * (1 + rng() % 400), K = 128 * (1 + rng() % 160);
    const bool silu = rng() % 4 == 0;
    const GemmPlan own = plan_gemm(1, M, N, K, silu, 1, kMaxSplitsAny);
    CHECK(own.splits == 1 || !silu);
    CHECK(own.splits == even_splits(K / kGBK, own.splits) && own.splits <= 16);
    const int cap = 1 + rng() % 16, s = silu ? 1 : plan_gemm(1, M, N, K, false, 1, cap).splits;
    CHECK(s <= cap || s == 1);
    const GemmPlan p = plan_launch(1, M, N, K, silu, s);
    CHECK(p.splits == s);
    if (s == own.splits) {
      CHECK(p.kernel == own.kernel && p.R == own.R && p.D == own.D && p.bm == own.bm && p.bn == own.bn &&
            p.n_first == own.n_first);
      continue;
    }
    // else the planner's choice at that split
    if (p.kernel == kKRing) {
      const GemmPlan ring = plan_ring(M, N, K, silu, s, s);
      CHECK(ring.R == p.R && ring.splits == s);
    } else if (p.kernel == kKDeep) {
      CHECK(M <= 16 && plan_deep(N, K, silu, s, s).R == p.R);
    } else {
      CHECK(p.kernel == kKTiled && M > 64 && (p.n_first == N || s == 1));
    }
  }
}

// Attention items stay within the workspace's capacity for any contexts.
static void test_decode_items_fit() {
  std::mt19937 rng(13);
  for (int it = 0; it < 20000; ++it) {
    const int n_kv = 1 << rng() % 5, hd = rng() % 2 ? 64 : 128, B = 1 + rng() % (it % 8 ? 16 : 400);
    const int64_t most = 1 + rng() % (it % 2 ? 1024 : 64);
    std::vector<int64_t> pages(B);
    int64_t total = 0, longest = 0;
    for (auto& p : pages) {
      p = 1 + rng() % most;
      total += p;
      longest = std::max(longest, p);
    }
    const int64_t pps = rollpack::decode_pages_per_item(n_kv, hd, total, longest, B);
    CHECK(pps >= 1);
    int64_t items = 0;
    for (int64_t p : pages) {
      CHECK((p + pps - 1) / pps <= rollpack::kMaxRowItems);
      items += (p + pps - 1) / pps;
    }
    CHECK(items <= rollpack::decode_split_target(n_kv) + B);
  }
}

int main() {
  test_decode_items_fit();
  test_gemm_plan_for_the_launched_split();
  test_pool_random();
  test_pool_misuse();
  test_plan_invariants();
  if (failures) {
    std::fprintf(stderr, "%d failures\n", failures);
    return 1;
  }
  std::printf("host tests passed\n");
  return 0;
}
