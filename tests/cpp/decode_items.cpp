// The engine's decode attention items, for tests that have to know which path a step takes.
#include "decode_plan.hpp"

// Pages of cached keys per item for B rows of these contexts (the newest token included, which is not cached yet).
extern "C" int pages_per_item(int n_kv, int head_dim, const int* ctx, int B) {
  int64_t total = 0, longest = 0;
  for (int i = 0; i < B; ++i) {
    const int64_t p = (ctx[i] - 1 + 63) / 64;
    total += p;
    longest = std::max(longest, p);
  }
  return rollpack::decode_pages_per_item(n_kv, head_dim, total, longest, B);
}
