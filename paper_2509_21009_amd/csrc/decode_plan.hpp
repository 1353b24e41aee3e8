// How a decode step's cached keys are cut into attention items, host code only.
#pragma once

#include <algorithm>
#include <cstdint>

namespace rollpack {

// Attention items of a step: at most this many and one more per row (the workspace holds so many partials).
inline int decode_split_target(int n_kv) { return std::max(1, 2048 / n_kv); }

// Items of one row at most: the merge kernel keeps their maxima and sums in LDS.
constexpr int kMaxRowItems = 512;

// Pages of cached keys per decode attention item.  An item is a block of four waves; two blocks fit a CU,
// which moves a page of one head (K and V, 32 KB at head_dim 128) in about 1.3 us whether it runs one
// block or two.  The cost of a size, in us: the fullest CU's pages and the items' own ends (2.5 us each),
// plus, when some row has more than one item, the merge (4.5 us).  Over sizes forced from 1 page to
// whole rows at 1-330 rows of 64-12,000 tokens (7B, 0.5B and 32B layers) its choices are within 1-2% of
// the fastest step; the optimum is flat.  (A row of 65,536 tokens gets 256 items at most: kMaxRowItems
// binds no choice.)
inline int decode_pages_per_item(int n_kv, int head_dim, int64_t total_pages, int64_t max_pages, int B) {
  const double page_us = head_dim == 128 ? 1.3 : 0.65, ends_us = 2.5, merge_us = 4.5;
  const int64_t target = decode_split_target(n_kv);  // the item capacity: total_pages / pps + B items at most
  const int64_t least = std::max<int64_t>({1, (total_pages + target - 1) / target, (max_pages + kMaxRowItems - 1) / kMaxRowItems});
  int64_t best = std::max(least, max_pages);
  double best_us = 1e300;
  for (int64_t pps = least;; pps += std::max<int64_t>(1, pps / 8)) {
    pps = std::min(pps, std::max(least, max_pages));
    const bool merge = pps < max_pages;
    const double items = merge ? (static_cast<double>(total_pages) / pps + 0.5 * B) * n_kv : static_cast<double>(B) * n_kv;
    const double one = pps * page_us + ends_us;
    const double all = (static_cast<double>(total_pages) * n_kv * page_us + items * ends_us) / 256;
    // up to one block per CU the longest item ends the step; past that the CUs even out to half an item
    const double us = (items <= 256 ? one : std::max(one, all + 0.5 * one)) + (merge ? merge_us : 0.0);
    if (us < best_us) {
      best_us = us;
      best = pps;
    }
    if (pps >= max_pages) break;
  }
  return static_cast<int>(best);
}

}  // namespace rollpack
