// What the autotuner times for the gradient forms (host code on the public C ABI).
#pragma once

#include <set>
#include <utility>
#include <vector>

#include "nr.h"

namespace nr {

// (bucket, variant) pairs to try in place of NR_VARIANT_AUTO, for the buckets
// that the batch uses: both forms where both exist, and the recompute form of
// the other NR_F64 buckets, whose default may be the form that chooses per node.
// Items beyond NR_MAX_LAYERS follow the last bucket's entry.
inline std::vector<std::pair<int, int>> form_candidates(const nr_batch_desc* d) {
  std::set<int> used;
  for (int i = 0; i < d->n_items; ++i) {
    const int L = (int)(d->row_off[i + 1] - d->row_off[i]) - 2;
    int k = 0;
    while (k + 1 < NR_NUM_BUCKETS && L > nr_bucket_lmax(k)) ++k;
    used.insert(k);
  }
  std::vector<std::pair<int, int>> out;
  const int smax = nr_store_max_layers(d->precision);
  for (int k : used) {
    const bool store = nr_bucket_lmax(k) <= smax;
    if (store) out.push_back({k, NR_VARIANT_STORE});
    if (store || d->precision == NR_F64) out.push_back({k, NR_VARIANT_RECOMPUTE});
  }
  return out;
}

}  // namespace nr
