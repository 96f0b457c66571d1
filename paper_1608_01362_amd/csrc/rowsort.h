// Relabelling and sorting of CSC rows under a vertex renumbering (rowsort.hip):
// the edge step of the clustering.
#pragma once

#include "common.h"

namespace cagra {

size_t row_sort_ws_bytes(int32_t V, int64_t E);

// out[new_off[i] .. new_off[i + 1]) = the new ids inv[u] of the sources u of old
// row perm[i], ascending, for every new row i. cum: exclusive prefix sums of
// the new out-degrees (any values are allowed: they only steer the work); total
// = their sum's last term, outdeg_new[V - 1]. E > 0.
cagra_status sort_rows(const int32_t *in_offsets, const int32_t *in_sources, int32_t V, int64_t E,
                       const int32_t *perm, const int32_t *inv, const int32_t *new_off, const int32_t *cum,
                       const int32_t *outdeg_new, int32_t *out, void *ws, size_t ws_bytes, hipStream_t st);

}  // namespace cagra
