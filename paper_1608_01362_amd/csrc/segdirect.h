// Segment-major reorder of the in-edge CSC in one counting and one scattering
// pass (segdirect.hip): what the segment builder calls.
#pragma once

#include "common.h"

namespace cagra {

// Most segments of the one-pass form; more go through two digit passes.
constexpr int32_t kDirectMaxSegments = 2048;

// First row of every group of kGroupEdges consecutive edges: rows[g] is the row
// that edge g * kGroupEdges belongs to, rows[number of groups] = V - 1.
constexpr int kGroupEdges = 1024;
int64_t edge_groups(int64_t E);
cagra_status launch_group_rows(const int32_t *in_offsets, int32_t V, int64_t E, int32_t *rows, hipStream_t st);

// Query pass: seg_edges[k] (cleared by the caller) += edges per segment,
// *runs += subgraph rows.
cagra_status launch_count_runs(const cagra_graph *g, int32_t N, int32_t k, const int32_t *rows, int32_t *seg_edges,
                               unsigned long long *runs, hipStream_t st);

// Build pass for k <= kDirectMaxSegments and E > 0: edge_src, row_ptr, row_dst,
// row_dst_lo and seg_row_begin of seg.
size_t direct_ws_bytes(int64_t E, int32_t k);
cagra_status build_direct(const cagra_graph *g, const cagra_segments *seg, void *ws, size_t ws_bytes,
                          hipStream_t st);

}  // namespace cagra
