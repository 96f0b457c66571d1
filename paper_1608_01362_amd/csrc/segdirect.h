// Segment-major reorder of the in-edge CSC in one counting and one scattering
// pass (segdirect.hip): what the segment builder calls.
#pragma once

#include "common.h"

namespace cagra {

// Most segments of the one-pass form; more go through two digit passes.
constexpr int32_t kDirectMaxSegments = 2048;

// The non-empty rows of a CSC in order, and for every unit of `unit` consecutive
// edges the list index of the row its first edge belongs to (first[number of
// units] = the last index). A unit's row starts lie between its first index and
// the next unit's, so finding them takes no longer however many empty rows lie
// in between.
struct RowList {
    int32_t *row, *start;  // row id and first edge
    int32_t *first;
    int32_t *count;        // scanned counts of nonempty rows per block of rows; the last entry is their number
};
size_t row_list_ws_bytes(int32_t V, int64_t E, int32_t unit);
// Takes the list's arrays from ar and fills them; E > 0.
cagra_status build_row_list(const int32_t *offsets, int32_t V, int64_t E, int32_t unit, Arena &ar, RowList *list,
                            hipStream_t st);

constexpr int kGroupEdges = 1024;  // edges a wave of the builder looks at together

// Query pass: seg_edges[k] (cleared by the caller) += edges per segment,
// *runs += subgraph rows.
cagra_status launch_count_runs(const cagra_graph *g, int32_t N, int32_t k, const RowList &rows, int32_t *seg_edges,
                               unsigned long long *runs, hipStream_t st);

// Build pass for k <= kDirectMaxSegments and E > 0: edge_src, row_ptr, row_dst,
// row_dst_lo and seg_row_begin of seg.
size_t direct_ws_bytes(int32_t V, int64_t E, int32_t k);
cagra_status build_direct(const cagra_graph *g, const cagra_segments *seg, void *ws, size_t ws_bytes,
                          hipStream_t st);

}  // namespace cagra
