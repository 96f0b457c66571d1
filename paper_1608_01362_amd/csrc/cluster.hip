// Frequency-based clustering (Section 5) and relabelling, before segmenting.
//
// 1. Vertex keys: out-degree where it is strictly above the average degree
//    E / V, else 0, stored bit-inverted so that a stable ascending radix sort
//    of (key, id) pairs gives the new order: clustered vertices by out-degree
//    from high to low (ties keep the original order), then every other vertex
//    in its original order.
// 2. inv[perm[i]] = i; new out-degrees and in-degrees follow perm; a scan of
//    the in-degrees gives the new row offsets.
// 3. Every new row takes its old row's sources under their new ids and sorts
//    them (rowsort.hip).
//
// The vertex sort is the stable radix passes of segsort.hip and the scans the
// builder's; clustering runs once per graph, off the iteration's hot path.
#include "common.h"
#include "radix.h"
#include "rowsort.h"

namespace cagra {

__global__ void k_cl_vertex_keys(const int32_t *__restrict__ outdeg, int32_t V, int64_t E,
                                 uint32_t *__restrict__ key, int32_t *__restrict__ id) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V) return;
    const int64_t od = outdeg[v];
    key[v] = ~(od * (int64_t)V > E ? (uint32_t)od : 0u);
    id[v] = (int32_t)v;
}

// inv, the new out-degrees and in-degrees, and the clustered-vertex count.
__global__ void k_cl_relabel(const int32_t *__restrict__ perm, const uint32_t *__restrict__ key_sorted,
                             const int32_t *__restrict__ in_offsets, const int32_t *__restrict__ outdeg, int32_t V,
                             int32_t *__restrict__ inv, int32_t *__restrict__ outdeg_new, int32_t *__restrict__ cnt,
                             int32_t *__restrict__ hot) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > V) return;
    if (i == V) {
        cnt[V] = 0;
        return;
    }
    const int32_t old = perm[i];
    inv[old] = (int32_t)i;
    outdeg_new[i] = outdeg[old];
    cnt[i] = in_offsets[old + 1] - in_offsets[old];
    if (hot) {
        // exactly one writer: the last clustered vertex, or vertex 0 when there is none
        // keys are stored bit-inverted: a clustered vertex has ~key > 0
        const bool last_hot = ~key_sorted[i] > 0u && (i + 1 == V || ~key_sorted[i + 1] == 0u);
        if (last_hot) *hot = (int32_t)(i + 1);
        if (i == 0 && ~key_sorted[0] == 0u) *hot = 0;
    }
}

static unsigned grid_of(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

// Temporary storage: the vertex sort, the scans and the row sort follow each other.
static size_t cluster_temps(int32_t V, int64_t E) {
    size_t n = sort_ws_bytes(V, 32, 4, 4);
    const size_t scan = scan_add_ws_bytes((int64_t)V + 1), rows = E > 0 ? row_sort_ws_bytes(V, E) : 0;
    if (scan > n) n = scan;
    return rows > n ? rows : n;
}

static size_t cluster_layout(int32_t V, int64_t E) {
    ArenaSize a;
    a.take<uint32_t>(V);              // key
    a.take<uint32_t>(V);              // key_sorted
    a.take<int32_t>(V);               // id
    a.take<int32_t>(V);               // inv
    a.take<int32_t>((int64_t)V + 1);  // in-degrees, then the out-degrees' prefix sums
    a.take<char>((int64_t)cluster_temps(V, E));
    return a.used + 256;
}

cagra_status cluster_workspace_bytes(int32_t V, int64_t E, size_t *bytes) {
    *bytes = cluster_layout(V, E);
    return CAGRA_OK;
}

cagra_status cluster_graph(const cagra_graph *g, int32_t *perm, int32_t *in_offsets_new, int32_t *in_sources_new,
                           int32_t *outdeg_new, int32_t *hot, void *ws, size_t ws_bytes, hipStream_t st) {
    const int32_t V = g->V;
    const int64_t E = g->E;
    const size_t need = cluster_layout(V, E);
    if (ws_bytes < need) return fail(CAGRA_E_BUFFER, "cluster workspace needs %zu bytes (got %zu)", need, ws_bytes);
    Arena ar{(char *)ws, ws_bytes, 0};
    uint32_t *key = ar.take<uint32_t>(V);
    uint32_t *key_sorted = ar.take<uint32_t>(V);
    int32_t *id = ar.take<int32_t>(V);
    int32_t *inv = ar.take<int32_t>(V);
    int32_t *cnt = ar.take<int32_t>((int64_t)V + 1);
    const size_t tmp_bytes = cluster_temps(V, E);
    char *tmp = ar.take<char>((int64_t)tmp_bytes);
    if (!key || !key_sorted || !id || !inv || !cnt || !tmp)
        return fail(CAGRA_E_BUFFER, "cluster workspace smaller than %zu bytes", need);

    // 1. new vertex order
    k_cl_vertex_keys<<<grid_of(V, 256), 256, 0, st>>>(g->out_degree, V, E, key, id);
    CAGRA_LAUNCH_CHECK();
    cagra_status s;
    if ((s = radix_sort_stable<uint32_t, int32_t>(key, id, key_sorted, perm, V, 32, tmp, tmp_bytes, st)) != CAGRA_OK)
        return s;
    // 2. relabel vertices, new row offsets
    k_cl_relabel<<<grid_of((int64_t)V + 1, 256), 256, 0, st>>>(perm, key_sorted, g->in_offsets, g->out_degree, V,
                                                                inv, outdeg_new, cnt, hot);
    CAGRA_LAUNCH_CHECK();
    if ((s = scan_add_exclusive(cnt, in_offsets_new, (int64_t)V + 1, tmp, tmp_bytes, st)) != CAGRA_OK) return s;
    if (E == 0) return CAGRA_OK;
    // 3. relabel and sort every row's sources; the out-degrees' prefix sums spread a row's slots
    if ((s = scan_add_exclusive(outdeg_new, cnt, V, tmp, tmp_bytes, st)) != CAGRA_OK) return s;
    return sort_rows(g->in_offsets, g->in_sources, V, E, perm, inv, in_offsets_new, cnt, outdeg_new, in_sources_new,
                     tmp, tmp_bytes, st);
}

}  // namespace cagra
