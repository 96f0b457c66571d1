// The segment-major reorder of Section 3.1 in two passes over the CSC.
//
// Rows and edges arrive in destination order and are regrouped by the segment
// of their sources, keeping destination order inside a segment: a stable
// counting sort with one digit, the segment id (up to 2,048 of them).
//   1. Chunks of consecutive edges count their edges and their runs (subgraph
//      rows) per segment; one device-wide scan of each count matrix, segment by
//      segment, gives every chunk its output positions.
//   2. Every chunk reads its edges again, ranks them and writes each finished
//      edge word, and for each run its destination, block offset and first edge
//      (row_ptr), straight to their places.
// Both passes take groups of 1,024 consecutive edges per wave. A wave marks the
// rows that start in its group (from a list of the non-empty rows) in LDS, so the
// row of an edge is the last mark at or before it, found with ballots; nothing per
// edge is kept in memory between the passes. Source reads are coalesced; each segment's part of a tile
// is staged in LDS by output position and leaves as one contiguous run, and
// consecutive chunks run on one XCD, so that its L2 joins the ends of the runs
// into whole lines.
//
// Bytes: 4 E (count) + 4 E + 2 E + 10 Q (scatter), against some 45 E + 40 Q of
// the sorted form it replaces (row marks, flags, two scans over the edges, keys
// and values through two digit passes). Query and build together, before ->
// now: R-MAT 24 / ef 24 (N = 32,768) 13.2 -> 4.7 ms, R-MAT 25 / ef 32 35.3 ->
// 15.9 ms. The scatter (2.5 ms of the 4.7) is bound by its ranking: 149 VALU
// instructions per 64 edges, 1.4 ms of issue, and the barriers between its
// phases. Timed when it took 4.4 and 14.6 ms: tiles of 4,096 edges (more,
// smaller workgroups) 4.8 and 17.8 ms, chunks of one or two tiles 4.5 and
// 15 ms, the segment match with a bit loop or waits between the steps 4.7 to
// 5.0 ms.
#include "segdirect.h"

#include "radix.h"
#include "wave.h"

namespace cagra {

// u / N for 0 <= u < 2^31 as one high product and a shift (Granlund &
// Montgomery 1994, "Division by invariant integers using multiplication":
// with l = ceil(log2 N), m = floor(2^(31 + l) / N) + 1 < 2^32). N = 1: m = 0
// and u itself added.
struct FastDiv {
    uint32_t m, shift, one;
};
static FastDiv fast_div(int32_t N) {
    if (N <= 1) return {0u, 0u, ~0u};
    int l = 1;
    while ((1ll << l) < (long long)N) ++l;
    return {(uint32_t)((1ull << (31 + l)) / (unsigned long long)N + 1ull), (uint32_t)(l - 1), 0u};
}
__device__ __forceinline__ int32_t quotient(FastDiv f, int32_t u) {
    return (int32_t)((__umulhi((uint32_t)u, f.m) + ((uint32_t)u & f.one)) >> f.shift);
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

constexpr int kSegWaves = 8;
constexpr int kSegThreads = kSegWaves * kWave;
constexpr int kSteps = kGroupEdges / kWave;           // edges per lane and group
constexpr int kTileEdges = kSegWaves * kGroupEdges;   // edges ranked and staged together
constexpr int kMaxChunkTiles = 4;
constexpr int kChunksWanted = 1024;  // below this many chunks a chunk is one tile
constexpr int kChipCus = 256;

// ---- non-empty rows

constexpr int kRlThreads = 256;
constexpr int kRlItems = 8;
constexpr int kRlRows = kRlThreads * kRlItems;  // rows of a workgroup

__global__ __launch_bounds__(kRlThreads) void k_rows_count(const int32_t *__restrict__ off, int32_t V,
                                                           int32_t *__restrict__ count) {
    __shared__ int32_t wsum[kRlThreads / kWave];
    int32_t n = 0;
#pragma unroll
    for (int j = 0; j < kRlItems; ++j) {
        const int64_t r = (int64_t)blockIdx.x * kRlRows + j * kRlThreads + threadIdx.x;
        const bool full = r < V && off[r < V ? r + 1 : 0] > off[r < V ? r : 0];
        n += (int32_t)__builtin_popcountll(ballot(full));
    }
    if (__lane_id() == 0) wsum[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int i = 0; i < kRlThreads / kWave; ++i) t += wsum[i];
        const bool one = gridDim.x == 1;  // a single block is its own scan
        count[blockIdx.x] = one ? 0 : t;
        if (blockIdx.x == gridDim.x - 1) count[gridDim.x] = one ? t : 0;
    }
}

__global__ __launch_bounds__(kRlThreads) void k_rows_list(const int32_t *__restrict__ off, int32_t V, int64_t units,
                                                          int32_t unit, RowList list) {
    __shared__ int32_t cnt[kRlItems][kRlThreads / kWave];
    const int lane = __lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t a[kRlItems], b[kRlItems];
    uint64_t m[kRlItems];
#pragma unroll
    for (int j = 0; j < kRlItems; ++j) {
        const int64_t r = (int64_t)blockIdx.x * kRlRows + j * kRlThreads + threadIdx.x;
        a[j] = off[r < V ? r : V];
        b[j] = off[r < V ? r + 1 : V];
        m[j] = ballot(b[j] > a[j]);
        if (lane == 0) cnt[j][w] = (int32_t)__builtin_popcountll(m[j]);
    }
    __syncthreads();
    int32_t at = list.count[blockIdx.x];
#pragma unroll
    for (int j = 0; j < kRlItems; ++j) {
        int32_t i = at;
        for (int x = 0; x < kRlThreads / kWave; ++x) {
            if (x < w) i += cnt[j][x];
            at += cnt[j][x];
        }
        i += (int32_t)__builtin_popcountll(m[j] & lanemask_lt());
        const bool full = b[j] > a[j];
        const int64_t r = (int64_t)blockIdx.x * kRlRows + j * kRlThreads + threadIdx.x;
        int64_t u0 = 0, u1 = 0;  // units whose first edge the row holds
        if (full) {
            list.row[i] = (int32_t)r;
            list.start[i] = a[j];
            u0 = ceil_div(a[j], unit);
            u1 = ceil_div(b[j], unit);
            if (u1 > units) u1 = units;
        }
        const bool many = u1 - u0 > 8;
        if (!many)
            for (int64_t u = u0; u < u1; ++u) list.first[u] = i;
        for (uint64_t mm = ballot(many); mm; mm &= mm - 1) {  // rows of many units are filled by the wave
            const int l = (int)__builtin_ctzll(mm);
            const int32_t f = __builtin_amdgcn_readlane((int32_t)u0, l), e = __builtin_amdgcn_readlane((int32_t)u1, l);
            const int32_t at_l = __builtin_amdgcn_readlane(i, l);
            for (int32_t u = f + lane; u < e; u += kWave) list.first[u] = at_l;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) list.first[units] = list.count[gridDim.x] - 1;
}

size_t row_list_ws_bytes(int32_t V, int64_t E, int32_t unit) {
    ArenaSize a;
    a.take<int32_t>(V < E ? V : E);
    a.take<int32_t>(V < E ? V : E);
    a.take<int32_t>(ceil_div(E, unit) + 1);
    a.take<int32_t>(ceil_div(V, kRlRows) + 1);
    return a.used + scan_add_ws_bytes(ceil_div(V, kRlRows) + 1) + 512;
}

cagra_status build_row_list(const int32_t *offsets, int32_t V, int64_t E, int32_t unit, Arena &ar, RowList *list,
                            hipStream_t st) {
    const int64_t blocks = ceil_div(V, kRlRows);
    list->row = ar.take<int32_t>(V < E ? V : E);  // at most one row per edge
    list->start = ar.take<int32_t>(V < E ? V : E);
    list->first = ar.take<int32_t>(ceil_div(E, unit) + 1);
    list->count = ar.take<int32_t>(blocks + 1);
    if (!list->row || !list->start || !list->first || !list->count)
        return fail(CAGRA_E_BUFFER, "workspace too small (row list)");
    k_rows_count<<<(unsigned)blocks, kRlThreads, 0, st>>>(offsets, V, list->count);
    CAGRA_LAUNCH_CHECK();
    if (blocks > 1) {
        const size_t at = align_up(ar.used, 256);  // the scan's temporaries are free again afterwards
        if (at > ar.cap) return fail(CAGRA_E_BUFFER, "workspace too small (row list)");
        if (cagra_status s = scan_add_exclusive(list->count, list->count, blocks + 1, ar.base + at, ar.cap - at, st))
            return s;
    }
    k_rows_list<<<(unsigned)blocks, kRlThreads, 0, st>>>(offsets, V, ceil_div(E, unit), unit, *list);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

// ---- passes over the edges

// Orders one wave's LDS accesses (lanes read what other lanes of it wrote).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Edges of group g.
__device__ __forceinline__ int32_t group_size(int64_t E, int64_t g) {
    const int64_t left = E - g * kGroupEdges;
    return left < kGroupEdges ? (int32_t)left : kGroupEdges;
}

// Sources of group g's edges, edge j * 64 + lane in u[j] (edges past E read the
// group's first), and the segment of the edge before the group.
__device__ __forceinline__ void load_group(const int32_t *__restrict__ src, int64_t E, int64_t g, int32_t (&u)[kSteps],
                                           int32_t &before) {
    const int64_t base = g * kGroupEdges;
    const int lane = __lane_id();
    const int32_t n = group_size(E, g);
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
        const int32_t e = j * kWave + lane;
        u[j] = src[base + (e < n ? e : 0)];
    }
    before = src[base > 0 ? base - 1 : 0];
}

// marks[i] = 1 + the row that starts at the group's edge i, 0 where none does.
__device__ __forceinline__ void mark_rows(const RowList &list, int64_t g, int32_t *marks) {
    const int lane = __lane_id();
    const int64_t base = g * kGroupEdges;
    const int32_t i0 = list.first[g], i1 = list.first[g + 1];
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < kSteps; ++j) marks[j * kWave + lane] = 0;
    wave_lds_order();
    for (int32_t ib = i0; ib <= i1; ib += kWave) {  // uniform; at most 17 rounds
        const int32_t i = ib + lane < i1 ? ib + lane : i1;
        const int64_t a = (int64_t)list.start[i] - base;
        if (ib + lane <= i1 && a >= 0 && a < kGroupEdges) marks[a] = list.row[i] + 1;
    }
    wave_lds_order();
}

// Segment per lane of one step and whether the edge starts a run: a row starts
// there, or the edge before it lies in another segment. last: segment of the
// edge before the step.
__device__ __forceinline__ bool run_begins(int32_t mark, int32_t s, int32_t &last) {
    const int32_t prev = dpp_i<kDppWaveShr1, 0xf>(last, s);
    last = __builtin_amdgcn_readlane(s, 63);
    return mark != 0 || s != prev;
}

// Edges and runs per segment of a chunk, one LDS atomic per run and step:
// edges << 16 | runs (a chunk has at most 32,768 of either).
__global__ __launch_bounds__(kSegThreads) void k_seg_count(const int32_t *__restrict__ src,
                                                           RowList list, int64_t E, FastDiv div, int32_t k,
                                                           int32_t chunks, int32_t chunk_groups,
                                                           int32_t *__restrict__ edge_counts,
                                                           int32_t *__restrict__ run_counts) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int32_t *marks = reinterpret_cast<int32_t *>(smem) + (threadIdx.x >> 6) * kGroupEdges;
    uint32_t *hist = reinterpret_cast<uint32_t *>(smem) + kTileEdges;
    for (int32_t s = threadIdx.x; s < k; s += kSegThreads) hist[s] = 0u;
    __syncthreads();
    const int32_t c = xcd_remap(blockIdx.x, chunks);
    const int64_t groups = (E + kGroupEdges - 1) / kGroupEdges;
    const int lane = __lane_id();
    for (int32_t i = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); i < chunk_groups; i += kSegWaves) {
        const int64_t g = (int64_t)c * chunk_groups + i;
        if (g >= groups) break;
        int32_t u[kSteps], before;
        load_group(src, E, g, u, before);
        mark_rows(list, g, marks);
        int32_t last = quotient(div, before);
        const int32_t n = group_size(E, g);
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            const bool valid = j * kWave + lane < n;
            const int32_t s = quotient(div, u[j]);
            const bool start = run_begins(marks[j * kWave + lane], s, last) && valid;
            const uint64_t m = ballot(start) | 1ull, act = ballot(valid);
            if (valid && (start || lane == 0)) {  // length up to the next start or the step's end
                const uint64_t next = lane == 63 ? 0ull : m & (~0ull << (lane + 1));
                const int end = next ? (int)__builtin_ctzll(next) : (int)__builtin_popcountll(act);
                atomicAdd(&hist[s], ((uint32_t)(end - lane) << 16) | (start ? 1u : 0u));
            }
        }
    }
    __syncthreads();
    for (int32_t s = threadIdx.x; s < k; s += kSegThreads) {
        edge_counts[(int64_t)s * chunks + c] = (int32_t)(hist[s] >> 16);
        run_counts[(int64_t)s * chunks + c] = (int32_t)(hist[s] & 0xffffu);
    }
}

// The query's totals: edges per segment (LDS histogram when it fits) and runs.
__global__ __launch_bounds__(kSegThreads) void k_count_runs(const int32_t *__restrict__ src,
                                                            RowList list, int64_t E, FastDiv div, int32_t k,
                                                            int use_lds, int32_t *__restrict__ seg_edges,
                                                            unsigned long long *__restrict__ runs) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = __lane_id();
    int32_t *marks = reinterpret_cast<int32_t *>(smem) + w * kGroupEdges;
    int32_t *hist = reinterpret_cast<int32_t *>(smem) + kTileEdges;
    __shared__ unsigned long long wave_runs[kSegWaves];
    if (use_lds)
        for (int32_t s = threadIdx.x; s < k; s += kSegThreads) hist[s] = 0;
    __syncthreads();
    const int64_t groups = (E + kGroupEdges - 1) / kGroupEdges;
    unsigned long long nr = 0;
    for (int64_t g = (int64_t)blockIdx.x * kSegWaves + w; g < groups; g += (int64_t)gridDim.x * kSegWaves) {
        int32_t u[kSteps], before;
        load_group(src, E, g, u, before);
        mark_rows(list, g, marks);
        int32_t last = quotient(div, before);
        const int32_t n = group_size(E, g);
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            const bool valid = j * kWave + lane < n;
            const int32_t s = quotient(div, u[j]);
            const bool start = run_begins(marks[j * kWave + lane], s, last) && valid;
            const uint64_t ms = ballot(start), m = ms | 1ull, act = ballot(valid);
            nr += (unsigned long long)__builtin_popcountll(ms);
            if (valid && (start || lane == 0)) {
                const uint64_t next = lane == 63 ? 0ull : m & (~0ull << (lane + 1));
                const int end = next ? (int)__builtin_ctzll(next) : (int)__builtin_popcountll(act);
                atomicAdd(use_lds ? &hist[s] : &seg_edges[s], end - lane);
            }
        }
    }
    if (lane == 0) wave_runs[w] = nr;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int x = 1; x < kSegWaves; ++x) nr += wave_runs[x];
        if (nr) atomicAdd(runs, nr);
    }
    if (use_lds) {
        for (int32_t s = threadIdx.x; s < k; s += kSegThreads)
            if (hist[s]) atomicAdd(&seg_edges[s], hist[s]);
    }
}

// As many workgroups as the chip holds at once: each adds its histogram and its runs
// to the totals at its end, and these atomics go through memory one after the other on
// each address, about 13 ns apiece. 2,048 workgroups that added their runs wave by wave
// took 290 us for a query of 16 M edges, where the sorted form's count pass had taken
// 150; now 115 (195 M edges: 416, 720, 335; 16 M edges in 15,888 segments: 343, 195,
// 148).
cagra_status launch_count_runs(const cagra_graph *g, int32_t N, int32_t k, const RowList &rows, int32_t *seg_edges,
                               unsigned long long *runs, hipStream_t st) {
    if (cagra_status a_ = ensure_dynamic_lds((const void *)k_count_runs)) return a_;
    const int use_lds = k <= 16384 ? 1 : 0;
    int64_t grid = ceil_div(ceil_div(g->E, kGroupEdges), kSegWaves);
    const size_t lds = kTileEdges * sizeof(int32_t) + (use_lds ? (size_t)k * sizeof(int32_t) : 0);
    const int64_t per_cu = CAGRA_LDS_BYTES / lds, resident = kChipCus * (per_cu < 4 ? per_cu : 4);
    if (grid > resident) grid = resident;
    k_count_runs<<<(unsigned)grid, kSegThreads, lds, st>>>(g->in_sources, rows, g->E, fast_div(N), k, use_lds,
                                                           seg_edges, runs);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

// Segment and edge word of an edge held in registers; 16-bit words share one.
template <typename W>
struct EdgeTag;
template <>
struct EdgeTag<uint16_t> {
    uint32_t x;
    __device__ __forceinline__ void set(bool ok, int32_t s, uint32_t local, bool start) {
        x = ok ? ((uint32_t)s << 16) | local | (start ? EdgeWord<uint16_t>::kFlag : 0u) : ~0u;
    }
    __device__ __forceinline__ bool valid() const { return x != ~0u; }  // segments are below 2^16 - 1
    __device__ __forceinline__ int32_t segment() const { return (int32_t)(x >> 16); }
    __device__ __forceinline__ uint32_t word() const { return x & 0xffffu; }
};
template <>
struct EdgeTag<uint32_t> {
    uint32_t x;
    int32_t s;
    __device__ __forceinline__ void set(bool ok, int32_t sg, uint32_t local, bool start) {
        x = local | (start ? EdgeWord<uint32_t>::kFlag : 0u);
        s = ok ? sg : -1;
    }
    __device__ __forceinline__ bool valid() const { return s >= 0; }
    __device__ __forceinline__ int32_t segment() const { return s; }
    __device__ __forceinline__ uint32_t word() const { return x; }
};

// LDS of the scatter: the ranking's marks and per-wave counts, then (over them)
// a tile's edge words or its runs by output position; and the positions of each
// segment's part.
static size_t scatter_lds(int32_t k) {
    const size_t rank = kTileEdges * 4 + (size_t)kSegWaves * k * 4;
    const size_t stage = kTileEdges * 8;
    return (rank > stage ? rank : stage) + (size_t)k * 8;
}

template <typename W, int KBITS>
__global__ __launch_bounds__(kSegThreads, 4) void k_seg_scatter(
    const int32_t *__restrict__ src, RowList list, int64_t E, FastDiv div, int32_t N, int32_t k, int32_t chunks, int32_t chunk_tiles,
    const int32_t *__restrict__ edge_base, const int32_t *__restrict__ run_base, FastDiv bdiv, int32_t B,
    W *__restrict__ edge_src, int32_t *__restrict__ row_ptr, int32_t *__restrict__ row_dst,
    uint16_t *__restrict__ row_dst_lo) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ uint32_t wsum[kSegWaves];
    const int tid = threadIdx.x, lane = __lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // per-segment positions: output index of a tile's edge (run) = edge_at[s] + local position
    int32_t *edge_at = reinterpret_cast<int32_t *>(smem), *run_at = edge_at + k;
    unsigned char *area = smem + (size_t)k * 8;
    int32_t *marks = reinterpret_cast<int32_t *>(area) + w * kGroupEdges;
    uint32_t *counts = reinterpret_cast<uint32_t *>(area + kTileEdges * 4);  // [wave][segment], edges << 16 | runs
    uint32_t *mine = counts + w * k;
    W *st_word = reinterpret_cast<W *>(area);                                         // edges: word, segment
    uint16_t *st_seg = reinterpret_cast<uint16_t *>(area + kTileEdges * 4);
    int32_t *st_dst = reinterpret_cast<int32_t *>(area);                              // runs: destination, segment,
    uint16_t *st_pos = reinterpret_cast<uint16_t *>(area + kTileEdges * 6);           // position of the first edge
    const int32_t c = xcd_remap(blockIdx.x, chunks);
    const int64_t groups = (E + kGroupEdges - 1) / kGroupEdges;
    // a thread owns per consecutive segments
    const int32_t per = (k + kSegThreads - 1) / kSegThreads;
    constexpr int kMaxPer = kDirectMaxSegments / kSegThreads;
    int32_t next_edge[kMaxPer], next_run[kMaxPer];
#pragma unroll
    for (int i = 0; i < kMaxPer; ++i) {
        const int32_t s = tid * per + i;
        const bool own = i < per && s < k;
        next_edge[i] = own ? edge_base[(int64_t)s * chunks + c] : 0;
        next_run[i] = own ? run_base[(int64_t)s * chunks + c] : 0;
    }
    for (int32_t t = 0; t < chunk_tiles; ++t) {
        const int64_t tile = ((int64_t)c * chunk_tiles + t) * kTileEdges;
        if (tile >= E) break;  // uniform over the workgroup
        const int32_t cnt = (int32_t)(E - tile < kTileEdges ? E - tile : kTileEdges);
        const int64_t g = tile / kGroupEdges + w;
        int32_t dst[kSteps];    // the edge's row
        uint32_t rank[kSteps];  // edges << 16 | runs before it in its segment (wave, then tile)
        EdgeTag<W> tag[kSteps]; // segment and edge word, row-start flag included
        for (int32_t s = lane; s < k; s += kWave) mine[s] = 0u;
        const int32_t n = g < groups ? group_size(E, g) : 0;
        if (n > 0) {  // uniform over the wave
            int32_t before;
            int32_t u[kSteps];
            load_group(src, E, g, u, before);
            int32_t row1 = list.row[list.first[g]] + 1;  // 1 + the row of the edge before the step's first mark
            mark_rows(list, g, marks);
            int32_t last = quotient(div, before);
            // kPart steps at a time: the first lane of each segment in a step
            // adds the step's edges and runs of that segment to the wave's count
            // and gets what came before. The LDS carries out one wave's accesses
            // in program order, so these adds need no wait between the steps;
            // their results are handed to the segment's other lanes afterwards.
            constexpr int kPart = 8;
#pragma unroll
            for (int j0 = 0; j0 < kSteps; j0 += kPart) {
                uint32_t had[kPart];
                int first[kPart];
#pragma unroll
                for (int i = 0; i < kPart; ++i) {
                    const int j = j0 + i;
                    const bool valid = j * kWave + lane < n;
                    const int32_t s = quotient(div, u[j]);
                    const int32_t mk = marks[j * kWave + lane];
                    const bool start = run_begins(mk, s, last) && valid;
                    // marks ascend, so the last one at or before a lane is the largest
                    row1 = max(wave_incl_max(mk), row1);
                    dst[j] = row1 - 1;
                    row1 = __builtin_amdgcn_readlane(row1, 63);
                    tag[j].set(valid, s, (uint32_t)(u[j] - s * N), start);
                    // lanes of the step in the same segment, one compare per bit of the id
                    const uint64_t act = ballot(valid), ms = ballot(start);
                    uint32_t plo = (uint32_t)act, phi = (uint32_t)(act >> 32);
#pragma unroll
                    for (int b = 0; b < KBITS; ++b) {
                        const int32_t bit = (int32_t)((uint32_t)s << (31 - b)) >> 31;  // 0 or -1
                        const uint64_t set = ballot(bit < 0);
                        plo &= ~((uint32_t)set ^ (uint32_t)bit);
                        phi &= ~((uint32_t)(set >> 32) ^ (uint32_t)bit);
                    }
                    const uint64_t peers = (uint64_t)phi << 32 | plo, below = peers & lanemask_lt();
                    rank[j] = ((uint32_t)__popcll(below) << 16) | (uint32_t)__popcll(below & ms);
                    first[i] = peers ? (int)__builtin_ctzll(peers) : 0;
                    had[i] = 0u;
                    if (valid && below == 0ull)
                        had[i] = atomicAdd(&mine[s], ((uint32_t)__popcll(peers) << 16) | (uint32_t)__popcll(peers & ms));
                }
#pragma unroll
                for (int i = 0; i < kPart; ++i)
                    rank[j0 + i] += (uint32_t)__builtin_amdgcn_ds_bpermute(first[i] << 2, (int32_t)had[i]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < kSteps; ++j) tag[j].set(false, 0, 0u, false);
        }
        __syncthreads();
        // exclusive scan of the tile's counts over the segments (a tile holds at
        // most 8,192 edges and runs, so the halves do not carry), then the start
        // of every wave's part of a segment
        uint32_t tot[kMaxPer], sum = 0;
#pragma unroll
        for (int i = 0; i < kMaxPer; ++i) {
            const int32_t s = tid * per + i;
            tot[i] = 0;
            if (i < per && s < k)
                for (int x = 0; x < kSegWaves; ++x) tot[i] += counts[x * k + s];
            sum += tot[i];
        }
        uint32_t incl = sum;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        uint32_t at = incl - sum, all = 0;
        for (int x = 0; x < kSegWaves; ++x) {
            if (x < w) at += wsum[x];
            all += wsum[x];
        }
#pragma unroll
        for (int i = 0; i < kMaxPer; ++i) {
            const int32_t s = tid * per + i;
            if (i < per && s < k) {
                edge_at[s] = next_edge[i] - (int32_t)(at >> 16);
                run_at[s] = next_run[i] - (int32_t)(at & 0xffffu);
                next_edge[i] += (int32_t)(tot[i] >> 16);
                next_run[i] += (int32_t)(tot[i] & 0xffffu);
                for (int x = 0; x < kSegWaves; ++x) {
                    const uint32_t y = counts[x * k + s];
                    counts[x * k + s] = at;
                    at += y;
                }
            }
        }
        const int32_t nruns = (int32_t)(all & 0xffffu);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSteps; ++j)
            if (tag[j].valid()) rank[j] += mine[tag[j].segment()];
        __syncthreads();  // the counts are read; the staged edges take their place
#pragma unroll
        for (int j = 0; j < kSteps; ++j)
            if (tag[j].valid()) {
                st_word[rank[j] >> 16] = (W)tag[j].word();
                st_seg[rank[j] >> 16] = (uint16_t)tag[j].segment();
            }
        __syncthreads();
#pragma unroll 4
        for (int32_t p = tid; p < cnt; p += kSegThreads) edge_src[(int64_t)edge_at[st_seg[p]] + p] = st_word[p];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSteps; ++j)
            if (tag[j].valid() && (tag[j].word() & EdgeWord<W>::kFlag)) {
                const uint32_t p = rank[j] & 0xffffu;
                st_dst[p] = dst[j];
                st_seg[p] = (uint16_t)tag[j].segment();
                st_pos[p] = (uint16_t)(rank[j] >> 16);
            }
        __syncthreads();
#pragma unroll 4
        for (int32_t p = tid; p < nruns; p += kSegThreads) {
            const int32_t s = st_seg[p], d = st_dst[p];
            const int64_t r = (int64_t)run_at[s] + p;
            row_ptr[r] = edge_at[s] + (int32_t)st_pos[p];
            row_dst[r] = d;
            row_dst_lo[r] = (uint16_t)(d - quotient(bdiv, d) * B);
        }
        __syncthreads();  // the next tile reuses the area and the positions
    }
}

__global__ void k_seg_begin(const int32_t *__restrict__ run_base, int32_t k, int32_t chunks, int32_t E, int32_t Q,
                            int32_t *__restrict__ seg_row_begin, int32_t *__restrict__ row_ptr) {
    const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < k) seg_row_begin[s] = run_base[(int64_t)s * chunks];
    if (s == k) {
        seg_row_begin[k] = Q;
        row_ptr[Q] = E;
    }
}

// Tiles per chunk: more of them shrink the count matrices, fewer fill the chip
// with a small graph.
static int32_t chunk_tiles_for(int64_t E) {
    const int64_t t = ceil_div(E, kTileEdges) / kChunksWanted;
    return (int32_t)(t < 1 ? 1 : (t > kMaxChunkTiles ? kMaxChunkTiles : t));
}

size_t direct_ws_bytes(int32_t V, int64_t E, int32_t k) {
    const int64_t chunks = ceil_div(E, (int64_t)chunk_tiles_for(E) * kTileEdges);
    ArenaSize a;
    a.take<char>((int64_t)row_list_ws_bytes(V, E, kGroupEdges));
    a.take<int32_t>(chunks * k);
    a.take<int32_t>(chunks * k);
    return a.used + scan_add_ws_bytes(chunks * k) + 512;
}

template <typename W, int KBITS>
static cagra_status launch_scatter_b(const cagra_graph *g, const cagra_segments *seg, const RowList &rows,
                                     int32_t chunks, int32_t chunk_tiles, const int32_t *edge_base,
                                     const int32_t *run_base, hipStream_t st) {
    if (cagra_status a_ = ensure_dynamic_lds((const void *)k_seg_scatter<W, KBITS>)) return a_;
    k_seg_scatter<W, KBITS><<<(unsigned)chunks, kSegThreads, scatter_lds(seg->k), st>>>(
        g->in_sources, rows, g->E, fast_div(seg->N), seg->N, seg->k, chunks, chunk_tiles, edge_base,
        run_base, fast_div(seg->B), seg->B, static_cast<W *>(seg->edge_src), seg->row_ptr, seg->row_dst,
        seg->row_dst_lo);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

// The segment ids' bits are compared one ballot each, unrolled; the width is
// rounded up to one of a few.
template <typename W>
static cagra_status launch_scatter(const cagra_graph *g, const cagra_segments *seg, const RowList &rows,
                                   int32_t chunks, int32_t chunk_tiles, const int32_t *edge_base,
                                   const int32_t *run_base, hipStream_t st) {
    static_assert(kDirectMaxSegments <= 1 << 11, "widest segment id");
    const int32_t k = seg->k;
    auto f = k <= 1 << 4 ? launch_scatter_b<W, 4> : k <= 1 << 7 ? launch_scatter_b<W, 7>
             : k <= 1 << 9 ? launch_scatter_b<W, 9> : k <= 1 << 10 ? launch_scatter_b<W, 10> : launch_scatter_b<W, 11>;
    return f(g, seg, rows, chunks, chunk_tiles, edge_base, run_base, st);
}

cagra_status build_direct(const cagra_graph *g, const cagra_segments *seg, void *ws, size_t ws_bytes,
                          hipStream_t st) {
    const int64_t E = g->E;
    const int32_t k = seg->k, tiles = chunk_tiles_for(E);
    const int64_t chunks = ceil_div(E, (int64_t)tiles * kTileEdges), n = chunks * k;
    if (n > INT32_MAX) return fail(CAGRA_E_OVERFLOW, "segment count matrix too large");
    Arena ar{(char *)ws, ws_bytes, 0};
    RowList rows;
    cagra_status s;
    if ((s = build_row_list(g->in_offsets, g->V, E, kGroupEdges, ar, &rows, st)) != CAGRA_OK) return s;
    int32_t *ce = ar.take<int32_t>(n), *cr = ar.take<int32_t>(n);
    if (!ce || !cr) return fail(CAGRA_E_BUFFER, "build workspace too small (segment counts)");
    char *tmp = ar.base + align_up(ar.used, 256);
    const size_t tmp_bytes = ws_bytes - align_up(ar.used, 256);
    if (cagra_status a_ = ensure_dynamic_lds((const void *)k_seg_count)) return a_;
    k_seg_count<<<(unsigned)chunks, kSegThreads, kTileEdges * 4 + (size_t)k * 4, st>>>(
        g->in_sources, rows, E, fast_div(seg->N), k, (int32_t)chunks, tiles * kSegWaves, ce, cr);
    CAGRA_LAUNCH_CHECK();
    if ((s = scan_add_exclusive(ce, ce, n, tmp, tmp_bytes, st)) != CAGRA_OK) return s;
    if ((s = scan_add_exclusive(cr, cr, n, tmp, tmp_bytes, st)) != CAGRA_OK) return s;
    s = edge16(seg->N) ? launch_scatter<uint16_t>(g, seg, rows, (int32_t)chunks, tiles, ce, cr, st)
                       : launch_scatter<uint32_t>(g, seg, rows, (int32_t)chunks, tiles, ce, cr, st);
    if (s != CAGRA_OK) return s;
    k_seg_begin<<<(unsigned)ceil_div((int64_t)k + 1, 256), 256, 0, st>>>(cr, k, (int32_t)chunks, (int32_t)E,
                                                                        (int32_t)seg->Q, seg->seg_row_begin,
                                                                        seg->row_ptr);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

}  // namespace cagra
