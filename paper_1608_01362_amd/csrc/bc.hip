// Betweenness centrality from sampled starts (Brandes) as level-synchronous
// segmented pulls: EdgeMap with an active frontier (Section 4). A forward level
// gathers sigma over in-edges from the vertices at depth d; a backward level
// gathers (1 + delta) / sigma over the reverse graph from the vertices at depth
// d + 1. The frontier enters as a bitmask of active segments: tiles and merge
// ranges of segments without a frontier vertex are skipped, so the sparse
// levels at both ends of a BFS cost little.
#include "common.h"

namespace cagra {

cagra_status launch_gather_active(const cagra_segments *seg, int32_t op, int32_t value_type, const void *values,
                                  void *partial, const uint32_t *seg_active, hipStream_t st);
cagra_status launch_merge_active(const cagra_segments *seg, int32_t op, const void *partial, void *out,
                                 const uint32_t *seg_active, hipStream_t st);

constexpr int kBcThreads = 256;       // the start and the backward update
constexpr int kBcSpanThreads = 1024;  // the kernels over spans

__global__ void k_bc_start(int32_t V, int32_t source, int32_t *__restrict__ depth, float *__restrict__ sigma,
                           float *__restrict__ delta) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V) return;
    depth[v] = v == source ? 0 : -1;
    sigma[v] = v == source ? 1.0f : 0.0f;
    delta[v] = 0.0f;
}

__global__ void k_zero_words(uint32_t *__restrict__ w, int32_t n) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) w[i] = 0u;
}

// The vertex kernels give each workgroup a contiguous span of vertices. The
// segments of its frontier vertices are first marked in an LDS bitmask that
// covers only the span's segments, then OR-ed into the global mask, one atomic
// per non-zero word; the new-frontier count is reduced in the workgroup and
// added once. (One global atomic per wave on a handful of words serialises:
// half a million of them took 1.5-1.9 ms per level at scale 25.)
// The span shrinks with the graph so that about kBcWorkgroups workgroups cover
// it: with 16,384 vertices each, 2 M vertices gave 128 workgroups, half the
// chip's CUs. More and smaller ones lose again: their atomics on the one count
// and the few words go through memory one after the other, about 13 ns each
// (2,048 workgroups of 1,024 vertices: 28-31 us where the frontier is dense,
// 13-18 us now; a word that has the bits already is left alone).
constexpr int kBcMaxSpan = 16384;                 // vertices per workgroup
constexpr int kBcMinSpan = 4096;
constexpr int kBcWorkgroups = 512;
constexpr int kBcMaskWords = kBcMaxSpan / 32 + 2; // segments of a span, in 32-bit words, for N >= 1

// A thread takes kBcBatch vertices of the span per round and loads all they may
// need before it looks at any (also sigma and delta of vertices outside the
// frontier, which are bytes, not round trips). The last round of a span may be a
// part of one (2.5 M vertices: spans of 5,120).
constexpr int kBcBatch = 4;
static_assert(kBcMinSpan % (kBcBatch * kBcSpanThreads) == 0, "the shortest span is whole rounds");

struct SpanMask {
    int32_t v0, v1;     // the workgroup's vertices [v0, v1)
    int32_t w_lo, w_hi; // global mask words covering their segments
    int32_t seg;        // their segment, or -1 if the span covers several
};

__device__ __forceinline__ SpanMask span_begin(int32_t V, int32_t N, int32_t span, uint32_t *lmask) {
    SpanMask m;
    m.v0 = (int32_t)blockIdx.x * span;
    m.v1 = V - m.v0 < span ? V : m.v0 + span;
    const int32_t s0 = m.v0 / N, s1 = (m.v1 - 1) / N;
    m.w_lo = s0 >> 5;
    m.w_hi = s1 >> 5;
    m.seg = s0 == s1 ? s0 : -1;
    for (int i = threadIdx.x; i <= m.w_hi - m.w_lo; i += kBcSpanThreads) lmask[i] = 0u;
    __syncthreads();
    return m;
}

// Marks the segments of the wave's active vertices (active[u]: vertex v + u *
// kBcSpanThreads) in the span's LDS mask: one LDS atomic per wave where they share one.
__device__ __forceinline__ void mark_segments(const SpanMask &m, uint32_t *lmask, uint32_t v, int32_t N,
                                              const bool (&active)[kBcBatch]) {
    if (m.seg >= 0) {  // uniform
        bool any = false;
#pragma unroll
        for (int u = 0; u < kBcBatch; ++u) any |= active[u];
        if (__builtin_amdgcn_ballot_w64(any) && __lane_id() == 0)
            atomicOr(&lmask[(m.seg >> 5) - m.w_lo], 1u << (m.seg & 31));
        return;
    }
#pragma unroll
    for (int u = 0; u < kBcBatch; ++u) {
        const uint64_t any = __builtin_amdgcn_ballot_w64(active[u]);
        if (!any) continue;
        const int32_t s = active[u] ? (int32_t)((v + u * kBcSpanThreads) / (uint32_t)N) : 0;
        const int first = (int)__builtin_ctzll(any);
        const int32_t s0 = __builtin_amdgcn_readlane(s, first);
        if (__builtin_amdgcn_ballot_w64(active[u] && s != s0) == 0) {
            if (__lane_id() == first) atomicOr(&lmask[(s0 >> 5) - m.w_lo], 1u << (s0 & 31));
        } else if (active[u]) {
            atomicOr(&lmask[(s >> 5) - m.w_lo], 1u << (s & 31));
        }
    }
}

__device__ __forceinline__ void span_flush(const SpanMask &m, const uint32_t *lmask, uint32_t *mask) {
    __syncthreads();
    for (int i = threadIdx.x; i <= m.w_hi - m.w_lo; i += kBcSpanThreads) {
        const uint32_t bits = lmask[i];
        // bits are only ever added: an old value read here costs an atomic, no more
        if (bits && (mask[m.w_lo + i] & bits) != bits) atomicOr(&mask[m.w_lo + i], bits);
    }
}

// x[u] = a[v + u * kBcSpanThreads], clamped to the span. (Unsigned: the last span may
// end at the largest int32.)
template <typename T>
__device__ __forceinline__ void load_batch(T (&x)[kBcBatch], const T *a, uint32_t v, uint32_t v1) {
#pragma unroll
    for (int u = 0; u < kBcBatch; ++u) x[u] = a[min(v + u * kBcSpanThreads, v1 - 1u)];
}

// vals[u] = sigma[u] for the frontier (depth d), else 0; frontier segments marked.
__global__ __launch_bounds__(kBcSpanThreads) void k_bc_fwd_values(int32_t V, int32_t N, int32_t span, int32_t d,
                                                              const int32_t *__restrict__ depth,
                                                              const float *__restrict__ sigma,
                                                              float *__restrict__ vals, uint32_t *__restrict__ mask,
                                                              int32_t *__restrict__ count) {
    __shared__ uint32_t lmask[kBcMaskWords];
    const SpanMask m = span_begin(V, N, span, lmask);
    if (blockIdx.x == 0 && threadIdx.x == 0) *count = 0;  // next frontier size, counted by k_bc_fwd_update
    for (int32_t r = 0; r < m.v1 - m.v0; r += kBcBatch * kBcSpanThreads) {
        const uint32_t v = (uint32_t)m.v0 + r + threadIdx.x;
        int32_t dep[kBcBatch];
        float sg[kBcBatch];
        bool in[kBcBatch];
        load_batch(dep, depth, v, m.v1);
        load_batch(sg, sigma, v, m.v1);
#pragma unroll
        for (int u = 0; u < kBcBatch; ++u) {
            const bool own = v + u * kBcSpanThreads < (uint32_t)m.v1;
            in[u] = own && dep[u] == d;
            if (own) vals[v + u * kBcSpanThreads] = in[u] ? sg[u] : 0.0f;
        }
        mark_segments(m, lmask, v, N, in);
    }
    span_flush(m, lmask, mask);
}

// Unvisited vertices reached at this level: depth d + 1, sigma = the sum.
__global__ __launch_bounds__(kBcSpanThreads) void k_bc_fwd_update(int32_t V, int32_t span, int32_t d, const float *__restrict__ sums,
                                                              int32_t *__restrict__ depth,
                                                              float *__restrict__ sigma,
                                                              int32_t *__restrict__ count) {
    __shared__ int32_t red[kBcSpanThreads / kWave];
    const int32_t v0 = (int32_t)blockIdx.x * span;
    const int32_t v1 = V - v0 < span ? V : v0 + span;
    int32_t reached = 0;
    for (int32_t r = 0; r < v1 - v0; r += kBcBatch * kBcSpanThreads) {
        const uint32_t v = (uint32_t)v0 + r + threadIdx.x;
        int32_t dep[kBcBatch];
        float x[kBcBatch];
        load_batch(dep, depth, v, v1);
        load_batch(x, sums, v, v1);
#pragma unroll
        for (int u = 0; u < kBcBatch; ++u) {
            const uint32_t w = v + u * kBcSpanThreads;
            if (w < (uint32_t)v1 && dep[u] < 0 && x[u] > 0.0f) {
                depth[w] = d + 1;
                sigma[w] = x[u];
                ++reached;
            }
        }
    }
    for (int o = 32; o >= 1; o >>= 1) reached += __shfl_down(reached, o, 64);
    if (__lane_id() == 0) red[threadIdx.x >> 6] = reached;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int i = 0; i < kBcSpanThreads / kWave; ++i) t += red[i];
        if (t) atomicAdd(count, t);
    }
}

// vals[w] = (1 + delta[w]) / sigma[w] for the vertices at depth d + 1, else 0;
// their segments (in the reverse graph's segmentation) marked.
__global__ __launch_bounds__(kBcSpanThreads) void k_bc_bwd_values(int32_t V, int32_t N, int32_t span, int32_t d,
                                                              const int32_t *__restrict__ depth,
                                                              const float *__restrict__ sigma,
                                                              const float *__restrict__ delta,
                                                              float *__restrict__ vals, uint32_t *__restrict__ mask) {
    __shared__ uint32_t lmask[kBcMaskWords];
    const SpanMask m = span_begin(V, N, span, lmask);
    for (int32_t r = 0; r < m.v1 - m.v0; r += kBcBatch * kBcSpanThreads) {
        const uint32_t v = (uint32_t)m.v0 + r + threadIdx.x;
        int32_t dep[kBcBatch];
        float sg[kBcBatch], dl[kBcBatch];
        bool in[kBcBatch];
        load_batch(dep, depth, v, m.v1);
        load_batch(sg, sigma, v, m.v1);
        load_batch(dl, delta, v, m.v1);
#pragma unroll
        for (int u = 0; u < kBcBatch; ++u) {
            const bool own = v + u * kBcSpanThreads < (uint32_t)m.v1;
            in[u] = own && dep[u] == d + 1;
            if (own) vals[v + u * kBcSpanThreads] = in[u] ? (1.0f + dl[u]) / sg[u] : 0.0f;
        }
        mark_segments(m, lmask, v, N, in);
    }
    span_flush(m, lmask, mask);
}

// Vertices at depth d: delta = sigma * sum; the centrality of every vertex
// other than the start accumulates delta.
__global__ __launch_bounds__(kBcThreads) void k_bc_bwd_update(int32_t V, int32_t d, int32_t source,
                                                              const float *__restrict__ sums,
                                                              const int32_t *__restrict__ depth,
                                                              const float *__restrict__ sigma,
                                                              float *__restrict__ delta, float *__restrict__ bc) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V || depth[v] != d) return;
    const float dl = sigma[v] * sums[v];
    delta[v] = dl;
    if (v != source) bc[v] += dl;
}

// Vertices per workgroup: a multiple of its threads.
static int32_t span_for(int32_t V) {
    const int64_t s = ceil_div(ceil_div(V, kBcWorkgroups), kBcSpanThreads) * kBcSpanThreads;
    return (int32_t)(s < kBcMinSpan ? kBcMinSpan : (s > kBcMaxSpan ? kBcMaxSpan : s));
}
static unsigned spans_for(int32_t V) { return (unsigned)ceil_div(V > 0 ? V : 1, span_for(V)); }

static unsigned blocks_for(int64_t n) { return (unsigned)ceil_div(n > 0 ? n : 1, kBcThreads); }

size_t bc_mask_words(const cagra_segments *seg) { return (size_t)ceil_div(seg->k, 32); }

cagra_status launch_bc_start(int32_t V, int32_t source, int32_t *depth, float *sigma, float *delta, hipStream_t st) {
    k_bc_start<<<blocks_for(V), kBcThreads, 0, st>>>(V, source, depth, sigma, delta);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

cagra_status launch_bc_forward(const cagra_segments *seg, int32_t d, int32_t *depth, float *sigma, float *vals,
                               float *partial, float *sums, int32_t *count, uint32_t *mask, hipStream_t st) {
    const int32_t V = seg->V, words = (int32_t)bc_mask_words(seg);
    k_zero_words<<<(unsigned)ceil_div(words, 256), 256, 0, st>>>(mask, words);
    CAGRA_LAUNCH_CHECK();
    k_bc_fwd_values<<<spans_for(V), kBcSpanThreads, 0, st>>>(V, seg->N, span_for(V), d, depth, sigma, vals, mask, count);
    CAGRA_LAUNCH_CHECK();
    cagra_status s;
    if ((s = launch_gather_active(seg, CAGRA_SUM_F32, CAGRA_F32, vals, partial, mask, st)) != CAGRA_OK) return s;
    if ((s = launch_merge_active(seg, CAGRA_SUM_F32, partial, sums, mask, st)) != CAGRA_OK) return s;
    k_bc_fwd_update<<<spans_for(V), kBcSpanThreads, 0, st>>>(V, span_for(V), d, sums, depth, sigma, count);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

cagra_status launch_bc_backward(const cagra_segments *seg_t, int32_t d, int32_t source, const int32_t *depth,
                                const float *sigma, float *delta, float *bc, float *vals, float *partial,
                                float *sums, uint32_t *mask, hipStream_t st) {
    const int32_t V = seg_t->V, words = (int32_t)bc_mask_words(seg_t);
    k_zero_words<<<(unsigned)ceil_div(words, 256), 256, 0, st>>>(mask, words);
    CAGRA_LAUNCH_CHECK();
    k_bc_bwd_values<<<spans_for(V), kBcSpanThreads, 0, st>>>(V, seg_t->N, span_for(V), d, depth, sigma, delta, vals, mask);
    CAGRA_LAUNCH_CHECK();
    cagra_status s;
    if ((s = launch_gather_active(seg_t, CAGRA_SUM_F32, CAGRA_F32, vals, partial, mask, st)) != CAGRA_OK) return s;
    if ((s = launch_merge_active(seg_t, CAGRA_SUM_F32, partial, sums, mask, st)) != CAGRA_OK) return s;
    k_bc_bwd_update<<<blocks_for(V), kBcThreads, 0, st>>>(V, d, source, sums, depth, sigma, delta, bc);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

}  // namespace cagra
