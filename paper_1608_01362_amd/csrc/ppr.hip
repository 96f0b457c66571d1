// Personalized PageRank for many restart vertices at once: the segmented pull
// of Sections 3.2-3.3 applied to a [V x 64] block of vertex values (a segmented
// sparse-times-dense product). Lane j of a wave owns column j, so every gathered
// source row is one 256-byte load and every buffer row one 256-byte store.
//
// With 256 bytes per vertex, a segment that fits LDS would hold only 512
// vertices and q would approach the average degree; the natural segment sizes
// here are L2- or Infinity-Cache-sized (Section 3.4's trade-off with a larger
// vertex record), and the gathers read whole cache lines through that level.
//
// The merge keeps the paper's order exactly: for each block of destinations,
// subgraphs in ascending order, each subgraph's rows spread over the waves
// (distinct destinations), FP32 accumulators in LDS.
#include <math.h>

#include "common.h"
#include "wave.h"

namespace cagra {

constexpr int kCols = CAGRA_PPR_COLS;
constexpr int kPprWaves = CAGRA_TILE_WAVES;
constexpr int kPprThreads = kPprWaves * kWave;
constexpr int kBatch = 16;  // source rows per wave whose loads are in flight together
static_assert(kWave == 4 * kBatch, "four batches per 64 edge words");
constexpr int kMergeBatch = 8;  // merge rows / vertices per wave whose loads are in flight together

// Each wave takes an equal share of the tile's edges; lane j adds column j. Row sums
// are FP64 (at least as exact as FP32 with a compensation term, and a conversion and
// an add per edge instead of seven instructions), a row's place comes from the lane
// that read the edge word as the load's scalar offset, and the row starts of 64 edges
// are one mask: 3 vector instructions per edge (11 before, which kept the vector unit
// busy 86% of the time).
//
// Bound by the source rows: from the caches at 2^18 vertices (16 edges each, tiles of
// 16,384 edges) 208 -> 168 us for an iteration; at 2^21, where 60% of the lines miss L2,
// by memory's rate for scattered lines: 785 -> 750 us for the gather. (Half rows per
// workgroup, each L2 holding twice as many, cut these misses by 18% and took 819 us.)
//
// FAR: segments of 4 GiB and more, whose rows a scalar offset does not reach.
// AHEAD: the next 16 source rows are loaded before the last 16 are added, on one
// workgroup per CU instead of two. STREAM: edge words and buffer rows leave no copy
// in the caches. SPLIT: a tile is the work of `parts` workgroups (a divisor of its
// shares). A part takes the rows that start in its shares, to their ends, so no sum
// crosses workgroups; its own shares' first rows are found by counting row starts.
// The rules for these are at the launch.
template <typename W, bool FAR, bool AHEAD, bool STREAM, bool SPLIT>
__global__ __launch_bounds__(kPprThreads) void k_gather_cols(const W *__restrict__ edge_src,
                                                             const int32_t *__restrict__ tile_edge,
                                                             const int32_t *__restrict__ tile_seg,
                                                             const int32_t *__restrict__ span_row,
                                                             const float *__restrict__ values, int32_t N,
                                                             uint32_t seg_bytes, int32_t ntiles,
                                                             const int32_t *__restrict__ row_ptr, int32_t parts,
                                                             float *__restrict__ partial) {
    __shared__ float fix_head[kPprWaves][kCols];
    __shared__ float fix_last[kPprWaves][kCols];
    __shared__ int32_t fix_row[kPprWaves];
    __shared__ int32_t fix_has[kPprWaves];

    const int tp = xcd_remap(blockIdx.x, SPLIT ? ntiles * parts : ntiles), t = SPLIT ? tp / parts : tp;
    int64_t e0 = tile_edge[t], e1 = tile_edge[t + 1];
    int32_t first = 0;  // SPLIT: first row of the part
    if constexpr (SPLIT) {
        const int part = tp - t * parts;
        const int32_t *span = span_row + (int64_t)t * kPprWaves + part * (kPprWaves / parts);
        first = span[0];
        const int64_t end = part == parts - 1 ? e1 : row_ptr[span[kPprWaves / parts]];
        if (part > 0) e0 = row_ptr[first];
        if (end < e1) e1 = end;
    }
    if (e0 >= e1) return;
    const int64_t vbase = (int64_t)tile_seg[t] * N;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t sl = (e1 - e0 + kPprWaves - 1) / kPprWaves;
    int64_t w0 = e0 + w * sl;
    if (w0 > e1) w0 = e1;
    int64_t w1 = w0 + sl;
    if (w1 > e1) w1 = e1;
    int32_t row;  // row open at the share's start
    if constexpr (SPLIT) {
        int32_t n = 0;
        for (int64_t e = w0; e < w1; e += kWave) {
            const uint32_t word = e + lane < w1 ? (uint32_t)edge_src[e + lane] : 0u;
            n += (int32_t)__popcll(__builtin_amdgcn_ballot_w64((word & EdgeWord<W>::kFlag) != 0));
        }
        if (lane == 0) fix_row[w] = n;
        __syncthreads();
        row = first - 1;
        for (int i = 0; i < w; ++i) row += fix_row[i];
        row = __builtin_amdgcn_readfirstlane(row);
        __syncthreads();  // fix_row is written again at the end
    } else {
        row = span_row[(int64_t)t * kPprWaves + w] - 1;
    }
    int32_t seen = 0;
    double acc = 0.0;
    float head = 0.0f;
    const float *vals = values + vbase * kCols;
    const __amdgpu_buffer_rsrc_t rows =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(vals), 0, (int)seg_bytes, kBufFlags);

    auto load_word = [&](int64_t e) {
        return e >= w1 ? 0u : (uint32_t)(STREAM ? __builtin_nontemporal_load(edge_src + e) : edge_src[e]);
    };
    // a row's index (FAR) or byte offset in the segment
    auto place = [](uint32_t word) {
        return FAR ? word & EdgeWord<W>::kIndex : (word & EdgeWord<W>::kIndex) * (kCols * 4u);
    };
    // the rows of edges jb .. jb + kBatch - 1 of the 64 (the segment's first for those past the share)
    auto load = [&](float (&x)[kBatch], uint32_t at, int jb) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int32_t)at, jb + u);
            if constexpr (FAR) x[u] = vals[(int64_t)o * kCols + lane];
            else x[u] = __int_as_float((int32_t)__builtin_amdgcn_raw_buffer_load_b32(rows, lane * 4, o, 0));
        }
    };
    auto add = [&](float (&x)[kBatch], uint64_t starts, int jb, int n) {
        if (n - jb < kBatch) {  // the share ends here: the edges after it add nothing
#pragma unroll
            for (int u = 0; u < kBatch; ++u) x[u] = jb + u < n ? x[u] : 0.0f;
        }
        const uint32_t m = (uint32_t)(starts >> jb);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (m >> u & 1u) {  // a row starts: the open row is complete
                float *const to = partial + (int64_t)row * kCols + lane;
                if (!seen) head = (float)acc;
                else if constexpr (STREAM) __builtin_nontemporal_store((float)acc, to);
                else *to = (float)acc;
                seen = 1;
                ++row;
                acc = 0.0;
            }
            acc += (double)x[u];
        }
    };

    if constexpr (AHEAD) {
        if (w0 < w1) {
            float xa[kBatch], xb[kBatch];
            uint32_t word = load_word(w0 + lane), next = load_word(w0 + kWave + lane), at = place(word);
            load(xa, at, 0);
            for (int64_t b0 = w0; b0 < w1; b0 += kWave) {
                const uint64_t starts = __builtin_amdgcn_ballot_w64((word & EdgeWord<W>::kFlag) != 0);
                const int n = (int)(w1 - b0 < kWave ? w1 - b0 : kWave);
                word = next;
                next = load_word(b0 + 2 * kWave + lane);
                // the barriers keep each batch's loads before the sums of the one before it
                load(xb, at, kBatch);
                __builtin_amdgcn_sched_barrier(0);
                add(xa, starts, 0, n);
                load(xa, at, 2 * kBatch);
                __builtin_amdgcn_sched_barrier(0);
                add(xb, starts, kBatch, n);
                load(xb, at, 3 * kBatch);
                __builtin_amdgcn_sched_barrier(0);
                add(xa, starts, 2 * kBatch, n);
                at = place(word);
                load(xa, at, 0);
                __builtin_amdgcn_sched_barrier(0);
                add(xb, starts, 3 * kBatch, n);
            }
        }
    } else {
        for (int64_t b0 = w0; b0 < w1; b0 += kWave) {
            const uint32_t word = load_word(b0 + lane), at = place(word);
            const uint64_t starts = __builtin_amdgcn_ballot_w64((word & EdgeWord<W>::kFlag) != 0);
            const int n = (int)(w1 - b0 < kWave ? w1 - b0 : kWave);
            for (int jb = 0; jb < n; jb += kBatch) {
                float x[kBatch];
                load(x, at, jb);
                add(x, starts, jb, n);
            }
        }
    }
    fix_head[w][lane] = seen ? head : (float)acc;
    fix_last[w][lane] = (float)acc;
    if (lane == 0) {
        fix_row[w] = row;
        fix_has[w] = seen;
    }
    __syncthreads();
    if (fix_has[w]) {
        float tot = fix_last[w][lane];
        for (int x2 = w + 1; x2 < kPprWaves; ++x2) {
            tot += fix_head[x2][lane];
            if (fix_has[x2]) break;
        }
        partial[(int64_t)fix_row[w] * kCols + lane] = tot;
    }
}

// Merge in the paper's order plus the personalized vertex update:
//   r'(v, j) = d * sum_rows(v, j) + [v == seed_j] * ((1 - d) + d * D_j)
__global__ __launch_bounds__(kPprThreads) void k_merge_ppr(
    const int32_t *__restrict__ row_dst, const int32_t *__restrict__ block_ptr, const float *__restrict__ partial,
    int32_t V, int32_t k, int32_t B, int32_t nb, int32_t ncols, const int32_t *__restrict__ seeds,
    const float *__restrict__ rank_in, const int32_t *__restrict__ outdeg, const double *__restrict__ scalars_in,
    double damping, float *__restrict__ rank_out, float *__restrict__ contrib_out, double *__restrict__ blk) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float *acc = reinterpret_cast<float *>(smem);  // [B][kCols]
    __shared__ double red[kPprWaves][kCols];
    const int b = xcd_remap(blockIdx.x, nb);
    const int64_t vb = (int64_t)b * B;
    const int32_t nv = (int32_t)((int64_t)V - vb < B ? (int64_t)V - vb : B);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < nv * kCols; i += kPprThreads) acc[i] = 0.0f;
    __syncthreads();
    // kMergeBatch rows per wave and pass, their loads issued before any is
    // applied (rows past the range re-read its first row, unused); a
    // subgraph's rows have distinct destinations, and the barrier after each
    // subgraph keeps the subgraphs in ascending order for every destination
    for (int32_t s = 0; s < k; ++s) {
        const int32_t lo = block_ptr[(int64_t)b * k + s], hi = block_ptr[(int64_t)(b + 1) * k + s];
        for (int32_t i0 = lo + w; i0 < hi; i0 += kPprWaves * kMergeBatch) {
            int32_t d[kMergeBatch];
            float x[kMergeBatch];
#pragma unroll
            for (int j = 0; j < kMergeBatch; ++j) {
                const int32_t i = i0 + j * kPprWaves;
                const int32_t ii = i < hi ? i : lo;
                d[j] = row_dst[ii];
                x[j] = partial[(int64_t)ii * kCols + lane];
            }
#pragma unroll
            for (int j = 0; j < kMergeBatch; ++j)
                if (i0 + j * kPprWaves < hi) acc[(int32_t)(d[j] - vb) * kCols + lane] += x[j];
        }
        __syncthreads();
    }
    const double dd = damping;
    const bool live = lane < ncols;
    const int32_t seed = live ? seeds[lane] : -1;
    const double Dj = live ? scalars_in[lane * 4 + 0] : 0.0;
    double dang = 0.0, res = 0.0, mass = 0.0;
    // kMergeBatch vertices per wave and pass, their loads issued together
    // (vertices past the block re-read its first, unused); the sums keep the
    // vertex order
    for (int i0 = w; i0 < nv; i0 += kPprWaves * kMergeBatch) {
        float rin[kMergeBatch];
        int32_t odv[kMergeBatch];
#pragma unroll
        for (int j = 0; j < kMergeBatch; ++j) {
            const int i = i0 + j * kPprWaves;
            const int64_t v = vb + (i < nv ? i : 0);
            rin[j] = rank_in[v * kCols + lane];
            odv[j] = outdeg[v];
        }
#pragma unroll
        for (int j = 0; j < kMergeBatch; ++j) {
            const int i = i0 + j * kPprWaves;
            if (i >= nv) break;
            const int64_t v = vb + i;
            double r = dd * (double)acc[i * kCols + lane];
            if (v == seed) r += (1.0 - dd) + dd * Dj;
            const float rf = live ? (float)r : 0.0f;
            rank_out[v * kCols + lane] = rf;
            const int32_t od = odv[j];
            contrib_out[v * kCols + lane] = od > 0 ? rf / (float)od : 0.0f;
            if (od == 0) dang += (double)rf;
            res += fabs((double)rf - (double)rin[j]);
            mass += (double)rf;
        }
    }
    // per-column partial sums over the waves, in wave order
    double *out = blk + (int64_t)b * kCols * 4;
    red[w][lane] = dang;
    __syncthreads();
    if (w == 0) {
        double s0 = 0.0;
        for (int x = 0; x < kPprWaves; ++x) s0 += red[x][lane];
        out[lane * 4 + 0] = s0;
    }
    __syncthreads();
    red[w][lane] = res;
    __syncthreads();
    if (w == 0) {
        double s1 = 0.0;
        for (int x = 0; x < kPprWaves; ++x) s1 += red[x][lane];
        out[lane * 4 + 1] = s1;
    }
    __syncthreads();
    red[w][lane] = mass;
    __syncthreads();
    if (w == 0) {
        double s2 = 0.0;
        for (int x = 0; x < kPprWaves; ++x) s2 += red[x][lane];
        out[lane * 4 + 2] = s2;
        out[lane * 4 + 3] = 0.0;
    }
}

// r_0(v, j) = [v == seed_j]; contributions and per-column dangling mass.
constexpr int kPprInitSpan = 256;  // vertices per init block
__global__ __launch_bounds__(256) void k_ppr_init(int32_t V, int32_t ncols, const int32_t *__restrict__ seeds,
                                                  const int32_t *__restrict__ outdeg, float *__restrict__ rank_out,
                                                  float *__restrict__ contrib_out, double *__restrict__ blk) {
    __shared__ double red[4][kCols][2];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const bool live = lane < ncols;
    const int32_t seed = live ? seeds[lane] : -1;
    double dang = 0.0, mass = 0.0;
    const int64_t lo = (int64_t)blockIdx.x * kPprInitSpan;
    for (int64_t v = lo + w; v < lo + kPprInitSpan && v < V; v += 4) {
        const float r = (v == seed) ? 1.0f : 0.0f;
        rank_out[v * kCols + lane] = r;
        const int32_t od = outdeg[v];
        contrib_out[v * kCols + lane] = od > 0 ? r / (float)od : 0.0f;
        if (od == 0) dang += r;
        mass += r;
    }
    red[w][lane][0] = dang;
    red[w][lane][1] = mass;
    __syncthreads();
    if (w == 0) {
        double* out = blk + (int64_t)blockIdx.x * kCols * 4;
        out[lane * 4 + 0] = red[0][lane][0] + red[1][lane][0] + red[2][lane][0] + red[3][lane][0];
        out[lane * 4 + 1] = 0.0;
        out[lane * 4 + 2] = red[0][lane][1] + red[1][lane][1] + red[2][lane][1] + red[3][lane][1];
        out[lane * 4 + 3] = 0.0;
    }
}

// Fixed-order sums over n blocks of [kCols][4] partials: one workgroup per column.
__global__ __launch_bounds__(256) void k_reduce_cols(const double *__restrict__ blk, int32_t n,
                                                     double *__restrict__ out) {
    __shared__ double red[4];
    const int j = blockIdx.x;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int32_t b = threadIdx.x; b < n; b += 256)
        for (int c = 0; c < 4; ++c) a[c] += blk[((int64_t)b * kCols + j) * 4 + c];
    for (int c = 0; c < 4; ++c) {
        double t = block_sum_f64<256>(a[c], red);
        if (threadIdx.x == 0) out[j * 4 + c] = t;
    }
}

int32_t ppr_init_blocks(int32_t V) { return (int32_t)ceil_div(V, kPprInitSpan); }

size_t ppr_merge_lds_bytes(int32_t B) { return (size_t)B * kCols * sizeof(float); }

cagra_status launch_ppr_init(const cagra_graph *g, int32_t ncols, const int32_t *seeds, float *rank_out,
                             float *contrib_out, double *scalars_out, double *blk, hipStream_t st) {
    const int32_t nblk = ppr_init_blocks(g->V);
    k_ppr_init<<<nblk, 256, 0, st>>>(g->V, ncols, seeds, g->out_degree, rank_out, contrib_out, blk);
    CAGRA_LAUNCH_CHECK();
    k_reduce_cols<<<kCols, 256, 0, st>>>(blk, nblk, scalars_out);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

template <typename W>
static void launch_gather_cols(const cagra_segments *seg, const float *values, float *partial, hipStream_t st) {
    const int64_t row_bytes = kCols * 4, bytes = (seg->N < seg->V ? seg->N : seg->V) * row_bytes;
    const bool far = bytes > UINT32_MAX;
    // Few tiles are split until there is a workgroup per CU, as long as parts keep 256
    // edges. An iteration, whole tiles and split, us: 2^10 vertices, one tile 72 and 29;
    // 2^14, 1 / 4 / 14 tiles 898 and 90 / 273 and 41 / 93 and 39; 2^17, 30 / 119 tiles 289
    // and 91 / 103 and 89; 2^19, 122 tiles 405 and 341. Two workgroups per CU: 30 tiles
    // 104, 119 tiles 99, 241 tiles 195 against 166 whole.
    int32_t parts = 1;
    while (!far && seg->row_ptr && parts < kPprWaves && (int64_t)seg->ntiles * parts * 2 <= 256 &&
           seg->E >= (int64_t)256 * 2 * parts * seg->ntiles)
        parts *= 2;
    // Shares of 512 edges and more gain from loading ahead, shorter ones from the
    // second workgroup. An iteration with and without, us: 2^20 vertices, shares of
    // 1,024 edges 637 and 707, of 256 edges 682 and 629; 2^18, 4,096 edges 327 and 357,
    // 256 edges 165 and 156.
    const bool ahead = seg->E >= (int64_t)512 * kPprWaves * parts * seg->ntiles;
    // Values and buffer rows that exceed the 256 MB of Infinity Cache: streams that
    // leave no copies keep the values in it. With and without, us: 2^21 vertices, eight
    // segments 1,360 and 1,435; 2^20 619 and 629; but 2^18 of eight segments (218 MB)
    // 214 and 205, 2^14 99 and 97.
    const bool stream = ((int64_t)seg->V + seg->Q) * row_bytes > (int64_t)256 << 20;
    auto kern = ahead ? (stream ? k_gather_cols<W, false, true, true, false> : k_gather_cols<W, false, true, false, false>)
                      : (stream ? k_gather_cols<W, false, false, true, false> : k_gather_cols<W, false, false, false, false>);
    if (parts > 1) kern = ahead ? k_gather_cols<W, false, true, false, true> : k_gather_cols<W, false, false, false, true>;
    if constexpr (sizeof(W) == 4)
        if (far) kern = k_gather_cols<W, true, false, true, false>;
    kern<<<seg->ntiles * parts, kPprThreads, 0, st>>>(static_cast<const W *>(seg->edge_src), seg->tile_edge,
                                                      seg->tile_seg, seg->tile_span_row, values, seg->N,
                                                      (uint32_t)bytes, seg->ntiles, seg->row_ptr, parts, partial);
}

cagra_status launch_ppr_iter(const cagra_graph *g, const cagra_segments *seg, double damping, int32_t ncols,
                             const int32_t *seeds, const float *rank_in, const float *contrib_in,
                             const double *scalars_in, float *partial, float *rank_out, float *contrib_out,
                             double *scalars_out, double *blk, hipStream_t st) {
    if (seg->ntiles > 0) {
        if (edge16(seg->N)) launch_gather_cols<uint16_t>(seg, contrib_in, partial, st);
        else launch_gather_cols<uint32_t>(seg, contrib_in, partial, st);
        CAGRA_LAUNCH_CHECK();
    }
    if (cagra_status a_ = ensure_dynamic_lds((const void *)k_merge_ppr)) return a_;
    k_merge_ppr<<<seg->nb, kPprThreads, ppr_merge_lds_bytes(seg->B), st>>>(
        seg->row_dst, seg->block_ptr, partial, seg->V, seg->k, seg->B, seg->nb, ncols, seeds, rank_in, g->out_degree,
        scalars_in, damping, rank_out, contrib_out, blk);
    CAGRA_LAUNCH_CHECK();
    k_reduce_cols<<<kCols, 256, 0, st>>>(blk, seg->nb, scalars_out);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

}  // namespace cagra
