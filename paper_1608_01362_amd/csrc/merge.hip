// Cache-aware merge (Section 3.3) and the per-vertex update that follows it
// (Section 4, VertexMap of the PageRank program).
//
// Destinations are cut into blocks of B vertices whose accumulators live in
// LDS. For block b, subgraph s contributes the buffer entries
// [block_ptr[b*k+s], block_ptr[(b+1)*k+s]); every read of the buffers and of
// row_dst is sequential, and every random update hits LDS.
//
// Two schedules:
//  * k_merge_ordered: the paper's order exactly -- subgraphs in ascending
//    order, the workgroup's threads over the entries of one subgraph's range
//    (distinct destinations, so no conflicts). Used by cagra_merge for float
//    sums (plain or Neumaier-compensated) and int minimum.
//  * k_merge_pr / k_merge_lp: all 16 waves of the workgroup stream the block's
//    entries at once (flattened over subgraphs), updating shared LDS
//    accumulators with atomics whose result does not depend on their order:
//    int32 minimum for labels, and for PageRank an int64 fixed-point sum
//    (each FP32 buffer value scaled by 2^56 and truncated), which adds the buffer
//    values exactly. The epilogue then applies the vertex update.
#include <math.h>

#include "blockwalk.h"
#include "wave.h"
#include "common.h"

namespace cagra {

cagra_status launch_gather(const cagra_segments *seg, int32_t op, int32_t value_type, const void *values,
                           void *partial, hipStream_t st);
cagra_status launch_gather_clear(const cagra_segments *seg, int32_t op, int32_t value_type, const void *values,
                                 void *partial, unsigned long long *clear, hipStream_t st);

// Dynamic LDS of the fused merges, and all of it: kPrStaticLds are the static arrays
// of the PageRank merges (merge_pr_block), kFusedStaticLds covers those of the others.
constexpr size_t kFusedStaticLds = 256;
constexpr size_t kPrStaticLds = 16 * sizeof(int32_t) + 4 * (kMergeThreads / 64) * sizeof(double);
// At least what the last block's sums need (reduce4_rows).
size_t merge_fused_lds_bytes(int32_t B, int32_t k, int acc_bytes) {
    const size_t n = align_up((size_t)B * acc_bytes, 16) + (size_t)(2 * (int64_t)k + 2) * sizeof(int32_t) + 64;
    return n < 192 ? 192 : n;
}
size_t merge_fused_lds_total(int32_t B, int32_t k, int acc_bytes) {
    return merge_fused_lds_bytes(B, k, acc_bytes) + kFusedStaticLds;
}
size_t merge_pr_lds_total(int32_t B, int32_t k) { return merge_fused_lds_bytes(B, k, 8) + kPrStaticLds; }

// ---------------------------------------------------------------- ordered (paper) merge

// A workgroup of W waves per block (or per part of a block), subgraphs strictly
// in ascending order: the entries of one subgraph's range have distinct
// destinations, so they are spread over the workgroup's threads, and a barrier
// separates the subgraphs. The ranges are first listed without the empty and
// the inactive ones, so that a sparse frontier pays for its own ranges only,
// and each thread keeps its entries of the next kOrdDepth - 1 ranges in flight.
//
// What bounds it is the chain of one LDS update and one barrier per subgraph,
// so W follows the mean range length (see ordered_waves). Blocks of high
// in-degree destinations (after clustering the first few hold 30 times the mean
// entries, and one workgroup per block left the chip waiting for the heaviest)
// are cut by destination into kOrdParts parts where their ranges are long (the
// rule is at launch_ordered), each a workgroup of its own with its piece of
// every range found by binary search; the order per destination stays the same. One wave per block before -> now, us, FP32 sum: R-MAT 21 / ef
// 16 165 -> 23, R-MAT 25 / ef 32 1,698 -> 1,457 (compensated 3,722 -> 2,200),
// the same graphs clustered 1,977 -> 57 and 41,000 -> 2,970.
constexpr int kOrdDepth = 8;       // pieces of ranges in flight
constexpr int kOrdWindow = 2048;   // subgraphs whose ranges are listed at a time
constexpr int kOrdParts = 8;       // parts of a heavy block
constexpr int kOrdHeavyWaves = 16;
constexpr int kChipWaves = 256 * 32;  // resident at once

template <class Op, bool COMP>
__device__ __forceinline__ void ord_apply(typename Op::T *acc, typename Op::T *cmp, int32_t d,
                                          typename Op::T x) {
    if (COMP) {
        // Neumaier (1974) compensated summation
        float sacc = acc[d];
        float tsum = sacc + x;
        if (fabsf(sacc) >= fabsf(x)) cmp[d] += (sacc - tsum) + x;
        else cmp[d] += (x - tsum) + sacc;
        acc[d] = tsum;
    } else {
        acc[d] = Op::apply(acc[d], x);
    }
}

// First entry in [lo, hi) whose block offset is at least d (hi if none).
__device__ __forceinline__ int32_t first_dst(const uint16_t *__restrict__ dlo, int32_t lo, int32_t hi, int32_t d) {
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if ((int32_t)dlo[mid] < d) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Lists the non-empty, active ranges of subgraphs [s0, s1) in block b, cut to
// the block offsets [d0, d1) when PARTS, into lo_s/hi_s in ascending subgraph
// order; returns their count. tmp: one int per wave. Every thread calls it.
template <int W, bool PARTS>
__device__ __forceinline__ int32_t list_ranges(const uint16_t *__restrict__ dlo,
                                               const int32_t *__restrict__ block_ptr, int b, int32_t k, int32_t s0,
                                               int32_t s1, int32_t d0, int32_t d1,
                                               const uint32_t *__restrict__ seg_active, int32_t *lo_s, int32_t *hi_s,
                                               int32_t *tmp) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t n = 0;
    for (int32_t sb = s0; sb < s1; sb += W * kWave) {  // uniform
        const int32_t s = sb + (int32_t)threadIdx.x;
        int32_t lo = 0, hi = 0;
        if (s < s1 && (!seg_active || ((seg_active[s >> 5] >> (s & 31)) & 1u))) {
            lo = block_ptr[(int64_t)b * k + s];
            hi = block_ptr[(int64_t)(b + 1) * k + s];
            if (PARTS) {
                lo = first_dst(dlo, lo, hi, d0);
                hi = first_dst(dlo, lo, hi, d1);
            }
        }
        const uint64_t m = __ballot(hi > lo);
        if (lane == 0) tmp[w] = (int32_t)__popcll(m);
        __syncthreads();
        int32_t at = n + (int32_t)__popcll(m & lanemask_lt());
        for (int x = 0; x < W; ++x) {
            if (x < w) at += tmp[x];
            n += tmp[x];
        }
        if (hi > lo) {
            lo_s[at] = lo;
            hi_s[at] = hi;
        }
        __syncthreads();
    }
    return n;
}

// HEAVY = false merges the blocks that are one work item (every block when
// block_items is null), HEAVY = true the split ones, in kOrdParts parts; of the nb
// blocks from b0 on.
template <class Op, bool COMP, int W, bool HEAVY>
__global__ __launch_bounds__(W * 64) void k_merge_ordered(const uint16_t *__restrict__ row_dst_lo,
                                                          const int32_t *__restrict__ block_ptr,
                                                          const int32_t *__restrict__ block_items,
                                                          const typename Op::T *__restrict__ partial, int32_t V,
                                                          int32_t k, int32_t B, int32_t b0, int32_t nb,
                                                          typename Op::T *__restrict__ out,
                                                          const uint32_t *__restrict__ seg_active) {
    using T = typename Op::T;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int32_t tmp[W];
    const int b = b0 + (HEAVY ? (int)(blockIdx.x / kOrdParts) : xcd_remap(blockIdx.x, nb));
    if (HEAVY || block_items)
        if ((block_items[b + 1] - block_items[b] > 1) != HEAVY) return;  // uniform over the workgroup
    const int64_t vb = (int64_t)b * B;
    const int32_t nv = (int32_t)((int64_t)V - vb < B ? (int64_t)V - vb : B);
    const int32_t part = HEAVY ? (int32_t)(blockIdx.x % kOrdParts) : 0, parts = HEAVY ? kOrdParts : 1;
    const int32_t d0 = (int32_t)((int64_t)nv * part / parts), d1 = (int32_t)((int64_t)nv * (part + 1) / parts);
    const int32_t window = k < kOrdWindow ? k : kOrdWindow;
    int32_t *lo_s = reinterpret_cast<int32_t *>(smem), *hi_s = lo_s + window;
    T *acc = reinterpret_cast<T *>(hi_s + window) - d0;  // indexed by block offset in [d0, d1)
    T *cmp = acc + (HEAVY ? B / kOrdParts + 1 : B);      // Neumaier compensation terms (COMP only)
    constexpr int NT = W * kWave;
    const int tid = threadIdx.x;
    for (int i = d0 + tid; i < d1; i += NT) {
        acc[i] = Op::identity();
        if (COMP) cmp[i] = Op::identity();
    }
    for (int32_t s0 = 0; s0 < k; s0 += window) {
        // its barriers also order the accumulators' start values and the
        // previous window's last updates before what follows
        const int32_t n = list_ranges<W, HEAVY>(row_dst_lo, block_ptr, b, k, s0, min(s0 + window, k), d0, d1,
                                                seg_active, lo_s, hi_s, tmp);
        if (n == 0) continue;  // uniform
        // A step is a piece of at most NT entries of one range. Loads are
        // unconditional: threads past the piece read its first entry and steps
        // past the last one read it again; both are dropped on use.
        // the offsets stay 16-bit until used: widened, they would be converted
        // at the loop's end, which waits for every load in flight
        T x[kOrdDepth];
        uint16_t d[kOrdDepth];
        int32_t cnt[kOrdDepth];
        // lane l of every wave holds range rb + l of the list, so that a step's
        // bounds cost a lane read instead of an LDS round trip
        int32_t rb = 0, r = 0;
        const int lane = tid & 63;
        int32_t vlo = lo_s[min(lane, n - 1)], vhi = hi_s[min(lane, n - 1)];
        int32_t lo = __builtin_amdgcn_readfirstlane(vlo), hi = __builtin_amdgcn_readfirstlane(vhi);
        auto fetch = [&](int slot) {
            const int32_t c = min(hi - lo, NT);  // 0 past the last piece
            const int32_t i = c > 0 ? lo + (tid < c ? tid : 0) : lo - 1;
            cnt[slot] = c;
            x[slot] = partial[i];
            d[slot] = row_dst_lo[i];
            lo += c;
            if (lo >= hi && r + 1 < n) {  // uniform
                ++r;
                if (r - rb == kWave) {
                    rb = r;
                    vlo = lo_s[min(rb + lane, n - 1)];
                    vhi = hi_s[min(rb + lane, n - 1)];
                }
                lo = __builtin_amdgcn_readlane(vlo, r - rb);
                hi = __builtin_amdgcn_readlane(vhi, r - rb);
            }
        };
#pragma unroll
        for (int c = 0; c < kOrdDepth - 1; ++c) fetch(c);
        for (bool more = true; more;) {
#pragma unroll
            for (int c = 0; c < kOrdDepth; ++c) {
                fetch((c + kOrdDepth - 1) % kOrdDepth);
                if (cnt[c] == 0) {  // uniform; every later step is empty too
                    more = false;
                    break;
                }
                // used before the branch, so that the wait for this step's loads is
                // on both paths and none is left for the loop's start to cover
                asm volatile("" ::"v"(x[c]), "v"(d[c]));
                if (tid < cnt[c]) ord_apply<Op, COMP>(acc, cmp, (int32_t)d[c], x[c]);
                __syncthreads();  // the next subgraph's entries may update the same destinations
            }
        }
    }
    __syncthreads();
    for (int i = d0 + tid; i < d1; i += NT) out[vb + i] = COMP ? (T)(acc[i] + cmp[i]) : acc[i];
}

static size_t ordered_lds(int32_t B, int32_t k, bool comp, bool heavy) {
    const size_t window = (size_t)(k < kOrdWindow ? k : kOrdWindow);
    const size_t n = heavy ? (size_t)(B / kOrdParts + 1) : (size_t)B;
    return window * 2 * sizeof(int32_t) + n * 4 * (comp ? 2 : 1);
}

template <class Op, bool COMP, int W, bool HEAVY>
static cagra_status launch_ordered_w(const cagra_segments *seg, const int32_t *items, const void *partial, void *out,
                                     const uint32_t *seg_active, hipStream_t st) {
    using T = typename Op::T;
    auto kern = k_merge_ordered<Op, COMP, W, HEAVY>;
    if (cagra_status a_ = ensure_dynamic_lds((const void *)kern)) return a_;
    // a launch has fewer than 2^32 threads: with small blocks of many vertices it takes several
    constexpr int32_t parts = HEAVY ? kOrdParts : 1, most = (int32_t)(UINT32_MAX / (W * kWave * parts));
    for (int32_t b0 = 0; b0 < seg->nb; b0 += most) {
        const int32_t n = min(seg->nb - b0, most);
        kern<<<(unsigned)n * parts, W * kWave, ordered_lds(seg->B, seg->k, COMP, HEAVY), st>>>(
            seg->row_dst_lo, seg->block_ptr, items, (const T *)partial, seg->V, seg->k, seg->B, b0, n, (T *)out,
            seg_active);
        CAGRA_LAUNCH_CHECK();
        if (n < most) break;  // b0 + most may not fit
    }
    return CAGRA_OK;
}

// Waves per block from the mean range length Q / (k nb): a range should about
// fill the threads; more waves only make the barrier dearer. FP32 sum, us with
// 2 / 4 / 8 / 16 waves: mean 40 (V = 2 M, N = 4,096) 109 / 126 / 172 / 475,
// mean 137 (R-MAT 25) 2,125 / 1,457 / 1,503 / 4,055, mean 246 (R-MAT 23)
// 153 / 120 / 104 / 269, mean 670 (R-MAT 21) 67 / 41 / 33 / 23.
static int ordered_waves(const cagra_segments *seg) {
    const double mean = (double)seg->Q / ((double)seg->k * (double)seg->nb);
    return mean <= 60.0 ? 2 : mean <= 160.0 ? 4 : mean <= 384.0 ? 8 : 16;
}

// An upper bound of the mean range length of a split block: the work items beyond nb are
// those of the split blocks, an item has at most four times the mean entries of a block,
// and a range has at most B entries.
static double split_block_range(const cagra_segments *seg) {
    const double item = 4.0 * (double)ceil_div(seg->Q, seg->nb);
    const double most = item * ((double)seg->max_items - seg->nb + 1.0);
    const double range = (most < (double)seg->Q ? most : (double)seg->Q) / seg->k;
    return range < seg->B ? range : (double)seg->B;
}

// Split blocks get a launch of their own where their ranges take a workgroup more than two
// steps: that launch is a chain over the subgraphs behind the first one's, which shorter
// ranges do not get back. Up to eight waves are taken to make them short enough, as long
// as all blocks stay resident at once; beyond that a split block's longer chain hides
// behind the other blocks, and four steps are better still. FP32 sum, us, one wave per
// block / always two launches / with this rule: 9 K vertices, one row in 9 ranges 8.8 /
// 12.4 / 9.5; 500 K vertices, a block of 50 long rows over 489 segments 179 / 208 / 94;
// clustered R-MAT 20 in blocks of 1,024 958 / 594 / 313, clustered R-MAT 21 in blocks of
// 8,192 / 512 1,967 / 62 / 62 and 103 / 158 / 46.
template <class Op, bool COMP>
static cagra_status launch_ordered(const cagra_segments *seg, const void *partial, void *out,
                                   const uint32_t *seg_active, hipStream_t st) {
    cagra_status s;
    int waves = ordered_waves(seg);
    const int32_t *items = nullptr;  // not read where every block is merged whole
    if (seg->max_items > seg->nb) {
        const double range = split_block_range(seg);
        auto resident = [&](int w) { return (int64_t)seg->nb * w <= kChipWaves; };
        int w = waves;
        while (2 * w * kWave < range && w < 8 && resident(2 * w)) w *= 2;
        if ((resident(2 * w) ? 2 : 4) * w * kWave < range) items = seg->block_items;
        else waves = w;
    }
    switch (waves) {
        case 2: s = launch_ordered_w<Op, COMP, 2, false>(seg, items, partial, out, seg_active, st); break;
        case 4: s = launch_ordered_w<Op, COMP, 4, false>(seg, items, partial, out, seg_active, st); break;
        case 8: s = launch_ordered_w<Op, COMP, 8, false>(seg, items, partial, out, seg_active, st); break;
        default: s = launch_ordered_w<Op, COMP, 16, false>(seg, items, partial, out, seg_active, st);
    }
    if (s != CAGRA_OK || !items) return s;
    return launch_ordered_w<Op, COMP, kOrdHeavyWaves, true>(seg, items, partial, out, seg_active, st);
}

size_t merge_ordered_lds_bytes(int32_t B, int32_t op) {
    return (size_t)B * 4 * (op == CAGRA_SUM_F32_COMP ? 2 : 1);
}

cagra_status launch_merge_active(const cagra_segments *seg, int32_t op, const void *partial, void *out,
                                 const uint32_t *seg_active, hipStream_t st) {
    if (seg->nb == 0) return CAGRA_OK;
    switch (op) {
        case CAGRA_SUM_F32: return launch_ordered<OpSum, false>(seg, partial, out, seg_active, st);
        case CAGRA_SUM_F32_COMP: return launch_ordered<OpSum, true>(seg, partial, out, seg_active, st);
        case CAGRA_MIN_I32: return launch_ordered<OpMin, false>(seg, partial, out, seg_active, st);
        default: return fail(CAGRA_E_INVALID, "unknown merge op %d", op);
    }
}

cagra_status launch_merge(const cagra_segments *seg, int32_t op, const void *partial, void *out, hipStream_t st) {
    return launch_merge_active(seg, op, partial, out, nullptr, st);
}

// ---------------------------------------------------------------- fused merges

// round(x * 2^24) as int64 (exact for |x| < 2^38; halves round up in magnitude).
__device__ __forceinline__ unsigned long long fix24(float x) {
    const uint32_t u = __float_as_uint(x);
    const int e = (int)((u >> 23) & 0xffu);
    const uint64_t m = (uint64_t)((u & 0x7fffffu) | (e ? 0x800000u : 0u));
    const int sh = (e ? e : 1) - 126;
    uint64_t r = 0;
    if (sh >= 0) r = m << (sh & 63);
    else if (sh > -26) r = ((m >> (-sh - 1)) + 1) >> 1;
    return (u >> 31) ? (unsigned long long)(-(int64_t)r) : (unsigned long long)r;
}

// Streams block b's buffer entries (the ranges of all subgraphs, flattened).
// Each wave takes a contiguous share and walks it in windows of 64 entries,
// kUnroll windows per pass so that many loads are in flight (RangeWalk). Only
// the last pass of a share tests its lanes. The entries of a graph whose buffer
// is past the caches come at the card's read rate (R-MAT 25: 840 us for 3.9 GB
// in place of 856); with the buffer in the caches the walk's own instructions,
// 35 per window before and 20 now, are what is left: 38 -> 33 us for 3 M vertices.
// apply(d, x) updates the LDS accumulator of block offset d. The loads keep the
// default cache policy: the cache line at each end of a (subgraph, block) range
// is shared with the neighbouring block, which is merged at the same time on
// the same XCD and finds the line in L2.
template <typename PT, bool DENSE, class Apply>
__device__ __forceinline__ void stream_block(const uint16_t *__restrict__ dlo, const PT *__restrict__ partial,
                                             const int32_t *ofs, const int32_t *pre, int32_t k, int32_t F0,
                                             int32_t F1, Apply apply) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int32_t share = ((((F1 - F0) + 15) / 16) + 63) & ~63;
    const int32_t fa = min(F0 + w * share, F1), fb = min(fa + share, F1);
    if (fa >= fb) return;  // uniform over the wave
    RangeWalk<DENSE> walk(ofs, pre, k, __builtin_amdgcn_readfirstlane(run_of(pre, k, fa)));
    int32_t f0 = fa;
    for (; f0 + kWave * kUnroll <= fb; f0 += kWave * kUnroll) {
        uint16_t d[kUnroll];
        PT x[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int32_t fs = f0 + u * kWave;
            const uint32_t i = (uint32_t)walk.index(fs + kWave - 1, fs + lane);
            d[u] = dlo[i];
            x[u] = partial[i];
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) apply((int32_t)d[u], x[u]);
    }
    if (f0 >= fb) return;
    int32_t d[kUnroll];
    PT x[kUnroll];
    int32_t i_safe = 0;  // an entry of the share, for idle lanes
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const int32_t fs = f0 + u * kWave;
        const int32_t f = fs + lane;
        const bool valid = f < fb;
        int32_t i = i_safe;  // a window past the share: loads of an entry already read, results dropped
        if (fs < fb) {       // uniform, and so for u = 0
            const int32_t ii = walk.index(min(fs + kWave - 1, fb - 1), f);
            i_safe = __builtin_amdgcn_readfirstlane(ii);  // lane 0's entry is in the share
            i = valid ? ii : i_safe;
        }
        const int32_t dd = (int32_t)dlo[i];
        x[u] = partial[i];
        d[u] = valid ? dd : -1;
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
        if (d[u] >= 0) apply(d[u], x[u]);
}

// ---- sums over the workgroups, taken by the last one to finish
//
// A reduction of the blocks' FP64 partial sums as a launch of its own costs 3 us
// and a launch gap per iteration, a seventh of a small graph's. Where there are
// few blocks they instead count themselves off and the last one adds the partials, in the same
// fixed order. The partials are exchanged (not stored) at device scope, and a
// workgroup counts itself off after its exchanges have returned, so every
// partial is in place at the point all XCDs share before its count is; the last
// workgroup reads them there, past its own L2.
constexpr int kReduceThreads = 256;

// Writes a partial sum for the last workgroup to read; returns when it is in place.
__device__ __forceinline__ void publish4(double *blk_out, const double (&v)[4]) {
    unsigned long long old[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
        old[c] = __hip_atomic_exchange(reinterpret_cast<unsigned long long *>(blk_out + c),
                                       (unsigned long long)__double_as_longlong(v[c]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int c = 0; c < 4; ++c) asm volatile("" ::"v"(old[c]) : "memory");  // the exchanges have returned
}

// out[c] = sum of n rows of 4 partials by the workgroup's first kReduceThreads
// threads, in an order that depends on n alone; carry[3] is added to out[3].
// SHARED: rows published by running workgroups. BATCH: rows per thread loaded
// together (the order of the sum is the same). red: 4 * kReduceThreads / 64
// doubles of LDS. The whole workgroup calls it.
template <bool SHARED, int BATCH = 4>
__device__ __forceinline__ void reduce4_rows(const double *__restrict__ blk, int32_t n, double *__restrict__ out,
                                             const double *__restrict__ carry, double *red) {
    auto row = [&](int64_t i) -> double {
        if constexpr (SHARED)
            return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long *>(blk + i),
                                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        else return blk[i];
    };
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    if (threadIdx.x < kReduceThreads) {
        int32_t j = threadIdx.x;
        if constexpr (BATCH > 1)
            for (; j + (BATCH - 1) * kReduceThreads < n; j += BATCH * kReduceThreads) {
                double x[BATCH][4];
#pragma unroll
                for (int r = 0; r < BATCH; ++r)
#pragma unroll
                    for (int c = 0; c < 4; ++c) x[r][c] = row((int64_t)(j + r * kReduceThreads) * 4 + c);
#pragma unroll
                for (int r = 0; r < BATCH; ++r)
#pragma unroll
                    for (int c = 0; c < 4; ++c) a[c] += x[r][c];
            }
        for (; j < n; j += kReduceThreads) {
            double x[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c] = row((int64_t)j * 4 + c);
#pragma unroll
            for (int c = 0; c < 4; ++c) a[c] += x[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
            for (int d = 32; d >= 1; d >>= 1) a[c] += __shfl_down(a[c], d, 64);
        if ((threadIdx.x & 63) == 0)
            for (int c = 0; c < 4; ++c) red[c * (kReduceThreads / 64) + (threadIdx.x >> 6)] = a[c];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int c = threadIdx.x;
        double t = 0.0;
        for (int i = 0; i < kReduceThreads / 64; ++i) t += red[c * (kReduceThreads / 64) + i];
        out[c] = c == 3 && carry ? t + carry[3] : t;
    }
}

// Counts a finished workgroup off; true (in every thread) for the last of n.
// flag: an int of LDS. Called after publish4 by the same thread.
__device__ __forceinline__ bool last_of(unsigned long long *ticket, int32_t n, int32_t *flag) {
    if (threadIdx.x == 0)
        *flag = __hip_atomic_fetch_add(ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                (unsigned long long)(n - 1);
    __syncthreads();
    return *flag != 0;
}

constexpr int kEpiBatch = 8;  // vertices per thread whose loads are in flight together

// PageRank vertex update of block b from its exact sums acc (LDS, int64 fixed
// point); writes the block's FP64 partial sums to blk_out[0..3]: dangling mass,
// L1 residual, mass, and the range flag (1 when the buffer values merged into
// the block -- `am` is this thread's share of their absolute sum -- were
// non-finite or too large for exact fixed-point sums, else 0).
template <bool BF16OUT, int EPI = kEpiBatch>
__device__ __forceinline__ void pr_epilogue(const unsigned long long *acc, int32_t V, int64_t vb, int32_t nv,
                                            const float *__restrict__ rank_in, const int32_t *__restrict__ outdeg,
                                            const double *__restrict__ scalars_in, double damping, int32_t seed,
                                            float *__restrict__ rank_out, void *__restrict__ contrib_out,
                                            double *__restrict__ blk_out, double am, double *red) {
    const double dd = damping;
    // teleport and dangling mass: spread over all vertices, or (personalized,
    // seed >= 0) returned to the seed vertex alone
    const double base = seed < 0 ? (1.0 - dd) / (double)V + dd * scalars_in[0] / (double)V : 0.0;
    const double sbase = (1.0 - dd) + dd * scalars_in[0];
    double dang = 0.0, res = 0.0, mass = 0.0;
    // EPI vertices per thread per pass; sums keep the vertex order. The loads are
    // conditional, so they go out pair by pair: measured faster than issuing all
    // of them at once, which crowds the memory queue that the CU's other
    // workgroup streams its buffer entries through.
    for (int i0 = threadIdx.x; i0 < nv; i0 += kMergeThreads * EPI) {
        float rin[EPI];
        int32_t odv[EPI];
#pragma unroll
        for (int u = 0; u < EPI; ++u) {
            const int i = i0 + u * kMergeThreads;
            rin[u] = i < nv ? rank_in[vb + i] : 0.0f;
            odv[u] = i < nv ? outdeg[vb + i] : 0;
        }
#pragma unroll
        for (int u = 0; u < EPI; ++u) {
            const int i = i0 + u * kMergeThreads;
            if (i >= nv) break;
            const int64_t v = vb + i;
            const double sum = (double)(long long)acc[i] * kFixInv;
            const float r = (float)((v == seed ? sbase : base) + dd * sum);
            rank_out[v] = r;
            const int32_t od = odv[u];
            const float c = od > 0 ? r / (float)od : 0.0f;
            if (BF16OUT) reinterpret_cast<uint16_t *>(contrib_out)[v] = f32_to_bf16(c);
            else reinterpret_cast<float *>(contrib_out)[v] = c;
            if (od == 0) dang += (double)r;
            res += fabs((double)r - (double)rin[u]);
            mass += (double)r;
        }
    }
    double v4[4] = {dang, res, mass, am};
    block_sum4_f64<kMergeThreads>(v4, red);
    if (threadIdx.x == 0) {
        blk_out[0] = v4[0];
        blk_out[1] = v4[1];
        blk_out[2] = v4[2];
        blk_out[3] = range_flag(v4[3]);
    }
}

template <int EPI>
__device__ __forceinline__ void load_vertices(const float *__restrict__ rank_in, const int32_t *__restrict__ outdeg,
                                              int64_t vb, int32_t nv, int i0, float (&rin)[EPI], int32_t (&odv)[EPI]) {
#pragma unroll
    for (int u = 0; u < EPI; ++u) {
        const int i = i0 + u * kMergeThreads;
        rin[u] = i < nv ? rank_in[vb + i] : 0.0f;
        odv[u] = i < nv ? outdeg[vb + i] : 0;
    }
}

// The same for the blocks of a small graph, alone on their CUs: the inputs of
// their first kMergeThreads * EPI vertices (rin, odv, loaded before the buffer
// entries) and the dangling mass are at hand, which takes one round trip to
// memory out of the chain, and the sums go to the last block (publish4).
template <bool BF16OUT, int EPI>
__device__ __forceinline__ void pr_epilogue_small(const unsigned long long *acc, int32_t V, int64_t vb, int32_t nv,
                                                  const float *__restrict__ rank_in,
                                                  const int32_t *__restrict__ outdeg, double dangling, double damping,
                                                  int32_t seed, float *__restrict__ rank_out,
                                                  void *__restrict__ contrib_out, double *__restrict__ blk_out,
                                                  double am, double *red, float (&rin)[EPI], int32_t (&odv)[EPI]) {
    const double dd = damping;
    const double base = seed < 0 ? (1.0 - dd) / (double)V + dd * dangling / (double)V : 0.0;
    const double sbase = (1.0 - dd) + dd * dangling;
    double dang = 0.0, res = 0.0, mass = 0.0;
    for (int i0 = threadIdx.x; i0 < nv; i0 += kMergeThreads * EPI) {
        if (i0 >= kMergeThreads * EPI) load_vertices<EPI>(rank_in, outdeg, vb, nv, i0, rin, odv);
#pragma unroll
        for (int u = 0; u < EPI; ++u) {
            const int i = i0 + u * kMergeThreads;
            if (i >= nv) break;
            const int64_t v = vb + i;
            const double sum = (double)(long long)acc[i] * kFixInv;
            const float r = (float)((v == seed ? sbase : base) + dd * sum);
            rank_out[v] = r;
            const int32_t od = odv[u];
            const float c = od > 0 ? r / (float)od : 0.0f;
            if (BF16OUT) reinterpret_cast<uint16_t *>(contrib_out)[v] = f32_to_bf16(c);
            else reinterpret_cast<float *>(contrib_out)[v] = c;
            if (od == 0) dang += (double)r;
            res += fabs((double)r - (double)rin[u]);
            mass += (double)r;
        }
    }
    double v4[4] = {dang, res, mass, am};
    block_sum4_f64<kMergeThreads>(v4, red);
    if (threadIdx.x == 0) {
        v4[3] = range_flag(v4[3]);
        publish4(blk_out, v4);
    }
}

// Item j of the S items of block b: the block's entries (flattened over
// subgraphs) [P*j/S, P*(j+1)/S). With S == 1 the item is the whole block and
// the vertex update follows at once. Otherwise the item stores its exact int64
// sums in its own slot of the workspace and the absolute sum of its buffer
// values in *item_abs, and k_merge_pr_finish adds the S slots of the block
// (exactly, so the split does not change any result) and applies the update.
template <bool BF16OUT, bool DENSE, int EPI = kEpiBatch, bool SMALL = false>
__device__ __forceinline__ void merge_pr_block(
    const uint16_t *__restrict__ row_dst_lo, const int32_t *__restrict__ block_ptr,
    const float *__restrict__ partial, int32_t V, int32_t k, int32_t B, int b, int32_t j, int32_t S,
    const float *__restrict__ rank_in, const int32_t *__restrict__ outdeg, const double *__restrict__ scalars_in,
    double damping, int32_t seed, float *__restrict__ rank_out, void *__restrict__ contrib_out,
    double *__restrict__ blk_out, unsigned long long *__restrict__ slot, double *__restrict__ item_abs,
    unsigned char *smem) {
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(smem);
    int32_t *ofs = reinterpret_cast<int32_t *>(smem + align_up((size_t)B * 8, 16));
    int32_t *pre = ofs + k;
    __shared__ int32_t tmp[16];
    __shared__ double red[4 * (kMergeThreads / 64)];
    static_assert(sizeof(tmp) + sizeof(red) <= kPrStaticLds, "the LDS that the capacity check counts");

    const int64_t vb = (int64_t)b * B;
    const int32_t nv = (int32_t)((int64_t)V - vb < B ? (int64_t)V - vb : B);
    [[maybe_unused]] float rin[EPI];
    [[maybe_unused]] int32_t odv[EPI];
    [[maybe_unused]] double dangling;
    if constexpr (SMALL) {
        load_vertices<EPI>(rank_in, outdeg, vb, nv, threadIdx.x, rin, odv);
        dangling = scalars_in[0];
    }
    for (int i = threadIdx.x; i < nv; i += kMergeThreads) acc[i] = 0ull;
    const int32_t P = load_block_ranges(block_ptr, b, k, ofs, pre, tmp);
    const int32_t F0 = (int32_t)((int64_t)P * j / S), F1 = (int32_t)((int64_t)P * (j + 1) / S);
    float am = 0.0f;  // this thread's share of the absolute buffer mass (range check)
    stream_block<float, DENSE>(row_dst_lo, partial, ofs, pre, k, F0, F1, [&](int32_t d, float x) {
        atomicAdd(&acc[d], fix56_wave(x));
        am += fabsf(x);
    });
    __syncthreads();
    if (S > 1) {
        for (int i = threadIdx.x; i < nv; i += kMergeThreads) slot[i] = acc[i];
        const double tot = block_sum_f64<kMergeThreads>((double)am, red);
        if (threadIdx.x == 0) *item_abs = tot;
        return;
    }
    if constexpr (SMALL)
        pr_epilogue_small<BF16OUT, EPI>(acc, V, vb, nv, rank_in, outdeg, dangling, damping, seed, rank_out,
                                        contrib_out, blk_out, (double)am, red, rin, odv);
    else
        pr_epilogue<BF16OUT, EPI>(acc, V, vb, nv, rank_in, outdeg, scalars_in, damping, seed, rank_out, contrib_out,
                                  blk_out, (double)am, red);
}

// Slot of item j of a split block b whose first item is items_b: 2*(items_b - b)
// + j. items_b - b counts the extra items of earlier blocks; a split block has
// S >= 2 items and adds S - 1 >= S / 2 extra ones, so the slot ranges of split
// blocks are disjoint and all lie below 2 * (items[nb] - nb).
__device__ __forceinline__ int64_t split_slot(int32_t items_b, int32_t b, int32_t j) {
    return 2 * (int64_t)(items_b - b) + j;
}

constexpr int32_t kItemGroup = 4;  // work items per XCD group (1, 2, 4 and 16 time alike; contiguous is slower)

template <bool BF16OUT, bool DENSE>
__global__ __launch_bounds__(kMergeThreads) void k_merge_pr(
    const uint16_t *__restrict__ row_dst_lo, const int32_t *__restrict__ block_ptr,
    const int32_t *__restrict__ block_items, const float *__restrict__ partial, int32_t V, int32_t k, int32_t B,
    int32_t nb, const float *__restrict__ rank_in, const int32_t *__restrict__ outdeg,
    const double *__restrict__ scalars_in, double damping, int32_t seed, float *__restrict__ rank_out,
    void *__restrict__ contrib_out, double *__restrict__ blk, unsigned long long *__restrict__ slots,
    double *__restrict__ item_abs, int32_t one_item) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // the grid is the bound max_items; slots past the actual item count exit,
    // and the XCD remap spreads the actual items (not the bound) over the XCDs.
    // one_item (the bound equals nb): every block is one item, known without
    // reading the item table; each block is then merged whole, which is right
    // whatever the table holds
    const int32_t total = one_item ? nb : block_items[nb];
    if (total > (int32_t)gridDim.x) {
        // a bound below the item count (an invalid max_items): the slot
        // workspace may be too small, so nothing is merged and the scalars
        // become NaN (block 0's partial sums feed the reduction)
        if (blockIdx.x == 0 && threadIdx.x < 4) blk[threadIdx.x] = __builtin_nan("");
        return;
    }
    if ((int32_t)blockIdx.x >= total) return;  // uniform over the workgroup
    const ItemPlace ip = place_item(block_items, nb, total, xcd_group_map(blockIdx.x, total, kItemGroup));
    const int32_t b = ip.b, j = ip.j, S = ip.S;
    unsigned long long *slot = S > 1 ? slots + split_slot(block_items[b], b, j) * B : nullptr;
    double *ia = S > 1 ? item_abs + block_items[b] + j : nullptr;
    merge_pr_block<BF16OUT, DENSE>(row_dst_lo, block_ptr, partial, V, k, B, b, j, S, rank_in, outdeg, scalars_in,
                                   damping, seed, rank_out, contrib_out, blk + (int64_t)b * 4, slot, ia, smem);
}

// The merge of a small graph: every block is one work item, and the last block
// to finish adds the blocks' sums (the accumulators' LDS is free by then).
template <bool BF16OUT>
__global__ __launch_bounds__(kMergeThreads) void k_merge_pr_small(
    const uint16_t *__restrict__ row_dst_lo, const int32_t *__restrict__ block_ptr, const float *__restrict__ partial,
    int32_t V, int32_t k, int32_t B, int32_t nb, const float *__restrict__ rank_in,
    const int32_t *__restrict__ outdeg, const double *scalars_in, double damping, int32_t seed,
    float *__restrict__ rank_out, void *__restrict__ contrib_out, double *__restrict__ blk,
    unsigned long long *__restrict__ ticket, double *scalars_out) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int b = xcd_remap(blockIdx.x, nb);
    merge_pr_block<BF16OUT, false, kEpiBatch, true>(row_dst_lo, block_ptr, partial, V, k, B, b, 0, 1, rank_in, outdeg,
                                                   scalars_in, damping, seed, rank_out, contrib_out,
                                                   blk + (int64_t)b * 4, nullptr, nullptr, smem);
    if (last_of(ticket, nb, reinterpret_cast<int32_t *>(smem)))
        reduce4_rows<true>(blk, nb, scalars_out, scalars_in, reinterpret_cast<double *>(smem) + 1);
}

// Sum of the item slots of each split block, written into its first slot.
// kSlotParts workgroups share a block (one part of its vertices each), so the
// heaviest block's slots are read at the rate of several CUs.
constexpr int kSlotParts = 8;
constexpr int kSlotThreads = 256;
__global__ __launch_bounds__(kSlotThreads) void k_slot_sum(const int32_t *__restrict__ block_items, int32_t V,
                                                           int32_t B, int32_t nb, int32_t max_items, int32_t parts,
                                                           unsigned long long *__restrict__ slots) {
    if (block_items[nb] > max_items) return;  // invalid bound: slots not written (see k_merge_pr)
    const int32_t b = blockIdx.x / parts, part = blockIdx.x % parts;
    const int32_t S = block_items[b + 1] - block_items[b];
    if (S <= 1) return;  // merged in one piece
    const int64_t vb = (int64_t)b * B;
    const int32_t nv = (int32_t)((int64_t)V - vb < B ? (int64_t)V - vb : B);
    const int32_t span = (nv + parts - 1) / parts;
    const int32_t lo = part * span, hi = min(lo + span, nv);
    unsigned long long *first = slots + split_slot(block_items[b], b, 0) * B;
    constexpr int kSlotBatch = 8;  // independent loads in flight per thread
    for (int32_t i = lo + threadIdx.x; i < hi; i += kSlotThreads) {
        unsigned long long t = first[i];
        int32_t j = 1;
        for (; j + kSlotBatch <= S; j += kSlotBatch) {
            unsigned long long x[kSlotBatch];
#pragma unroll
            for (int u = 0; u < kSlotBatch; ++u) x[u] = first[(int64_t)(j + u) * B + i];
#pragma unroll
            for (int u = 0; u < kSlotBatch; ++u) t += x[u];
        }
        for (; j < S; ++j) t += first[(int64_t)j * B + i];
        first[i] = t;
    }
}

// Vertex update of the split blocks from the summed first slot.
template <bool BF16OUT>
__global__ __launch_bounds__(kMergeThreads) void k_merge_pr_finish(
    const int32_t *__restrict__ block_items, int32_t V, int32_t B, int32_t nb, const float *__restrict__ rank_in,
    const int32_t *__restrict__ outdeg, const double *__restrict__ scalars_in, double damping, int32_t seed,
    float *__restrict__ rank_out, void *__restrict__ contrib_out, double *__restrict__ blk,
    const unsigned long long *__restrict__ slots, const double *__restrict__ item_abs, int32_t max_items) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ double red[4 * (kMergeThreads / 64)];
    const int32_t b = blockIdx.x;
    if (block_items[nb] > max_items) return;  // invalid bound: slots not written (see k_merge_pr)
    if (block_items[b + 1] - block_items[b] <= 1) return;  // merged in one piece
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(smem);
    const int64_t vb = (int64_t)b * B;
    const int32_t nv = (int32_t)((int64_t)V - vb < B ? (int64_t)V - vb : B);
    const unsigned long long *first = slots + split_slot(block_items[b], b, 0) * B;
    for (int i = threadIdx.x; i < nv; i += kMergeThreads) acc[i] = first[i];
    // absolute buffer mass of the block: its items' sums in item order (thread 0)
    double am = 0.0;
    if (threadIdx.x == 0)
        for (int32_t it = block_items[b]; it < block_items[b + 1]; ++it) am += item_abs[it];
    __syncthreads();
    pr_epilogue<BF16OUT>(acc, V, vb, nv, rank_in, outdeg, scalars_in, damping, seed, rank_out, contrib_out,
                         blk + (int64_t)b * 4, am, red);
}

// Order-free merge of float buffer values into float sums (int64 fixed point,
// 2^-24 resolution, |sums| < 2^38): used where the values are not bounded by
// one, e.g. sums of log-degrees.
__global__ __launch_bounds__(kMergeThreads) void k_merge_sum_fixed24(
    const uint16_t *__restrict__ row_dst_lo, const int32_t *__restrict__ block_ptr,
    const float *__restrict__ partial, int32_t V, int32_t k, int32_t B, int32_t nb, float *__restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(smem);
    int32_t *ofs = reinterpret_cast<int32_t *>(smem + align_up((size_t)B * 8, 16));
    int32_t *pre = ofs + k;
    __shared__ int32_t tmp[16];
    const int b = xcd_remap(blockIdx.x, nb);
    const int64_t vb = (int64_t)b * B;
    const int32_t nv = (int32_t)((int64_t)V - vb < B ? (int64_t)V - vb : B);
    for (int i = threadIdx.x; i < nv; i += kMergeThreads) acc[i] = 0ull;
    const int32_t P = load_block_ranges(block_ptr, b, k, ofs, pre, tmp);
    stream_block<float, false>(row_dst_lo, partial, ofs, pre, k, 0, P,
                               [&](int32_t d, float x) { atomicAdd(&acc[d], fix24(x)); });
    __syncthreads();
    for (int i = threadIdx.x; i < nv; i += kMergeThreads)
        out[vb + i] = (float)((double)(long long)acc[i] * (1.0 / 16777216.0));
}

cagra_status launch_merge_sum_fixed24(const cagra_segments *seg, const float *partial, float *out, hipStream_t st) {
    if (cagra_status a_ = ensure_dynamic_lds((const void *)k_merge_sum_fixed24)) return a_;
    if (merge_fused_lds_total(seg->B, seg->k, 8) > CAGRA_LDS_BYTES)
        return fail(CAGRA_E_CAPACITY, "B=%d with k=%d exceeds the merge kernel's LDS", seg->B, seg->k);
    k_merge_sum_fixed24<<<seg->nb, kMergeThreads, merge_fused_lds_bytes(seg->B, seg->k, 8), st>>>(
        seg->row_dst_lo, seg->block_ptr, partial, seg->V, seg->k, seg->B, seg->nb, out);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

// Many graphs: one workgroup per entry of the global block list (they stride past
// the largest grid).
__global__ __launch_bounds__(kMergeThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_multi_merge(
    const MultiDesc *__restrict__ desc, const int32_t *__restrict__ block_graph, int64_t total_blocks, int parity,
    double damping, double *__restrict__ blk, unsigned long long *__restrict__ tickets) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    for (int64_t gb = blockIdx.x; gb < total_blocks; gb += gridDim.x) {
        __syncthreads();  // LDS reuse across blocks
        const int gi = uniform(block_graph[gb]);
        const MultiDesc &d = desc[gi];
        // kept within 64 VGPRs (two workgroups per CU): at 66 one fitted, and the
        // merge of 48 graphs took 22.5 us and its sums 4.6 us more; now 21.4 us
        // with the sums
        merge_pr_block<false, false, 4, true>(
            uniform(d.row_dst_lo), uniform(d.block_ptr), uniform(d.partial), uniform(d.V), uniform(d.k), uniform(d.B),
            uniform((int32_t)(gb - d.block_base)), 0, 1, uniform(d.rank[parity]), uniform(d.out_degree),
            uniform(d.scalars[parity]), damping, -1, uniform(d.rank[1 - parity]), uniform(d.contrib[1 - parity]),
            blk + gb * 4, nullptr, nullptr, smem);
        if (!tickets) continue;
        // the last block of a graph adds that graph's sums (its descriptor is
        // read again rather than held in registers over the merge)
        int gr = gi;
        asm volatile("" : "+s"(gr));
        const MultiDesc &e = desc[gr];
        if (last_of(tickets + gr, e.nb, reinterpret_cast<int32_t *>(smem)))
            reduce4_rows<true, 1>(blk + e.block_base * 4, e.nb, e.scalars[1 - parity], e.scalars[parity],
                                  reinterpret_cast<double *>(smem) + 1);
    }
}

// Uniform start vectors of many graphs, over the block list as above.
__global__ __launch_bounds__(256) void k_multi_start(const MultiDesc *__restrict__ desc,
                                                     const int32_t *__restrict__ block_graph, int64_t total_blocks,
                                                     double *__restrict__ blk) {
    __shared__ double red[4];
    for (int64_t gb = blockIdx.x; gb < total_blocks; gb += gridDim.x) {
        const int gi = block_graph[gb];
        const MultiDesc &d = desc[gi];
        const int64_t lo = (gb - d.block_base) * (int64_t)d.B;
        const int64_t hi = lo + d.B < d.V ? lo + d.B : d.V;
        const float r = 1.0f / (float)d.V;
        double dang = 0.0, mass = 0.0;
        for (int64_t v = lo + threadIdx.x; v < hi; v += 256) {
            d.rank[0][v] = r;
            const int32_t od = d.out_degree[v];
            d.contrib[0][v] = od > 0 ? r / (float)od : 0.0f;
            if (od == 0) dang += (double)r;
            mass += (double)r;
        }
        dang = block_sum_f64<256>(dang, red);
        mass = block_sum_f64<256>(mass, red);
        if (threadIdx.x == 0) {
            blk[gb * 4 + 0] = dang;
            blk[gb * 4 + 1] = 0.0;
            blk[gb * 4 + 2] = mass;
            blk[gb * 4 + 3] = 0.0;
        }
    }
}

// Per graph: fixed-order sum of its blocks' partials into scalars[parity]. With
// carry, the range count [3] also adds the previous step's (scalars[1 - parity]).
__global__ __launch_bounds__(kReduceThreads) void k_multi_reduce(const MultiDesc *__restrict__ desc,
                                                                 const double *__restrict__ blk, int parity,
                                                                 int carry) {
    __shared__ double red[4 * kReduceThreads / 64];
    const MultiDesc &d = desc[blockIdx.x];
    reduce4_rows<false>(blk + d.block_base * 4, d.nb, d.scalars[parity], carry ? d.scalars[1 - parity] : nullptr, red);
}

cagra_status launch_multi_start(const MultiDesc *desc, const int32_t *block_graph, int64_t total_blocks,
                                int32_t ngraphs, double *blk, int grid, hipStream_t st) {
    if (total_blocks == 0) return CAGRA_OK;
    k_multi_start<<<grid, 256, 0, st>>>(desc, block_graph, total_blocks, blk);
    CAGRA_LAUNCH_CHECK();
    k_multi_reduce<<<ngraphs, kReduceThreads, 0, st>>>(desc, blk, 0, 0);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

cagra_status launch_multi_merge(const MultiDesc *desc, const int32_t *block_graph, int64_t total_blocks,
                                int32_t ngraphs, int parity, double damping, double *blk, unsigned long long *tickets,
                                size_t lds, int grid, hipStream_t st) {
    if (cagra_status a_ = ensure_dynamic_lds((const void *)k_multi_merge)) return a_;
    if (total_blocks == 0) return CAGRA_OK;
    k_multi_merge<<<grid, kMergeThreads, lds, st>>>(desc, block_graph, total_blocks, parity, damping, blk, tickets);
    CAGRA_LAUNCH_CHECK();
    if (tickets) return CAGRA_OK;
    k_multi_reduce<<<ngraphs, kReduceThreads, 0, st>>>(desc, blk, 1 - parity, 1);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

template <bool DENSE>
__global__ __launch_bounds__(kMergeThreads) void k_merge_lp(
    const uint16_t *__restrict__ row_dst_lo, const int32_t *__restrict__ block_ptr,
    const int32_t *__restrict__ partial, int32_t V, int32_t k, int32_t B, int32_t nb,
    const int32_t *__restrict__ labels_in, int32_t *__restrict__ labels_out, int32_t *__restrict__ blk_changed) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int32_t *acc = reinterpret_cast<int32_t *>(smem);
    int32_t *ofs = reinterpret_cast<int32_t *>(smem + align_up((size_t)B * 4, 16));
    int32_t *pre = ofs + k;
    __shared__ int32_t tmp[16];
    __shared__ int32_t cnt[16];

    const int b = xcd_remap(blockIdx.x, nb);
    const int64_t vb = (int64_t)b * B;
    const int32_t nv = (int32_t)((int64_t)V - vb < B ? (int64_t)V - vb : B);
    // kEpiBatch labels per thread and pass (conditional loads, as in the
    // PageRank vertex update) before the accumulators take them
    for (int i0 = threadIdx.x; i0 < nv; i0 += kMergeThreads * kEpiBatch) {
        int32_t l[kEpiBatch];
#pragma unroll
        for (int u = 0; u < kEpiBatch; ++u) {
            const int i = i0 + u * kMergeThreads;
            l[u] = i < nv ? labels_in[vb + i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kEpiBatch; ++u) {
            const int i = i0 + u * kMergeThreads;
            if (i < nv) acc[i] = l[u];
        }
    }
    const int32_t P = load_block_ranges(block_ptr, b, k, ofs, pre, tmp);
    stream_block<int32_t, DENSE>(row_dst_lo, partial, ofs, pre, k, 0, P,
                                 [&](int32_t d, int32_t x) { atomicMin(&acc[d], x); });
    __syncthreads();
    int32_t changed = 0;
    for (int i0 = threadIdx.x; i0 < nv; i0 += kMergeThreads * kEpiBatch) {
        int32_t old[kEpiBatch];
#pragma unroll
        for (int u = 0; u < kEpiBatch; ++u) {
            const int i = i0 + u * kMergeThreads;
            old[u] = i < nv ? labels_in[vb + i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kEpiBatch; ++u) {
            const int i = i0 + u * kMergeThreads;
            if (i >= nv) break;
            const int32_t l = acc[i];
            labels_out[vb + i] = l;
            changed += (l != old[u]) ? 1 : 0;
        }
    }
    for (int dd = 32; dd >= 1; dd >>= 1) changed += __shfl_down(changed, dd, 64);
    if ((threadIdx.x & 63) == 0) cnt[threadIdx.x >> 6] = changed;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t tot = 0;
        for (int i = 0; i < kMergeThreads / 64; ++i) tot += cnt[i];
        blk_changed[b] = tot;
    }
}

// PageRank start vector: contributions, dangling mass and total mass.
constexpr int kInitSpan = 16384;  // vertices per init block

constexpr int kInitThreads = 1024;  // 16 vertices each; 256 threads took 28 us for 4 M vertices (50 MB)
constexpr int kInitBatch = 8;       // vertices per thread whose loads are in flight together

template <bool BF16OUT>
__global__ __launch_bounds__(kInitThreads) void k_pr_init(const float *__restrict__ rank,
                                                          const int32_t *__restrict__ outdeg, int32_t V,
                                                          void *__restrict__ contrib_out, double *__restrict__ blk) {
    __shared__ double red[4 * (kInitThreads / 64)];
    const int64_t lo = (int64_t)blockIdx.x * kInitSpan;
    const int64_t hi = lo + kInitSpan < V ? lo + kInitSpan : V;
    double part[4] = {0.0, 0.0, 0.0, 0.0};  // dangling mass, -, mass, non-finite ranks
    for (int64_t v0 = lo + threadIdx.x; v0 < hi; v0 += kInitThreads * kInitBatch) {
        float r[kInitBatch];
        int32_t od[kInitBatch];
#pragma unroll
        for (int j = 0; j < kInitBatch; ++j) {  // vertices past the span read its first again, unused
            const int64_t v = v0 + j * kInitThreads < hi ? v0 + j * kInitThreads : v0;
            r[j] = rank[v];
            od[j] = outdeg[v];
        }
#pragma unroll
        for (int j = 0; j < kInitBatch; ++j) {
            const int64_t v = v0 + j * kInitThreads;
            if (v >= hi) break;
            const float c = od[j] > 0 ? r[j] / (float)od[j] : 0.0f;
            if (BF16OUT) reinterpret_cast<uint16_t *>(contrib_out)[v] = f32_to_bf16(c);
            else reinterpret_cast<float *>(contrib_out)[v] = c;
            if (od[j] == 0) part[0] += (double)r[j];
            part[2] += (double)r[j];
            part[3] += isfinite(r[j]) ? 0.0 : 1.0;
        }
    }
    block_sum4_f64<kInitThreads>(part, red);
    if (threadIdx.x == 0)
        for (int c = 0; c < 4; ++c) blk[(int64_t)blockIdx.x * 4 + c] = part[c];
}

// Fixed-order FP64 reduction of n rows of 4 partial sums. With carry non-null,
// out[3] also adds carry[3] (the range count accumulates over iterations).
__global__ __launch_bounds__(kReduceThreads) void k_reduce4(const double *__restrict__ blk, int32_t n,
                                                            double *__restrict__ out,
                                                            const double *__restrict__ carry) {
    __shared__ double red[4 * kReduceThreads / 64];
    reduce4_rows<false>(blk, n, out, carry, red);
}

__global__ __launch_bounds__(256) void k_reduce_i32(const int32_t *__restrict__ blk, int32_t n,
                                                    int32_t *__restrict__ out) {
    __shared__ int32_t red[4];
    int32_t a = 0;
    for (int32_t j = threadIdx.x; j < n; j += 256) a += blk[j];
    for (int d = 32; d >= 1; d >>= 1) a += __shfl_down(a, d, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = red[0] + red[1] + red[2] + red[3];
}

// Fixed-order reductions of per-block partial sums (also used by the push path).
cagra_status launch_reduce4(const double *blk, int32_t n, double *out, const double *carry, hipStream_t st) {
    k_reduce4<<<1, kReduceThreads, 0, st>>>(blk, n, out, carry);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}
cagra_status launch_reduce_i32(const int32_t *blk, int32_t n, int32_t *out, hipStream_t st) {
    k_reduce_i32<<<1, 256, 0, st>>>(blk, n, out);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

int32_t init_blocks(int32_t V) { return (int32_t)ceil_div(V, kInitSpan); }

// Iteration workspace: the FP64 (or int32) per-block partial sums at offset 0,
// then the int64 slots of the work items of split merge blocks.
size_t ws_blk_bytes(int32_t V, int32_t nb) {
    const int64_t n = nb > init_blocks(V) ? nb : init_blocks(V);
    return align_up((size_t)n * 4 * sizeof(double), 256);
}
// One double per merge work item: the absolute buffer mass of a split item.
size_t ws_item_bytes(const cagra_segments *seg) { return align_up((size_t)seg->max_items * sizeof(double), 256); }
size_t ws_slot_bytes(const cagra_segments *seg) {
    return (size_t)2 * (size_t)(seg->max_items - seg->nb) * (size_t)seg->B * sizeof(unsigned long long);
}

cagra_status launch_pr_init(const cagra_graph *g, int32_t contrib_type, const float *rank, void *contrib_out,
                            double *scalars_out, void *ws, hipStream_t st) {
    const int32_t nblk = init_blocks(g->V);
    double *blk = reinterpret_cast<double *>(ws);
    if (contrib_type == CAGRA_BF16) k_pr_init<true><<<nblk, kInitThreads, 0, st>>>(rank, g->out_degree, g->V, contrib_out, blk);
    else k_pr_init<false><<<nblk, kInitThreads, 0, st>>>(rank, g->out_degree, g->V, contrib_out, blk);
    CAGRA_LAUNCH_CHECK();
    k_reduce4<<<1, kReduceThreads, 0, st>>>(blk, nblk, scalars_out, nullptr);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

template <bool BF16OUT, bool DENSE>
static cagra_status launch_merge_pr_t(const cagra_graph *g, const cagra_segments *seg, double damping, int32_t seed,
                                      const float *rank_in, const double *scalars_in, const float *partial,
                                      float *rank_out, void *contrib_out, double *scalars_out, void *ws,
                                      hipStream_t st) {
    if (cagra_status a_ = ensure_dynamic_lds((const void *)k_merge_pr<BF16OUT, DENSE>)) return a_;
    if (cagra_status a_ = ensure_dynamic_lds((const void *)k_merge_pr_finish<BF16OUT>)) return a_;
    double *blk = reinterpret_cast<double *>(ws);
    double *item_abs = reinterpret_cast<double *>(reinterpret_cast<char *>(ws) + ws_blk_bytes(seg->V, seg->nb));
    unsigned long long *slots = reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(ws) +
                                                                       ws_blk_bytes(seg->V, seg->nb) +
                                                                       ws_item_bytes(seg));
    k_merge_pr<BF16OUT, DENSE><<<seg->max_items, kMergeThreads, merge_fused_lds_bytes(seg->B, seg->k, 8), st>>>(
        seg->row_dst_lo, seg->block_ptr, seg->block_items, partial, seg->V, seg->k, seg->B, seg->nb, rank_in,
        g->out_degree, scalars_in, damping, seed, rank_out, contrib_out, blk, slots, item_abs,
        seg->max_items == seg->nb ? 1 : 0);
    CAGRA_LAUNCH_CHECK();
    // max_items is a bound on the item count; when it equals nb (a caller that
    // read block_items[nb] after the build may tighten it so) no block is split
    // and the slot pass has nothing to do
    if (seg->max_items > seg->nb) {
        const int32_t parts = (int64_t)seg->nb * kSlotParts <= INT32_MAX ? kSlotParts : 1;
        k_slot_sum<<<(unsigned)((int64_t)seg->nb * parts), kSlotThreads, 0, st>>>(
            seg->block_items, seg->V, seg->B, seg->nb, seg->max_items, parts, slots);
        CAGRA_LAUNCH_CHECK();
        k_merge_pr_finish<BF16OUT><<<seg->nb, kMergeThreads, (size_t)seg->B * 8, st>>>(
            seg->block_items, seg->V, seg->B, seg->nb, rank_in, g->out_degree, scalars_in, damping, seed, rank_out,
            contrib_out, blk, slots, item_abs, seg->max_items);
        CAGRA_LAUNCH_CHECK();
    }
    k_reduce4<<<1, kReduceThreads, 0, st>>>(blk, seg->nb, scalars_out, scalars_in);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

cagra_status launch_merge_pr(const cagra_graph *g, const cagra_segments *seg, double damping, int32_t seed,
                             int32_t contrib_type,
                             const float *rank_in, const double *scalars_in, const float *partial, float *rank_out,
                             void *contrib_out, double *scalars_out, void *ws, hipStream_t st) {
    const bool dense = short_ranges(seg);
    auto f = contrib_type == CAGRA_BF16 ? (dense ? launch_merge_pr_t<true, true> : launch_merge_pr_t<true, false>)
                                        : (dense ? launch_merge_pr_t<false, true> : launch_merge_pr_t<false, false>);
    return f(g, seg, damping, seed, rank_in, scalars_in, partial, rank_out, contrib_out, scalars_out, ws, st);
}

// Most blocks whose sums the last one takes. Each block then ends with two
// round trips to memory and an atomic on one address (about 40 ns each, one
// after the other), against a launch of about 3 us plus its gap: 20 iterations
// of a 4,096-vertex graph took 331 us with the reduction launch and 298 us
// without; replayed from a captured graph the two are level up to 64 blocks,
// and with 256 (1,024) blocks of 1,024 vertices the launch is 8% faster.
// A small graph's merge is a chain of round trips to memory: with the vertex
// inputs loaded at its end it takes 10.4 us, loaded first 9.9 us (the pass 287).
constexpr int32_t kOwnSumBlocks = 64;

template <bool BF16OUT>
static cagra_status launch_merge_pr_small_t(const cagra_graph *g, const cagra_segments *seg, double damping,
                                            int32_t seed, const float *rank_in, const double *scalars_in,
                                            const float *partial, float *rank_out, void *contrib_out,
                                            double *scalars_out, void *ws, unsigned long long *ticket,
                                            hipStream_t st) {
    if (cagra_status a_ = ensure_dynamic_lds((const void *)k_merge_pr_small<BF16OUT>)) return a_;
    k_merge_pr_small<BF16OUT><<<seg->nb, kMergeThreads, merge_fused_lds_bytes(seg->B, seg->k, 8), st>>>(
        seg->row_dst_lo, seg->block_ptr, partial, seg->V, seg->k, seg->B, seg->nb, rank_in, g->out_degree, scalars_in,
        damping, seed, rank_out, contrib_out, reinterpret_cast<double *>(ws), ticket, scalars_out);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

// One PageRank iteration. The merge's last block also takes the FP64 sums when
// the graph is small, every block is one work item and the gather runs before
// it and clears the counter (in the workspace's tail, behind the slots);
// otherwise they are a launch of their own. Both give the same bits.
cagra_status launch_pagerank_iter(const cagra_graph *g, const cagra_segments *seg, double damping, int32_t seed,
                                  int32_t contrib_type, const float *rank_in, const void *contrib_in,
                                  const double *scalars_in, float *partial, float *rank_out, void *contrib_out,
                                  double *scalars_out, void *ws, hipStream_t st) {
    cagra_status s;
    if (seg->ntiles == 0 || seg->max_items != seg->nb || seg->nb > kOwnSumBlocks) {
        if ((s = launch_gather(seg, CAGRA_SUM_F32, contrib_type, contrib_in, partial, st)) != CAGRA_OK) return s;
        return launch_merge_pr(g, seg, damping, seed, contrib_type, rank_in, scalars_in, partial, rank_out,
                               contrib_out, scalars_out, ws, st);
    }
    unsigned long long *ticket = reinterpret_cast<unsigned long long *>(
        static_cast<char *>(ws) + ws_blk_bytes(seg->V, seg->nb) + ws_item_bytes(seg) + ws_slot_bytes(seg));
    if ((s = launch_gather_clear(seg, CAGRA_SUM_F32, contrib_type, contrib_in, partial, ticket, st)) != CAGRA_OK)
        return s;
    auto f = contrib_type == CAGRA_BF16 ? launch_merge_pr_small_t<true> : launch_merge_pr_small_t<false>;
    return f(g, seg, damping, seed, rank_in, scalars_in, partial, rank_out, contrib_out, scalars_out, ws, ticket, st);
}

cagra_status launch_merge_lp(const cagra_segments *seg, const int32_t *labels_in, const int32_t *partial,
                             int32_t *labels_out, int32_t *changed_out, void *ws, hipStream_t st) {
    int32_t *blk = reinterpret_cast<int32_t *>(ws);
    const size_t lds = merge_fused_lds_bytes(seg->B, seg->k, 4);
    auto merge = short_ranges(seg) ? k_merge_lp<true> : k_merge_lp<false>;
    if (cagra_status a_ = ensure_dynamic_lds((const void *)merge)) return a_;
    merge<<<seg->nb, kMergeThreads, lds, st>>>(seg->row_dst_lo, seg->block_ptr, partial, seg->V, seg->k, seg->B,
                                               seg->nb, labels_in, labels_out, blk);
    CAGRA_LAUNCH_CHECK();
    k_reduce_i32<<<1, 256, 0, st>>>(blk, seg->nb, changed_out);
    CAGRA_LAUNCH_CHECK();
    return CAGRA_OK;
}

}  // namespace cagra
