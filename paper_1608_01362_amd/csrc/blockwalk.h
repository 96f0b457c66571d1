// Block-range walk shared by the cache-aware merge and the push expand:
// per-subgraph entry ranges of a vertex block loaded into LDS as an exclusive
// prefix, and the forward search that maps a flattened entry to its subgraph.
// Also the exact int64 fixed-point form of FP32 values that the order-free
// sums accumulate.
#pragma once

#include "common.h"
#include "wave.h"

namespace cagra {

constexpr int kMergeThreads = 1024;
constexpr double kFixInv = 1.0 / 72057594037927936.0;  // 2^-56

// In-place exclusive scan of a[0..n) in LDS by the whole 1024-thread block;
// returns the total (all threads). `tmp` holds 16 ints.
__device__ inline int32_t block_excl_scan_lds(int32_t *a, int32_t n, int32_t *tmp) {
    const int per = (n + kMergeThreads - 1) / kMergeThreads;
    const int lo = threadIdx.x * per;
    int32_t sum = 0;
    for (int i = 0; i < per; ++i)
        if (lo + i < n) sum += a[lo + i];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t incl = sum;
    for (int d = 1; d < 64; d <<= 1) {
        int32_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    if (lane == 63) tmp[w] = incl;
    __syncthreads();
    int32_t pre = incl - sum;
    for (int i = 0; i < w; ++i) pre += tmp[i];
    int32_t total = 0;
    for (int i = 0; i < kMergeThreads / 64; ++i) total += tmp[i];
    for (int i = 0; i < per; ++i)
        if (lo + i < n) {
            int32_t x = a[lo + i];
            a[lo + i] = pre;
            pre += x;
        }
    __syncthreads();
    return total;
}

// Loads the block's range bounds per subgraph into LDS: pre = exclusive prefix
// of the range lengths, ofs[s] = (first entry of subgraph s's range) - pre[s],
// so that flattened entry f of subgraph s is entry ofs[s] + f. Returns the
// block's entry count.
__device__ inline int32_t load_block_ranges(const int32_t *__restrict__ block_ptr, int b, int32_t k, int32_t *ofs,
                                            int32_t *pre, int32_t *tmp) {
    for (int s = threadIdx.x; s < k; s += kMergeThreads) {
        int32_t a = block_ptr[(int64_t)b * k + s], e = block_ptr[(int64_t)(b + 1) * k + s];
        ofs[s] = a;
        pre[s] = e - a;
    }
    __syncthreads();
    int32_t P = block_excl_scan_lds(pre, k, tmp);
    if (threadIdx.x == 0) pre[k] = P;
    for (int s = threadIdx.x; s < k; s += kMergeThreads) ofs[s] -= pre[s];
    __syncthreads();
    return P;
}

// Last subgraph s with pre[s] <= f (pre is non-decreasing; empty ranges skipped).
__device__ __forceinline__ int32_t run_of(const int32_t *pre, int32_t k, int32_t f) {
    int32_t lo = 0, hi = k;
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (pre[mid] <= f) lo = mid;
        else hi = mid;
    }
    return lo;
}

// |x| * 2^56 truncated toward zero, from the float's bits: |x| * 2^56 =
// m * 2^(e - 94) for the 24-bit significand m and biased exponent e, i.e. the
// 64-bit word m << 40 shifted right by 134 - e. The high dword of m << 40 is
// the float's bits shifted left by 8 with the leading one set; shifts of 64
// or more (|x| < 2^-56, zeros, denormals) give 0. Exact for |x| < 64.
__device__ __forceinline__ uint64_t fix56_magnitude(uint32_t u) {
    const uint32_t amt = 134u - ((u >> 23) & 0xffu);
    const uint32_t hi = amt < 64u ? (u << 8) | 0x80000000u : 0u;
    return ((uint64_t)hi << 32) >> (amt & 63u);
}

// trunc(x * 2^56) as a two's-complement int64: sums of these are exact, so
// they do not depend on the order of the additions (error below 2^-56 per term).
__device__ __forceinline__ unsigned long long fix56(float x) {
    const uint32_t u = __float_as_uint(x);
    const uint64_t m = fix56_magnitude(u);
    return (u >> 31) ? (unsigned long long)(-(int64_t)m) : (unsigned long long)m;
}

// The same with one uniform branch for the wave: where every (active) lane's x
// is in [0, 64), which contributions and ranks are, the two dwords come from two
// conversions -- x * 2^24 and its fraction times 2^32, both exact -- in 5
// instructions in place of the 16 of the general form.
__device__ __forceinline__ unsigned long long fix56_wave(float x) {
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(__float_as_uint(x) >= 0x42800000u) != 0, 0)) return fix56(x);
    const float y = x * 16777216.0f;
    const uint32_t hi = (uint32_t)y, lo = (uint32_t)(__builtin_amdgcn_fractf(y) * 4294967296.0f);
    return ((unsigned long long)hi << 32) | lo;
}

// Walk of a wave over its block's ranges in windows of 64 consecutive flattened
// entries (ofs, pre: load_block_ranges). The wave steps over the range starts inside
// a window together, each lane keeping the offset of the last range that starts at
// or before its entry. The offsets and ends of the next 64 ranges are held one per
// lane, so a range start costs two lane reads, a compare and a select, and a window
// without one costs nothing. DENSE: a window with more than kFew starts marks them
// as bits of the window instead, and every entry takes the offset of the range that
// its count of bits names.
//
// Merge of R-MAT graphs, DENSE = false (a search per lane before): 25 -> 19 us
// with ranges of 1,052 entries in the mean, 47 -> 44 with 412. After clustering,
// where most blocks' ranges are much shorter than the mean, with DENSE: 310 -> 229
// us (mean 76; 255 without) and 464 -> 373 (19; 534 without) of 2^24 vertices,
// 232 -> 156 (8.4; 265 without) of 2^22, and 633 -> 534 of 2^25 (716 without).
template <bool DENSE>
struct RangeWalk {
    static constexpr int kFew = 6;  // 4 to 24: within 5%
    const int32_t *ofs, *pre;
    int32_t k, s0, j;    // ranges; range of lane 0; the current range's lane
    int32_t o, nxt;      // the current range's offset and end (uniform)
    int32_t vo, vn;      // those of range s0 + lane
    int32_t vp;          // its start (DENSE)

    __device__ __forceinline__ void fetch() {
        const int32_t s = min(s0 + (int32_t)(threadIdx.x & 63), k - 1);
        vo = ofs[s];
        vn = pre[s + 1];
        if constexpr (DENSE) vp = pre[s];
        asm volatile("" : "+v"(vo), "+v"(vn));  // here now: no wait for LDS in the loop's steps
    }
    __device__ __forceinline__ void take() {
        o = __builtin_amdgcn_readlane(vo, j);
        nxt = __builtin_amdgcn_readlane(vn, j);
    }
    // s: the range of the first entry
    __device__ __forceinline__ RangeWalk(const int32_t *ofs_, const int32_t *pre_, int32_t k_, int32_t s)
        : ofs(ofs_), pre(pre_), k(k_), s0(s), j(0) {
        fetch();
        take();
    }
    // Entry index of flattened entry f (lane 0: the window's first) of a window that
    // ends at wend < pre[k].
    __device__ __forceinline__ int32_t index(int32_t wend, int32_t f) {
        if constexpr (DENSE) return index_dense(wend, f);
        int32_t ov = o;
        while (nxt <= wend) {
            if (++j == kWave) {
                s0 += kWave;
                j = 0;
                fetch();
            }
            const int32_t at = nxt;
            take();
            ov = f >= at ? o : ov;
        }
        return ov + f;
    }
    __device__ __forceinline__ int32_t index_dense(int32_t wend, int32_t f) {
        int32_t ov = o;
        while (nxt <= wend) {
            if (j == kWave - 1) {
                s0 += kWave;
                j = -1;
                fetch();
            }
            // held ranges after the current one that start in the window (starts ascend;
            // lanes past the last range repeat it)
            int32_t n = (int32_t)__popcll(__builtin_amdgcn_ballot_w64(vp <= wend)) - 1 - j;
            if (n <= kFew) {
                for (; n > 0; --n) {
                    ++j;
                    const int32_t at = __builtin_amdgcn_readlane(vp, j);
                    o = __builtin_amdgcn_readlane(vo, j);
                    ov = f >= at ? o : ov;
                }
                nxt = __builtin_amdgcn_readlane(vn, j);
            } else {
                // the non-empty ones among them start at entries of their own
                const int32_t lane = __lane_id();
                const bool in = lane > j && vp <= wend && vn > vp;
                const uint32_t at = (uint32_t)(vp - __builtin_amdgcn_readfirstlane(f)) & 63u;
                // bit i: one starts at lane i's entry
                const uint64_t starts = wave_or64(in ? 1ull << at : 0ull);
                // lane r receives the offset of the r-th (the other lanes fill the lanes after)
                const uint64_t from = __builtin_amdgcn_ballot_w64(in);
                const int32_t rank = lanes_below(from);
                const int32_t to = in ? rank : (int32_t)__popcll(from) + lane - rank;
                const int32_t listed = __builtin_amdgcn_ds_permute(to << 2, vo);
                const int32_t r = lanes_below(starts >> 1) + (int32_t)(starts & 1ull);  // starts up to this entry
                const int32_t its = __builtin_amdgcn_ds_bpermute((r - 1) << 2, listed);
                ov = r > 0 ? its : ov;
                j += n;
                take();
            }
        }
        return ov + f;
    }
};
// Rule for DENSE: mean entries per (subgraph, block) range below one and a half
// windows. Merge with and without DENSE, us: mean 48: 389 and 396, 76 (clustered):
// 229 and 255, 103: 70 and 67, 192: 305 and 303. It is the rule of k_merge_pr,
// k_merge_lp and the push expand. The one-launch merge of small graphs, the merge of
// many graphs and the sums of the vertex features take the starts in turn (DENSE
// false) at any mean: at means of 2.7 to 1,376 none was slower than with a search per
// lane (many clustered graphs, mean 4.8: 160 -> 108 us; features, mean 67: 660 -> 468).
static inline bool short_ranges(const cagra_segments *seg) {
    return seg->Q < (int64_t)(kWave + kWave / 2) * seg->k * seg->nb;
}

constexpr int kUnroll = 8;

// Block of merge work item i: last b with items[b] <= i (items ascending).
__device__ __forceinline__ int32_t block_of_item(const int32_t *__restrict__ items, int32_t nb, int32_t i) {
    int32_t lo = 0, hi = nb;
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (items[mid] <= i) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Block b of work item it, and the item's index j among the S items of b.
// Every block has at least one item, so a total of nb items means one item per
// block and item it is block it: no search (a chain of dependent global loads)
// before the block's work starts.
struct ItemPlace {
    int32_t b, j, S;
};
__device__ __forceinline__ ItemPlace place_item(const int32_t *__restrict__ items, int32_t nb, int32_t total,
                                                int32_t it) {
    if (total == nb) return {it, 0, 1};
    const int32_t b = block_of_item(items, nb, it);
    return {b, it - items[b], items[b + 1] - items[b]};
}

// Groups of g consecutive work items share an XCD (workgroup id mod 8), and
// the groups cycle over the XCDs: neighbouring blocks still meet in one L2,
// while the heavy blocks at the front (high in-degree destinations after
// clustering) spread over all XCDs. Bijective on [0, n): ids past the last
// whole round of 8 g keep their place.
__device__ __forceinline__ int32_t xcd_group_map(int32_t id, int32_t n, int32_t g) {
    const int32_t round = 8 * g;
    if (id >= n / round * round) return id;
    const int32_t x = id & 7, q = id >> 3;
    return (q / g) * round + x * g + (q % g);
}

}  // namespace cagra
