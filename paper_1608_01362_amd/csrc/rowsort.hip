// Rows of a relabelled CSC: every row's sources are mapped to their new ids and
// sorted ascending.
//
// The rows are known, so this is a sort inside each row, not one of all edges.
// A workgroup takes a tile of whole rows (up to 8,192 edges), and one pass over
// it in LDS puts it in order:
//   1. Each edge gets a slot of its row, row start + floor(length * G(id)),
//      where G is a non-decreasing map of new ids to [0, 1) close to the share
//      of edges whose source lies below the id (a table of the new out-degrees'
//      prefix sums with 64 cells per power of two). In a row of n edges the
//      slots are then spread over the n places almost evenly.
//   2. LDS counts per slot, a scan, and every edge is placed among its slot's
//      few edges (mean two) by comparing with them, equal ids (repeated edges)
//      by their places there, so the result is unique however the counting
//      atomics fall.
// G only steers the work. A slot of more than kMaxSlot edges is spread over its
// own places, linearly between its smallest and largest id (rows of neighbouring
// ids, communities: one or two such passes), and what is still crowded after
// kRefine passes is put in order by a bitonic sort over (slot, id).
// Rows of more than 4,096 edges are cut into pieces of 8,192, each sorted the
// same way, and the pieces are merged pairwise, level by level, in units of
// 4,096 output edges (merge path), between the output and a buffer of E ids; the
// number of levels decides which of the two a row's pieces start in.
//
// Bytes: 4 E + 4 E (random reads of inv) + 4 E, against the 16 E of each of six
// or seven passes of the edge-key sort it replaces. Clustering R-MAT 24 / ef 24:
// 20.5 -> 9.2 ms (light tiles 5.4, pieces 1.9, merges 0.4), R-MAT 25 / ef 32
// 59.5 -> 25.3 ms. What bounds it is the lookup of the new ids: one random
// 4-byte read per edge through L2 and the Infinity Cache, about 65 G/s. Rows of 300
// neighbouring ids (60 M edges) take 1.67 against 1.81 ms, a star of 3 M edges 0.30
// against 0.32 ms (nine merge levels of runs in order). Dearer than the edge-key sort
// are rows of 10^5 and more sources in no order with little beside them: each merge
// level is a chain of some 20 us (five rows of 600,000 edges: 0.52 against 0.32 ms,
// fifty of 80,000: 0.38 against 0.35).
#include "rowsort.h"

#include <type_traits>

#include "segdirect.h"
#include "wave.h"

namespace cagra {

constexpr int kRsThreads = 512;
constexpr int kRsItems = 16;
constexpr int kRsCap = kRsThreads * kRsItems;  // edges of a tile at most, and of a piece
constexpr int kRsTile = kRsCap / 2;            // light rows that start in kRsTile output edges share a tile
constexpr int kLightMax = kRsCap - kRsTile;    // longest light row
constexpr int kMaxSlot = 96;                   // edges per slot beyond which a slot is spread again
constexpr int kRefine = 3;                     // times at most, before the tile is sorted
constexpr int kUnit = 4096;                    // output edges of a merge unit
constexpr int kShortItems = 10;                // items per thread for tiles of at most 5,120 edges
constexpr int kCellBits = 6;                   // cells of G per power of two
constexpr int kCells = (32 - kCellBits) << kCellBits;
static_assert(kLightMax >= kRsTile, "a longer row is the last one of its tile");

// ---- G: non-decreasing, 32-bit fraction

struct Cell {
    uint32_t c;     // table cell
    uint32_t frac;  // position inside it, 32-bit fraction
};
__device__ __forceinline__ Cell cell_of(uint32_t id) {
    const uint32_t x = id + (1u << kCellBits);
    const uint32_t sh = 31u - (uint32_t)kCellBits - (uint32_t)__clz((int)x);
    Cell r;
    r.c = (sh << kCellBits) + (x >> sh) - (1u << kCellBits);
    r.frac = (x << (31u - sh)) << 1;  // the sh low bits, at the top
    return r;
}
__device__ __forceinline__ uint32_t lowest_id(uint32_t c) {
    const uint32_t sh = c >> kCellBits, m = (c & ((1u << kCellBits) - 1u)) + (1u << kCellBits);
    const uint64_t x = (uint64_t)m << sh;
    return x > 0x7fffffffull ? 0x7fffffffu : (uint32_t)x - (1u << kCellBits);
}
__device__ __forceinline__ uint32_t fraction(const uint32_t *tab, uint32_t id) {
    const Cell r = cell_of(id);
    const uint32_t a = tab[r.c], b = tab[r.c + 1];
    return a + __umulhi(b - a, r.frac);
}

struct HeavyCount {
    unsigned long long rows_units;  // heavy rows << 32 | merge units
    int32_t levels;                 // most merge levels of a row
    int32_t crowded[2];             // light tiles and pieces left to the second kernel
    int32_t lengthy;                // light tiles of more than kShortItems edges per thread
    __device__ __forceinline__ int32_t units() const { return (int32_t)(uint32_t)rows_units; }
};

// tab[c] = share of the out-degrees below the cell's lowest id, made
// non-decreasing whatever the sums hold; clears the heavy counts. One workgroup.
__global__ __launch_bounds__(1024) void k_rs_table(const int32_t *__restrict__ cum,
                                                   const int32_t *__restrict__ outdeg, int32_t V,
                                                   uint32_t *__restrict__ tab, HeavyCount *__restrict__ hc) {
    if (threadIdx.x == 0) *hc = HeavyCount{0ull, 0, {0, 0}, 0};
    constexpr int kPer = (kCells + 1 + 1023) / 1024;
    __shared__ uint32_t wmax[16];
    const double total = (double)cum[V - 1] + (double)outdeg[V - 1];
    const int lo = threadIdx.x * kPer, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t v[kPer], m = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        v[i] = 0;
        if (lo + i <= kCells) {
            const uint32_t id = lo + i < kCells ? lowest_id((uint32_t)(lo + i)) : 0x7fffffffu;
            const double share = id < (uint32_t)V && total > 0.0 ? (double)cum[id] / total : 1.0;
            v[i] = share >= 1.0 ? ~0u : share > 0.0 ? (uint32_t)(share * 4294967295.0) : 0u;
        }
        m = max(m, v[i]);
        v[i] = m;
    }
    uint32_t incl = m;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl = max(incl, o);
    }
    if (lane == 63) wmax[w] = incl;
    uint32_t before = __shfl_up(incl, 1, 64);
    if (lane == 0) before = 0;
    __syncthreads();
    for (int i = 0; i < w; ++i) before = max(before, wmax[i]);
#pragma unroll
    for (int i = 0; i < kPer; ++i)
        if (lo + i <= kCells) tab[lo + i] = max(before, v[i]);
}

// ---- work units

static __device__ __forceinline__ int32_t merge_levels(int32_t len) {
    int32_t l = 0;
    while (((int64_t)kRsCap << l) < len) ++l;
    return l;
}

// The list of heavy rows with their units (in any order: no result depends on it).
__global__ __launch_bounds__(256) void k_rs_units(const int32_t *__restrict__ noff, int32_t V,
                                                  HeavyCount *__restrict__ hc, int32_t *__restrict__ hrow,
                                                  int32_t *__restrict__ hunit, int32_t *__restrict__ unit_row) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int lane = __lane_id();
    const int32_t len = r < V ? noff[r + 1] - noff[r] : 0;
    // heavy rows of the wave: one atomic gives them consecutive list places and units
    const bool heavy = len > kLightMax;
    const uint64_t hm = __builtin_amdgcn_ballot_w64(heavy);
    if (!hm) return;  // uniform
    const int32_t units = heavy ? (len + kUnit - 1) / kUnit : 0;
    const int32_t incl = wave_incl_sum(units), total = __builtin_amdgcn_readlane(incl, 63);
    int32_t levels = heavy ? merge_levels(len) : 0;
    for (int d = 32; d >= 1; d >>= 1) levels = max(levels, __shfl_xor(levels, d, 64));
    unsigned long long at = 0;
    if (lane == 0) {
        at = atomicAdd(&hc->rows_units, ((unsigned long long)__popcll(hm) << 32) | (unsigned long long)total);
        if (*(volatile int32_t *)&hc->levels < levels) atomicMax(&hc->levels, levels);
    }
    const int32_t h0 = __builtin_amdgcn_readfirstlane((int32_t)(at >> 32));
    const int32_t u0 = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)at);
    const int32_t h = h0 + (int32_t)__popcll(hm & lanemask_lt()), first_unit = u0 + incl - units;
    if (heavy) {
        hrow[h] = (int32_t)r;
        hunit[h] = first_unit;
    }
    for (uint64_t m = hm; m; m &= m - 1) {
        const int l = (int)__builtin_ctzll(m);
        const int32_t n = __builtin_amdgcn_readlane(units, l), u = __builtin_amdgcn_readlane(first_unit, l);
        const int32_t row = __builtin_amdgcn_readlane(h, l);
        for (int32_t i = lane; i < n; i += kWave) unit_row[u + i] = row;
    }
}

// ---- sorting a tile

// ITEMS: edges per thread, at most. Most light tiles hold about kRsTile edges: with
// kShortItems three workgroups fit a CU in place of two (registers), and more
// lookups of new ids are in flight (R-MAT 24 / ef 24: 6.06 -> 5.43 ms; at four
// workgroups the registers spill, 6.48 ms).
template <int ITEMS>
struct SortLds {
    static constexpr int kItems = ITEMS, kCap = ITEMS * kRsThreads;
    uint32_t key[kCap];                         // row tables before, ids after
    uint32_t cnt[kCap / 2 + 4];                 // two 16-bit slot counts (then starts) a word, and the end
    uint32_t tab[kCells + 1];
    unsigned long long starts[kRsCap / kWave];  // row starts of the tile, one bit an edge
    int32_t before[kRsCap / kWave];             // row starts before each 64 edges
    uint32_t wsum[kRsThreads / kWave];
    int32_t lo, hi, most;
};

__device__ __forceinline__ uint32_t get16(const uint32_t *a, uint32_t i) {
    return reinterpret_cast<const uint16_t *>(a)[i];
}

// Counts the tile's edges per slot (slots below the cap) and scans the counts:
// afterwards lo[j] = first place of item j's slot | its edges << 16, and
// slot[j] holds, above the slot, the edge's turn among those of its slot (as
// the atomics fell). Returns whether some slot holds more than kMaxSlot edges.
template <int ITEMS>
__device__ __forceinline__ bool count_slots(SortLds<ITEMS> &L, uint32_t (&slot)[ITEMS], uint32_t (&lo)[ITEMS],
                                            int32_t n) {
    constexpr int kCap = SortLds<ITEMS>::kCap;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    __syncthreads();  // whatever was in the counts is read
#pragma unroll
    for (int i = 0; i < kCap / 2 / kRsThreads; ++i) L.cnt[i * kRsThreads + tid] = 0u;
    if (tid == 0) L.most = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint32_t s = slot[j], sh = (s & 1u) * 16u;
        uint32_t had = 0;
        if (j * kRsThreads + tid < n) had = atomicAdd(&L.cnt[s >> 1], 1u << sh);
        slot[j] = s | ((had >> sh) << 16);
    }
    __syncthreads();
    // exclusive scan, ITEMS consecutive slots per thread
    uint32_t c[ITEMS / 2], sum = 0, most = 0;
#pragma unroll
    for (int i = 0; i < ITEMS / 2; ++i) {
        c[i] = L.cnt[tid * (ITEMS / 2) + i];
        sum += (c[i] & 0xffffu) + (c[i] >> 16);
        most = max(most, max(c[i] & 0xffffu, c[i] >> 16));
    }
    if (__builtin_amdgcn_ballot_w64(most > (uint32_t)kMaxSlot) && lane == 0) L.most = 1;
    uint32_t incl = sum;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    if (lane == 63) L.wsum[w] = incl;
    __syncthreads();
    uint32_t at = incl - sum;
    for (int x = 0; x < w; ++x) at += L.wsum[x];
#pragma unroll
    for (int i = 0; i < ITEMS / 2; ++i) {
        const uint32_t a = at, b = at + (c[i] & 0xffffu);
        at = b + (c[i] >> 16);
        L.cnt[tid * (ITEMS / 2) + i] = a | (b << 16);
    }
    if (tid == 0) L.cnt[kCap / 2] = (uint32_t)n;  // the end, read for the last slot
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {  // items past the tile have a slot too; unused
        const uint32_t s = slot[j] & 0xffffu, a = get16(L.cnt, s);
        lo[j] = a | ((get16(L.cnt, s + 1) - a) << 16);
    }
    return L.most != 0;  // uniform
}

// Spreads the slots of more than kMaxSlot edges over their places by linear
// interpolation between their smallest and largest id; the other slots become
// their first place. The order of slots stays the order of ids.
template <int ITEMS>
__device__ __forceinline__ void refine_slots(SortLds<ITEMS> &L, const uint32_t (&key)[ITEMS], uint32_t (&slot)[ITEMS],
                                             const uint32_t (&lo)[ITEMS], int32_t n) {
    constexpr int kCap = SortLds<ITEMS>::kCap;
    const int tid = threadIdx.x;
    uint32_t least[ITEMS];
    auto big = [&](int j) { return j * kRsThreads + tid < n && (lo[j] >> 16) > (uint32_t)kMaxSlot; };
    for (int i = tid; i < kCap; i += kRsThreads) L.key[i] = ~0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (big(j)) atomicMin(&L.key[lo[j] & 0xffffu], key[j]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) least[j] = big(j) ? L.key[lo[j] & 0xffffu] : 0u;
    __syncthreads();
    for (int i = tid; i < kCap; i += kRsThreads) L.key[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (big(j)) atomicMax(&L.key[lo[j] & 0xffffu], key[j]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        // rounding keeps the order; the last place takes what rounds up past it
        const uint32_t a = lo[j] & 0xffffu, m = lo[j] >> 16, span = L.key[a] - least[j];
        const uint32_t at = (uint32_t)((float)(key[j] - least[j]) * ((float)m / ((float)span + 1.0f)));
        slot[j] = a + (big(j) ? (at < m ? at : m - 1) : 0u);
    }
    __syncthreads();
}

// Orders the n edges held in (key, slot) across the workgroup (item j of thread
// t valid when j * kRsThreads + t < n) and writes them to out[0 .. n). Slots
// below the cap. With ANY = false a crowded tile is not written: false comes back.
template <bool ANY, int ITEMS>
__device__ __forceinline__ bool sort_tile(SortLds<ITEMS> &L, const uint32_t (&key)[ITEMS], uint32_t (&slot)[ITEMS],
                                          int32_t n, int32_t *__restrict__ out) {
    [[maybe_unused]] constexpr int kCap = SortLds<ITEMS>::kCap;
    static_assert(!ANY || (kCap & (kCap - 1)) == 0, "the bitonic sort's length");
    const int tid = threadIdx.x;
    uint32_t lo[ITEMS];
    bool crowded = count_slots(L, slot, lo, n);
    if constexpr (ANY) {
#pragma unroll 1
        for (int pass = 0; crowded && pass < kRefine; ++pass) {  // uniform
            refine_slots(L, key, slot, lo, n);
            crowded = count_slots(L, slot, lo, n);
        }
    } else if (crowded) {
        return false;
    }
    if (!ANY || !crowded) {
        static_assert(kMaxSlot < 128, "a slot's edges and an edge's turn in seven bits each");
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint32_t turn = slot[j] >> 16;
            if (j * kRsThreads + tid < n) L.key[(lo[j] & 0xffffu) + turn] = key[j];
            lo[j] |= turn << 23;  // one register for all three: a register more each would spill
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint32_t a = lo[j] & 0xffffu, m = j * kRsThreads + tid < n ? lo[j] >> 16 & 127u : 0u;
            const uint32_t turn = lo[j] >> 23;
            uint32_t less = 0;  // smaller ids, and equal ones placed before this one
            for (uint32_t q = 0; m > 1 && q < m; ++q) less += L.key[a + q] < key[j] + (q < turn ? 1u : 0u) ? 1u : 0u;
            lo[j] = a + less;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if (j * kRsThreads + tid < n) L.key[lo[j]] = key[j];
    } else {
        uint16_t *sl = reinterpret_cast<uint16_t *>(L.cnt);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int i = j * kRsThreads + tid;
            L.key[i] = i < n ? key[j] : ~0u;
            sl[i] = i < n ? (uint16_t)(slot[j] & 0xffffu) : (uint16_t)0xffffu;
        }
        for (int k = 2; k <= kCap; k <<= 1)
            for (int d = k >> 1; d >= 1; d >>= 1) {
                __syncthreads();
                for (int p = tid; p < kCap / 2; p += kRsThreads) {
                    const int a = 2 * p - (p & (d - 1)), b = a + d;
                    const uint32_t sa = sl[a], sb = sl[b], ka = L.key[a], kb = L.key[b];
                    const bool after = sa != sb ? sa > sb : ka > kb;
                    if (after == ((a & k) == 0) && (sa != sb || ka != kb)) {
                        L.key[a] = kb;
                        L.key[b] = ka;
                        sl[a] = (uint16_t)sb;
                        sl[b] = (uint16_t)sa;
                    }
                }
            }
    }
    __syncthreads();
    for (int i = tid; i < n; i += kRsThreads) out[i] = (int32_t)L.key[i];
    return true;
}

// Tile t: the light rows that start in output edges [t * kRsTile, (t + 1) * kRsTile).
// Returns 0, or why the tile was not written: kCrowded, or kLengthy (more edges
// than the workgroup takes).
enum { kSorted, kCrowded, kLengthy };
template <bool ANY, int ITEMS>
__device__ __forceinline__ int sort_light(SortLds<ITEMS> &L, const int32_t *__restrict__ in_offsets,
                                           const int32_t *__restrict__ in_sources, const int32_t *__restrict__ perm,
                                           const int32_t *__restrict__ inv, const RowList &list, int64_t E, int32_t t,
                                           int32_t *__restrict__ out) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int32_t last = list.first[(E + kRsTile - 1) / kRsTile];  // last list index
    const int64_t base = (int64_t)t * kRsTile;
    // the rows that start in the tile: list indices [i0, i1)
    const int32_t c0 = list.first[t], c1 = list.first[t + 1];
    const int64_t end = base + kRsTile;
    const int32_t i0 = c0 + ((int64_t)list.start[c0] < base ? 1 : 0);
    const int32_t i1 = c1 + ((int64_t)list.start[c1] < end ? 1 : 0);
    // row i ends where the next one starts
    auto row_end = [&](int32_t i) { return i + 1 <= last ? (int64_t)list.start[i + 1] : E; };
    for (int i = tid; i < kRsCap / kWave; i += kRsThreads) L.starts[i] = 0ull;
    if (tid == 0) {
        L.lo = kRsCap;
        L.hi = 0;
    }
    __syncthreads();
    for (int32_t i = i0 + tid; i < i1; i += kRsThreads) {
        const int32_t s = list.start[i], a = (int32_t)(s - base), len = (int32_t)(row_end(i) - s);
        if (len <= kLightMax) {
            atomicOr(&L.starts[a >> 6], 1ull << (a & 63));
            atomicMin(&L.lo, a);
            atomicMax(&L.hi, a + len);
        }
    }
    __syncthreads();
    const int32_t e0 = L.lo, e1 = L.hi;
    if (e1 == 0) return kSorted;  // uniform: no light row starts here
    if (ITEMS < kRsItems && e1 - e0 > SortLds<ITEMS>::kCap) return kLengthy;  // uniform
    // the light rows of a tile are consecutive: only the last row that starts in it can be heavy
    if (tid < kWave) {
        constexpr int kPer = kRsCap / kWave / kWave;  // 64-edge words per lane
        int32_t c[kPer], sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            c[i] = (int32_t)__popcll(L.starts[lane * kPer + i]);
            sum += c[i];
        }
        int32_t incl = sum;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        int32_t at = incl - sum;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            L.before[lane * kPer + i] = at;
            at += c[i];
        }
        // row tables: old position of the tile's edge e in row o = delta[o] + e; first edge of row o, from e0
        if (lane == 63) reinterpret_cast<uint16_t *>(L.cnt)[at] = (uint16_t)(e1 - e0);
    }
    __syncthreads();
    int32_t *delta = reinterpret_cast<int32_t *>(L.key);
    uint16_t *begin = reinterpret_cast<uint16_t *>(L.cnt);
    for (int32_t i = i0 + tid; i < i1; i += kRsThreads) {
        const int32_t s = list.start[i], a = (int32_t)(s - base), len = (int32_t)(row_end(i) - s);
        if (len <= kLightMax) {
            const int32_t o = L.before[a >> 6] + (int32_t)__popcll(L.starts[a >> 6] & ((1ull << (a & 63)) - 1ull));
            delta[o] = in_offsets[perm[list.row[i]]] - a;
            begin[o] = (uint16_t)(a - e0);
        }
    }
    __syncthreads();
    const int32_t n = e1 - e0;
    uint32_t key[ITEMS], slot[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        // items past the tile read its first edge, unused
        const int32_t e = e0 + (j * kRsThreads + tid < n ? j * kRsThreads + tid : 0);
        const int32_t o = L.before[e >> 6] + (int32_t)__popcll(L.starts[e >> 6] & (~0ull >> (63 - (e & 63)))) - 1;
        slot[j] = (uint32_t)begin[o] | ((uint32_t)(begin[o + 1] - begin[o]) << 16);
        key[j] = (uint32_t)in_sources[(int64_t)delta[o] + e];
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) key[j] = (uint32_t)inv[key[j]];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        slot[j] = (slot[j] & 0xffffu) + __umulhi(slot[j] >> 16, fraction(L.tab, key[j]));
    return sort_tile<ANY>(L, key, slot, n, out + base + e0) ? kSorted : kCrowded;
}

template <int ITEMS>
__device__ __forceinline__ void load_table(SortLds<ITEMS> &L, const uint32_t *__restrict__ tab) {
    for (int i = threadIdx.x; i <= kCells; i += kRsThreads) L.tab[i] = tab[i];
}

// One tile per workgroup; the crowded ones are listed for k_rs_light_crowded, whose
// further passes need more registers (two workgroups per CU; at one, a graph of 60 M
// edges between neighbours took 2.11 ms, 1.67 now), and the lengthy ones, whose last
// rows run far past kRsTile, for k_rs_light_lengthy.
__global__ __launch_bounds__(kRsThreads, 6) void k_rs_light(
    const int32_t *__restrict__ in_offsets, const int32_t *__restrict__ in_sources, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ inv, RowList list, int64_t E, const uint32_t *__restrict__ tab, int32_t tiles,
    HeavyCount *__restrict__ hc, int32_t *__restrict__ crowded, int32_t *__restrict__ lengthy,
    int32_t *__restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    auto &L = *reinterpret_cast<SortLds<kShortItems> *>(smem);
    load_table(L, tab);  // ordered by the barriers before its first use
    const int32_t t = xcd_remap(blockIdx.x, tiles);
    const int r = sort_light<false>(L, in_offsets, in_sources, perm, inv, list, E, t, out);
    if (threadIdx.x == 0) {
        if (r == kCrowded) crowded[atomicAdd(&hc->crowded[0], 1)] = t;
        if (r == kLengthy) lengthy[atomicAdd(&hc->lengthy, 1)] = t;
    }
}

__global__ __launch_bounds__(kRsThreads, 4) void k_rs_light_lengthy(
    const int32_t *__restrict__ in_offsets, const int32_t *__restrict__ in_sources, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ inv, RowList list, int64_t E, const uint32_t *__restrict__ tab,
    HeavyCount *__restrict__ hc, int32_t *__restrict__ crowded, const int32_t *__restrict__ lengthy,
    int32_t *__restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    auto &L = *reinterpret_cast<SortLds<kRsItems> *>(smem);
    const int32_t n = hc->lengthy;
    if ((int32_t)blockIdx.x >= n) return;
    load_table(L, tab);
    for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int32_t t = lengthy[i];
        if (sort_light<false>(L, in_offsets, in_sources, perm, inv, list, E, t, out) == kCrowded && threadIdx.x == 0)
            crowded[atomicAdd(&hc->crowded[0], 1)] = t;
        __syncthreads();  // the next tile reuses the LDS
    }
}

__global__ __launch_bounds__(kRsThreads, 4) void k_rs_light_crowded(
    const int32_t *__restrict__ in_offsets, const int32_t *__restrict__ in_sources, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ inv, RowList list, int64_t E, const uint32_t *__restrict__ tab,
    const HeavyCount *__restrict__ hc, const int32_t *__restrict__ crowded,
    int32_t *__restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    auto &L = *reinterpret_cast<SortLds<kRsItems> *>(smem);
    const int32_t n = hc->crowded[0];
    if ((int32_t)blockIdx.x >= n) return;
    load_table(L, tab);
    for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
        sort_light<true>(L, in_offsets, in_sources, perm, inv, list, E, crowded[i], out);
        __syncthreads();  // the next tile reuses the LDS
    }
}

// The piece that starts at merge unit u (every other unit of a heavy row).
template <bool ANY>
__device__ __forceinline__ bool sort_piece(SortLds<kRsItems> &L, const int32_t *__restrict__ in_offsets,
                                           const int32_t *__restrict__ in_sources, const int32_t *__restrict__ perm,
                                           const int32_t *__restrict__ inv, const int32_t *__restrict__ noff,
                                           int32_t row, int32_t i, int32_t *__restrict__ out,
                                           int32_t *__restrict__ tmp) {
    const int tid = threadIdx.x;
    const int32_t len = noff[row + 1] - noff[row], p0 = i * kUnit;
    const int32_t n = len - p0 < kRsCap ? len - p0 : kRsCap;
    const int32_t *src = in_sources + (int64_t)in_offsets[perm[row]] + p0;
    uint32_t key[kRsItems], slot[kRsItems];
#pragma unroll
    for (int j = 0; j < kRsItems; ++j) {
        const int32_t e = j * kRsThreads + tid;
        key[j] = (uint32_t)src[e < n ? e : 0];
    }
#pragma unroll
    for (int j = 0; j < kRsItems; ++j) key[j] = (uint32_t)inv[key[j]];
#pragma unroll
    for (int j = 0; j < kRsItems; ++j) {
        const uint32_t f = fraction(L.tab, key[j]);
        slot[j] = ANY ? f >> 1 : __umulhi((uint32_t)n, f);
    }
    if constexpr (ANY) {
        // the piece's own span of G over its places: most crowded pieces hold neighbouring
        // ids (a row's edges come in the old order, which most vertices keep)
        int32_t least = 0x7fffffff, most = 0;
#pragma unroll
        for (int j = 0; j < kRsItems; ++j) {  // items past the piece hold its first edge again
            least = min(least, (int32_t)slot[j]);
            most = max(most, (int32_t)slot[j]);
        }
        least = __builtin_amdgcn_readlane(wave_incl_max(0x7fffffff - least), 63);
        most = __builtin_amdgcn_readlane(wave_incl_max(most), 63);
        if ((tid & 63) == 0) {
            L.wsum[tid >> 6] = (uint32_t)least;
            L.before[tid >> 6] = most;
        }
        __syncthreads();
        for (int x = 0; x < kRsThreads / kWave; ++x) {
            least = max(least, (int32_t)L.wsum[x]);
            most = max(most, L.before[x]);
        }
        least = 0x7fffffff - least;
        const float scale = (float)n / ((float)(most - least) + 1.0f);
#pragma unroll
        for (int j = 0; j < kRsItems; ++j) {  // rounding keeps the order
            const uint32_t at = (uint32_t)((float)((int32_t)slot[j] - least) * scale);
            slot[j] = min(at, (uint32_t)(n - 1));
        }
    }
    int32_t *to = merge_levels(len) & 1 ? tmp : out;
    return sort_tile<ANY>(L, key, slot, n, to + (int64_t)noff[row] + p0);
}

__global__ __launch_bounds__(kRsThreads, 4) void k_rs_pieces(
    const int32_t *__restrict__ in_offsets, const int32_t *__restrict__ in_sources, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ inv, const int32_t *__restrict__ noff, HeavyCount *__restrict__ hc,
    const int32_t *__restrict__ hrow, const int32_t *__restrict__ hunit, const int32_t *__restrict__ unit_row,
    const uint32_t *__restrict__ tab, int32_t *__restrict__ crowded, int32_t *__restrict__ out,
    int32_t *__restrict__ tmp) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    auto &L = *reinterpret_cast<SortLds<kRsItems> *>(smem);
    const int32_t units = hc->units();
    if ((int32_t)blockIdx.x >= units) return;
    load_table(L, tab);
    __syncthreads();
    for (int32_t u = blockIdx.x; u < units; u += gridDim.x) {
        const int32_t h = unit_row[u], i = u - hunit[h];
        if (i & 1) continue;  // uniform: a piece is two units
        if (!sort_piece<false>(L, in_offsets, in_sources, perm, inv, noff, hrow[h], i, out, tmp) && threadIdx.x == 0)
            crowded[atomicAdd(&hc->crowded[1], 1)] = u;
        __syncthreads();  // the next piece reuses the LDS
    }
}

__global__ __launch_bounds__(kRsThreads, 2) void k_rs_pieces_crowded(
    const int32_t *__restrict__ in_offsets, const int32_t *__restrict__ in_sources, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ inv, const int32_t *__restrict__ noff, const HeavyCount *__restrict__ hc,
    const int32_t *__restrict__ hrow, const int32_t *__restrict__ hunit, const int32_t *__restrict__ unit_row,
    const uint32_t *__restrict__ tab, const int32_t *__restrict__ crowded, int32_t *__restrict__ out,
    int32_t *__restrict__ tmp) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    auto &L = *reinterpret_cast<SortLds<kRsItems> *>(smem);
    const int32_t n = hc->crowded[1];
    if ((int32_t)blockIdx.x >= n) return;
    load_table(L, tab);
    __syncthreads();
    for (int32_t c = blockIdx.x; c < n; c += gridDim.x) {
        const int32_t u = crowded[c], h = unit_row[u];
        sort_piece<true>(L, in_offsets, in_sources, perm, inv, noff, hrow[h], u - hunit[h], out, tmp);
        __syncthreads();  // the next piece reuses the LDS
    }
}

// ---- merging the pieces

constexpr int kMgThreads = 256;
constexpr int kMgItems = kUnit / kMgThreads;
static_assert(kRsCap == 2 * kUnit, "a piece is two merge units");

// Number of A's elements among the first d of A and B merged (B's first among equals):
// the first a in [max(0, d - nb), min(d, na)] with A[a] >= B[d - 1 - a], found by
// the whole wave, 64 probes a round.
__device__ __forceinline__ int32_t merge_split(const int32_t *__restrict__ A, int32_t na,
                                               const int32_t *__restrict__ B, int32_t nb, int32_t d) {
    const int lane = __lane_id();
    int32_t lo = d > nb ? d - nb : 0, hi = d < na ? d : na;  // answer in [lo, hi]
    while (lo < hi) {
        const int32_t step = (hi - lo + kWave - 1) / kWave;
        const int32_t a = lo + lane * step;
        const bool in = a < hi;
        const bool less = in && A[in ? a : lo] < B[d - 1 - (in ? a : lo)];  // a is below the answer
        const uint64_t m = __builtin_amdgcn_ballot_w64(less);
        const int32_t k = (int32_t)__popcll(m);  // probes 0 .. k - 1 are below it
        const int32_t nlo = k > 0 ? lo + (k - 1) * step + 1 : lo;
        const int32_t nhi = k < kWave && lo + k * step < hi ? lo + k * step : hi;
        lo = nlo;
        hi = nhi;
    }
    return lo;
}

__global__ __launch_bounds__(kMgThreads) void k_rs_merge(const int32_t *__restrict__ noff,
                                                         const HeavyCount *__restrict__ hc,
                                                         const int32_t *__restrict__ hrow,
                                                         const int32_t *__restrict__ hunit,
                                                         const int32_t *__restrict__ unit_row, int32_t level,
                                                         int32_t *__restrict__ out, int32_t *__restrict__ tmp) {
    __shared__ int32_t s[kUnit];
    __shared__ int32_t split[2];
    if (level >= hc->levels) return;
    const int32_t units = hc->units();
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t run = (int64_t)kRsCap << level;
    for (int32_t u = blockIdx.x; u < units; u += gridDim.x) {
        const int32_t h = unit_row[u], row = hrow[h], len = noff[row + 1] - noff[row];
        const int32_t levels = merge_levels(len);
        if (level >= levels) continue;  // uniform: the row is done
        const int64_t o0 = (int64_t)(u - hunit[h]) * kUnit, p0 = o0 / (2 * run) * (2 * run);
        const int32_t na = (int32_t)(len - p0 < run ? len - p0 : run);
        const int32_t nb = (int32_t)(len - p0 - na < run ? len - p0 - na : run);
        const int32_t d0 = (int32_t)(o0 - p0), d1 = d0 + kUnit < na + nb ? d0 + kUnit : na + nb, n = d1 - d0;
        const bool from_tmp = (levels - level) & 1;
        const int32_t *A = (from_tmp ? tmp : out) + (int64_t)noff[row] + p0, *B = A + na;
        int32_t *to = (from_tmp ? out : tmp) + (int64_t)noff[row] + o0;
        if (nb == 0 || A[na - 1] <= B[0]) {  // uniform: in order already, as pieces of neighbouring ids are
            for (int i = tid; i < n; i += kMgThreads) to[i] = A[d0 + i];
            continue;
        }
        if (w < 2) {
            const int32_t a = merge_split(A, na, B, nb, w == 0 ? d0 : d1);
            if ((tid & 63) == 0) split[w] = a;
        }
        __syncthreads();
        const int32_t a0 = split[0], b0 = d0 - a0, ma = split[1] - a0, mb = n - ma;
        for (int i = tid; i < n; i += kMgThreads) s[i] = i < ma ? A[a0 + i] : B[b0 + i - ma];
        __syncthreads();
        const int32_t *sa = s, *sb = s + ma;
        // this thread's kMgItems outputs
        const int32_t d = tid * kMgItems < n ? tid * kMgItems : n;
        int32_t lo = d > mb ? d - mb : 0, hi = d < ma ? d : ma;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (sa[mid] < sb[d - 1 - mid]) lo = mid + 1;
            else hi = mid;
        }
        int32_t a = lo, b = d - lo, v[kMgItems];
#pragma unroll
        for (int q = 0; q < kMgItems; ++q) {
            const int32_t x = a < ma ? sa[a] : 0x7fffffff, y = b < mb ? sb[b] : 0x7fffffff;
            const bool left = x < y;
            v[q] = left ? x : y;
            a += left ? 1 : 0;
            b += left ? 0 : 1;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kMgItems; ++q)
            if (d + q < n) s[d + q] = v[q];
        __syncthreads();
        for (int i = tid; i < n; i += kMgThreads) to[i] = s[i];
        __syncthreads();
    }
}

struct RsWs {
    int32_t *tmp, *hrow, *hunit, *unit_row, *crowded, *lengthy;
    uint32_t *tab;
    HeavyCount *hc;
};
template <class A>
static void rs_layout(A &a, int64_t E, RsWs *w) {
    const int64_t tiles = ceil_div(E, kRsTile), heavy = E / (kLightMax + 1) + 1, units = E / kUnit + heavy + 1;
    auto take = [&](auto *&p, int64_t n) {
        using T = typename std::remove_reference<decltype(*p)>::type;
        if constexpr (std::is_same<A, Arena>::value) p = a.template take<T>(n);
        else a.template take<T>(n);
    };
    take(w->tmp, E);
    take(w->hrow, heavy);
    take(w->hunit, heavy);
    take(w->unit_row, units);
    take(w->crowded, tiles > units ? tiles : units);  // tiles, then pieces
    take(w->lengthy, tiles);
    take(w->tab, kCells + 1);
    take(w->hc, 1);
}

size_t row_sort_ws_bytes(int32_t V, int64_t E) {
    ArenaSize a;
    RsWs w{};
    rs_layout(a, E, &w);
    return align_up(a.used, 256) + row_list_ws_bytes(V, E, kRsTile) + 256;
}

cagra_status sort_rows(const int32_t *in_offsets, const int32_t *in_sources, int32_t V, int64_t E,
                       const int32_t *perm, const int32_t *inv, const int32_t *new_off, const int32_t *cum,
                       const int32_t *outdeg_new, int32_t *out, void *ws, size_t ws_bytes, hipStream_t st) {
    Arena ar{(char *)ws, ws_bytes, 0};
    RsWs w{};
    rs_layout(ar, E, &w);
    if (!w.tmp || !w.hrow || !w.hunit || !w.unit_row || !w.crowded || !w.lengthy || !w.tab || !w.hc)
        return fail(CAGRA_E_BUFFER, "workspace too small (row sort)");
    for (const void *f : {(const void *)k_rs_light, (const void *)k_rs_light_lengthy, (const void *)k_rs_light_crowded,
                          (const void *)k_rs_pieces, (const void *)k_rs_pieces_crowded})
        if (cagra_status a_ = ensure_dynamic_lds(f)) return a_;
    const int32_t tiles = (int32_t)ceil_div(E, kRsTile);
    k_rs_table<<<1, 1024, 0, st>>>(cum, outdeg_new, V, w.tab, w.hc);
    CAGRA_LAUNCH_CHECK();
    RowList list;
    if (cagra_status s = build_row_list(new_off, V, E, kRsTile, ar, &list, st)) return s;
    k_rs_units<<<(unsigned)ceil_div(V, 256), 256, 0, st>>>(new_off, V, w.hc, w.hrow, w.hunit, w.unit_row);
    CAGRA_LAUNCH_CHECK();
    k_rs_light<<<(unsigned)tiles, kRsThreads, sizeof(SortLds<kShortItems>), st>>>(
        in_offsets, in_sources, perm, inv, list, E, w.tab, tiles, w.hc, w.crowded, w.lengthy, out);
    CAGRA_LAUNCH_CHECK();
    // grids of resident workgroups that walk lists whose lengths the host does not know
    const int64_t units = E / kUnit + E / (kLightMax + 1) + 1;
    const unsigned grid = (unsigned)(units < 2048 ? units : 2048);
    k_rs_light_lengthy<<<(unsigned)(tiles < 2048 ? tiles : 2048), kRsThreads, sizeof(SortLds<kRsItems>), st>>>(
        in_offsets, in_sources, perm, inv, list, E, w.tab, w.hc, w.crowded, w.lengthy, out);
    CAGRA_LAUNCH_CHECK();
    k_rs_light_crowded<<<(unsigned)(tiles < 512 ? tiles : 512), kRsThreads, sizeof(SortLds<kRsItems>), st>>>(
        in_offsets, in_sources, perm, inv, list, E, w.tab, w.hc, w.crowded, out);
    CAGRA_LAUNCH_CHECK();
    if (E <= kLightMax) return CAGRA_OK;  // no heavy row
    k_rs_pieces<<<grid, kRsThreads, sizeof(SortLds<kRsItems>), st>>>(in_offsets, in_sources, perm, inv, new_off, w.hc, w.hrow,
                                                           w.hunit, w.unit_row, w.tab, w.crowded, out, w.tmp);
    CAGRA_LAUNCH_CHECK();
    k_rs_pieces_crowded<<<grid < 256 ? grid : 256, kRsThreads, sizeof(SortLds<kRsItems>), st>>>(
        in_offsets, in_sources, perm, inv, new_off, w.hc, w.hrow, w.hunit, w.unit_row, w.tab, w.crowded, out, w.tmp);
    CAGRA_LAUNCH_CHECK();
    for (int32_t level = 0; ((int64_t)kRsCap << level) < E; ++level) {
        k_rs_merge<<<grid, kMgThreads, 0, st>>>(new_off, w.hc, w.hrow, w.hunit, w.unit_row, level, out, w.tmp);
        CAGRA_LAUNCH_CHECK();
    }
    return CAGRA_OK;
}

}  // namespace cagra
