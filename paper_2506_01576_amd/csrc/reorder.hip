// Point lookups on a batch partitioned by rank bucket.
//
// Section 7.4 observes that neighbouring lookups with close keys share their
// search paths, that globally sorting the batch gives this best, and that a
// block-local sort is the cheap approximation (the local form lives in
// qio.hpp).  On MI355X the global form pays at scale: a lookup into a
// 768 MiB index costs three to four 128-byte lines that miss L2 (random
// requests that miss L2 run at ~55 G/s whether the Infinity Cache or HBM
// serves them), while one XCD's 4 MiB L2 can hold the whole slice of the
// index that a narrow key range touches, and LDS the top of its search.  So
// the batch is partitioned -- one counting pass, not a sort -- into up to 1024
// buckets of neighbouring keys, each bucket is searched through a table of its
// own keys in LDS, and the answers are gathered back.  The order within a
// bucket is that of LDS atomics and changes from run to run; `place` below
// records it, and no answer depends on it.
//
//   1. splitters: NB - 1 index keys, in key order;
//   2. count: per tile of kPartTile queries, the queries of every bucket (a
//      table of key cells in LDS, then a search of the few splitters in the
//      query's cell), as a matrix;
//   3. scan of the matrix along each bucket;
//   4. scatter: each tile's queries, put in bucket order in LDS, leave in one
//      piece per bucket; every query's place within its tile goes to `place`,
//      in the caller's order;
//   5. lookup: spans of the partitioned batch, walked XCD by XCD so that the
//      buckets one XCD has in flight fit its L2;
//   6. gather: each tile reads its answers, a piece per bucket, back into LDS
//      in bucket order, and its queries' places give them out in order.
//
// Step 6 is why one pass suffices in both directions.  Writing the answers to
// their positions instead costs a 32-byte memory write per 4-byte answer (L2
// does not merge the writes of different waves), with a second pass to narrow
// them 3.2 ms per 2^27 lookups against 0.38 ms here.
//
// The partition is a pure function of the call: no state stays in the handle.
#include <type_traits>

#include "internal.hpp"
#include "access.hpp"
#include "qio.hpp"

namespace idx {
namespace {

constexpr uint32_t kPartThreads = 1024;
constexpr int kPartPer = 8;                            // queries per thread and tile
constexpr uint32_t kPartTile = kPartThreads * kPartPer;
constexpr uint32_t kMaxBuckets = 1024;                 // one thread per bucket in the tile's scan
constexpr uint64_t kBucketBytes = 3 * 512 * 1024;      // index bytes per bucket aimed at
constexpr uint64_t kBucketQueries = 1024;              // queries per bucket at least, on average
// Batches below this are looked up as they come: on BS, n = 2^21..2^26, the
// partition's launches take 62-170 us up to 2^18 queries, unpartitioned
// lookups 21-68 us; at 2^20 they take 65-221 and 59-271 us.  Range calls: 114-
// 236 and 71-128 us at 2^18, 143-405 and 164-402 us at 2^20.
constexpr uint64_t kPartMin = 3ull << 18;
// On smaller sets and other layouts the partition pays later, against the
// launches tuned for them.  us unpartitioned / partitioned, 64-bit keys:
//   BS   n = 2^17: 316 / 292 at 2^24 lookups, 2858 / 1967 at 2^27 (32-bit keys,
//        Zipf 1.1: 228 / 248 and 2097 / 1813); 2^18: 102 / 97 at 2^22, 195 / 158
//        at 2^23 (Zipf 1.1: 86 / 89 and 163 / 143); 2^20: 112 / 73 at 2^21, 211 /
//        103 at 2^22
//   EBS  n = 2^18: 119 / 139 at 2^22, 441 / 502 at 2^24; 2^20: 103 / 92 at 2^21,
//        193 / 141 at 2^22
//   EKS  k = 9, which reads few lines as it is; tables of a ninth of the keys:
//        n = 2^18: 86 / 93 at 2^22, 325 / 301 at 2^24; 2^20: 69 / 76 at 2^21, 136
//        / 103 at 2^22; 2^23: 67 / 89 at 2^20, 222 / 141 at 2^22; 2^26: 90 / 220
//        at 2^20, 309 / 348 at 2^22, 1183 / 725 at 2^24; n = 5 10^7, half misses,
//        Zipf 1.1: 335 / 354 at 7 10^6
inline uint64_t part_min(const idx_index *h) {
    const uint64_t n = h->n;
    const bool small = n < 3u << 18;
    if (h->layout == IDX_EKS) return small ? 3ull << 21 : (1ull << 21) + n / 8;
    if (h->layout == IDX_EBS) return small ? ~0ull : n < 1u << 21 ? 3ull << 20 : kPartMin;
    return n < 1u << 18 ? 1ull << 26 : small ? 1ull << 23 : kPartMin;
}

// The same for range calls: BS n = 2^18 123 / 130 at 2^20 ranges, 372 / 285 at
// 2^22; 2^20 164 / 142 and 539 / 309; EBS n = 2^18 407 / 482 at 2^22, 1554 / 1783
// at 2^24; 2^20 174 / 193 at 2^20, 573 / 527 at 2^22.
// k-ary counts that read whole nodes of up to 128 bytes by 16-byte loads touch
// few lines as they come: k = 9, 64-bit keys, n = 2^26: 436 / 468 at 2^22, 1579 /
// 1482 at 2^24; 32-bit keys 1633 / 1740; k = 17 and 5 alike.  The others pay for
// every probe:
//   interleaved, k = 17, 64-bit keys: n = 2^18 809 / 711 at 2^22; 2^21 704 / 479 at
//        2^21; 2^23 431 / 261 at 3 2^18, 5816 / 3162 at 2^24; 2^26 193 / 221 at 2^18,
//        559 / 341 at 3 2^18, 7774 / 3474 at 2^24; k = 5 n = 2^23 214 / 172 at 3 2^18;
//        k = 3 n = 2^22 153 / 157 at 3 2^18, 302 / 242 at 2^21
//   apart, k = 65: n = 2^20 1120 / 938 at 2^21; 2^26 747 / 586 at 3 2^18; k = 4 and 64-bit
//        keys: n = 2^20 439 / 368 at 2^22; 2^23 189 / 181 at 2^20, 324 / 253 at 2^21;
//        2^26 3085 / 1756 at 2^24; k = 2 and 32-bit keys: n = 2^18 923 / 1041 at 2^24;
//        2^20 326 / 325 at 2^22; 2^22 144 / 154 at 2^20, 242 / 219 at 2^21
inline uint64_t range_part_min(const idx_index *h) {
    const bool small = h->n < 3u << 18;
    if (h->layout == IDX_EKS) {
        const uint32_t g = h->geo.g, node = g * (h->u64 ? 8 : 4);
        const bool whole = !h->aos && g >= 4 && node % 16 == 0 && node <= 128;
        if (small || whole) return ~0ull;
        if (h->n < 1u << 22) return 1ull << 22;
        return (h->aos && g >= 4) || node > 128 ? kPartMin : 1ull << 21;
    }
    if (h->layout == IDX_EBS) return small ? ~0ull : h->n < 1u << 21 ? 3ull << 20 : kPartMin;
    return small ? 3ull << 19 : kPartMin;
}

// How a call is partitioned.
struct PartGeo {
    uint32_t NB;    // buckets (1: not worth a partition)
    uint32_t L;     // levels of a bucket's table in LDS
    uint32_t D;     // sorted array: a table entry for every 2^D keys, at least a run of them
    uint32_t top;   // binary Eytzinger layout: the splitters are the keys of the top `top` levels
    uint64_t step;  // sorted array: ranks per bucket, 2^(L + D); bucket b's keys have their lower bounds in
                    //   [b * step, (b + 1) * step), or at n

    // k-ary Eytzinger layout: buckets of up to `entries` neighbouring nodes of
    // one level.  Cut the tree above level c: its top c levels are k^c - 1 keys
    // in key order, and node j of level c holds the root of what lies between
    // keys j - 1 and j.  The first `left` nodes of level cut_l make the first
    // NB_l buckets, the nodes of level cut_r after them, [right, gaps), the
    // others: where the partial level ends, so that every bucket spans about as
    // many keys.
    uint32_t entries, cut_l, cut_r, NB_l, left, right, gaps;

    uint64_t tab;  // entries of the buckets' tables in memory: NB << L, or none
};

// How a partitioned batch is searched: through the tables of k_part_bs or
// k_part_eks, by k_part_ebs's descent, or by the handle's own lookup kernel.
enum class Search { sorted_tables, node_tables, subtrees, own };

Search point_search(const idx_index *h) {
    if (h->layout == IDX_EBS) return Search::subtrees;
    if (h->layout == IDX_BS) return h->learned && h->params.model != 2 ? Search::own : Search::sorted_tables;
    const uint64_t node = (uint64_t)h->geo.g * (h->u64 ? 8 : 4);
    return !h->aos && (node == 32 || node == 64 || node == 128) ? Search::node_tables : Search::own;
}

// Ranges: k_part_range_bs's tables, or the counting kernel over the batch.
Search range_search(const idx_index *h) { return h->layout == IDX_BS ? Search::sorted_tables : Search::own; }

// Bucket b of the k-ary Eytzinger layout: nodes [j0, j1) of level `cut`.
__host__ __device__ inline void bucket_nodes(const PartGeo &P, uint32_t b, uint32_t &cut, uint32_t &j0, uint32_t &j1) {
    const bool l = b < P.NB_l;
    const uint32_t end = l ? P.left : P.gaps;
    cut = l ? P.cut_l : P.cut_r;
    j0 = l ? b * P.entries : P.right + (b - P.NB_l) * P.entries;
    j1 = end - j0 < P.entries ? end : j0 + P.entries;
}

// Splitters of the sorted array: the last key of every bucket's ranks.
template <typename K, bool AOS>
__global__ void k_split_sorted(Load<K, AOS> L, uint64_t step, uint32_t NB, K *__restrict__ split) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= NB) return;
    split[j] = (j + 1 < NB) ? L.key((uint64_t)(j + 1) * step - 1) : key_max_v<K>();
}

// Key j, in key order, of a full tree of `levels` levels: its level and its
// position on that level.  j + 1 = k^e u with u not a multiple of k puts it on
// level levels - 1 - e, at (u - 1) - (u - 1) / k.
__device__ __forceinline__ uint64_t key_slot(const Geo &G, uint32_t j, uint32_t levels) {
    uint32_t u = j + 1, e = 0;
    while (u % G.k == 0) {
        u /= G.k;
        ++e;
    }
    return G.start[levels - 1 - e] + (u - 1) - (u - 1) / G.k;
}

// Splitters of an Eytzinger layout.  Binary: the keys of its top levels in key
// order (a full tree of NB - 1 keys), so that bucket b is the subtree of the
// b-th node below them.  k-ary: the key after each bucket's last node.
template <typename K, bool AOS>
__global__ void k_split_eyt(Load<K, AOS> L, Geo G, uint64_t off, PartGeo P, K *__restrict__ split) {
    const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= P.NB) return;
    if (b + 1 == P.NB) {
        split[b] = key_max_v<K>();
        return;
    }
    uint32_t cut = P.top, j0, j1 = b + 1;
    if (P.entries) bucket_nodes(P, b, cut, j0, j1);
    split[b] = L.key(off + key_slot(G, j1 - 1, cut));
}

// Bucket table: the key range from the first splitter to the second-largest
// one is cut into kCells cells of 2^sh keys (the last cell also takes every
// larger key, the first every smaller one).  Cell h's keys lie between the
// splitters cell_first[h] and cell_first[h + 1], so a lookup searches only
// those: none or one for uniform keys, never more than all B.
constexpr uint32_t kCellBits = 12;
constexpr uint32_t kCells = 1u << kCellBits;

template <typename K>
__device__ __forceinline__ uint32_t cell_of(K x, K base, uint32_t sh) {
    if (x < base) return 0;
    const uint64_t c = (uint64_t)(x - base) >> sh;
    return c < kCells - 1 ? (uint32_t)c : kCells - 1;
}

// Cell width: the smallest 2^sh for which the span from split[0] to
// split[B - 2] fits kCells cells.
template <typename K>
__device__ __forceinline__ uint32_t cell_shift(const K *s_split, uint32_t B) {
    const uint64_t span = B >= 2 ? (uint64_t)(s_split[B - 2] - s_split[0]) : 0;
    const uint32_t bits = span ? 64u - (uint32_t)__clzll((long long)span) : 0u;
    return bits > kCellBits ? bits - kCellBits : 0u;
}

// Fills cell_first[0, kCells]: the number of splitters whose cell is below h.
template <typename K>
__device__ __forceinline__ void build_cells(const K *s_split, uint32_t B, K base, uint32_t sh, uint16_t *cell_first) {
    for (uint32_t h = threadIdx.x; h <= kCells; h += blockDim.x) {
        uint32_t lo = 0, n = B;  // first splitter j with cell_of(split[j]) >= h
        while (n) {
            const uint32_t half = n >> 1;
            if (cell_of(s_split[lo + half], base, sh) < h) {
                lo += half + 1;
                n -= half + 1;
            } else {
                n = half;
            }
        }
        cell_first[h] = (uint16_t)lo;
    }
}

// Bucket of x = the number of splitters below x (splitters ascend, the last
// is the largest key): all those of lower cells plus those of x's own cell
// that are below x.
template <typename K>
__device__ __forceinline__ uint32_t bucket_of_cells(const K *s_split, const uint16_t *cell_first, K base, uint32_t sh,
                                                    K x) {
    const uint32_t h = cell_of(x, base, sh);
    uint32_t b = cell_first[h], n = (uint32_t)cell_first[h + 1] - b;
    while (n) {
        const uint32_t half = n >> 1;
        if (s_split[b + half] < x) {
            b += half + 1;
            n -= half + 1;
        } else {
            n = half;
        }
    }
    return b;
}

// LDS tables of the bucket function.
template <typename K>
struct Buckets {
    K *s_split;
    uint16_t *s_cell;
    K base;
    uint32_t sh;
    // Fills the tables (every thread of the workgroup); s_cell has kCells + 1 entries.
    __device__ __forceinline__ void build(const K *__restrict__ split, uint32_t NB) {
        for (uint32_t i = threadIdx.x; i < NB; i += blockDim.x) s_split[i] = split[i];
        __syncthreads();
        base = s_split[0];
        sh = cell_shift(s_split, NB);
        build_cells(s_split, NB, base, sh, s_cell);
        __syncthreads();
    }
    __device__ __forceinline__ uint32_t of(K x) const { return bucket_of_cells(s_split, s_cell, base, sh, x); }
};

constexpr size_t kCellBytes = ((kCells + 1) * 2 + 15) & ~(size_t)15;

// 2. Queries of every bucket in every tile: hist[b * tiles + tile].  The
// tiles are walked XCD by XCD, so the counts that share a line of the matrix
// are written by one XCD.
template <typename K>
__global__ __launch_bounds__(kPartThreads) void k_part_count(const K *__restrict__ q, uint64_t m,
                                                             const K *__restrict__ split, uint32_t NB, uint32_t tiles,
                                                             uint32_t iters, uint32_t *__restrict__ hist) {
    extern __shared__ __align__(16) char smem[];
    Buckets<K> B{(K *)smem, (uint16_t *)(smem + NB * sizeof(K)), K(0), 0};
    uint32_t *s_cnt = (uint32_t *)(smem + NB * sizeof(K) + kCellBytes);
    for (uint32_t b = threadIdx.x; b < NB; b += kPartThreads) s_cnt[b] = 0;
    B.build(split, NB);
    for (uint32_t it = blockIdx.x; it < iters; it += gridDim.x) {
        const uint32_t tile = (uint32_t)tile_of(it, tiles, 1);
        if (tile >= tiles) continue;  // workgroup-uniform
        const uint64_t t0 = (uint64_t)tile * kPartTile;
        K x[kPartPer];
#pragma unroll
        for (int u = 0; u < kPartPer; ++u) {
            const uint64_t i = t0 + (uint32_t)u * kPartThreads + threadIdx.x;
            x[u] = i < m ? q[i] : K(0);
        }
#pragma unroll
        for (int u = 0; u < kPartPer; ++u) {
            const uint64_t i = t0 + (uint32_t)u * kPartThreads + threadIdx.x;
            if (i < m) atomicAdd(&s_cnt[B.of(x[u])], 1u);
        }
        __syncthreads();
        if (threadIdx.x < NB) {  // NB <= kPartThreads
            hist[(uint64_t)threadIdx.x * tiles + tile] = s_cnt[threadIdx.x];
            s_cnt[threadIdx.x] = 0;
        }
        __syncthreads();
    }
}

// Exclusive scan of one value per thread over the workgroup; s_wave holds one
// entry per wave.  Barriers on both sides.
__device__ __forceinline__ uint32_t part_scan(uint32_t v, uint32_t *s_wave, uint32_t *total) {
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t t = (uint32_t)__shfl_up((int)incl, off, kWave);
        if (lane >= (uint32_t)off) incl += t;
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = 0, sum = 0;
    for (uint32_t w = 0; w < blockDim.x / kWave; ++w) {
        const uint32_t c = s_wave[w];
        before += w < wave ? c : 0;
        sum += c;
    }
    __syncthreads();
    *total = sum;
    return before + incl - v;
}

// 3. One workgroup per bucket: exclusive scan of its counts along the tiles,
// in place, and its total.
constexpr uint32_t kScanThreads = 256;
constexpr int kScanPer = 16;

__global__ __launch_bounds__(kScanThreads) void k_part_scan(uint32_t *__restrict__ hist, uint32_t tiles,
                                                            uint32_t *__restrict__ total) {
    __shared__ uint32_t s_wave[kScanThreads / kWave];
    uint32_t *row = hist + (uint64_t)blockIdx.x * tiles;
    uint32_t running = 0;
    for (uint32_t c0 = 0; c0 < tiles; c0 += kScanThreads * kScanPer) {
        uint32_t v[kScanPer], sum = 0;
        const uint32_t first = c0 + threadIdx.x * kScanPer;
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            v[j] = first + j < tiles ? row[first + j] : 0u;
            sum += v[j];
        }
        uint32_t all;
        uint32_t acc = running + part_scan(sum, s_wave, &all);
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            if (first + j < tiles) row[first + j] = acc;
            acc += v[j];
        }
        running += all;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = running;
}

// 4. The scatter.  Per tile: every query's bucket and its turn in it (LDS
// atomics), the buckets' starts within the tile, the queries into LDS in
// bucket order, and out, consecutive threads writing consecutive addresses of
// a bucket's piece.  A persistent workgroup per compute unit keeps the bucket
// tables; the next tile's queries are loaded while this one's leave.
// RANGE: a second key per query (the ranges' upper bounds) moves along.
// starts[b] (NB + 1 entries) receives the buckets' starts.
// Bound by memory: 18 B per 64-bit query, 0.67 ms per 2^27 (two passes of 28 and
// 30 B took 2.57 ms).
template <typename K>
size_t scatter_lds_bytes(uint32_t NB) {
    return (size_t)NB * sizeof(K) + kCellBytes + (size_t)NB * 12 + (size_t)kPartTile * (sizeof(K) + 2) + 16;
}

template <typename K, bool RANGE>
__global__ __launch_bounds__(kPartThreads) void k_part_scatter(const K *__restrict__ q, const K *__restrict__ q_hi,
                                                               uint64_t m, const K *__restrict__ split, uint32_t NB,
                                                               uint32_t tiles, uint32_t iters,
                                                               const uint32_t *__restrict__ hist,
                                                               const uint32_t *__restrict__ total,
                                                               K *__restrict__ q2, K *__restrict__ q2_hi,
                                                               uint16_t *__restrict__ place,
                                                               uint32_t *__restrict__ starts) {
    extern __shared__ __align__(16) char smem[];
    K *s_q = (K *)smem;
    char *p = smem + (size_t)kPartTile * sizeof(K);
    Buckets<K> B{(K *)p, (uint16_t *)(p + NB * sizeof(K)), K(0), 0};
    p += NB * sizeof(K) + kCellBytes;
    uint32_t *s_cnt = (uint32_t *)p;   // the tile's queries of each bucket
    uint32_t *s_start = s_cnt + NB;    // their start within the tile
    uint32_t *s_off = s_start + NB;    // place in q2 minus place in the tile
    uint16_t *s_run = (uint16_t *)(s_off + NB);
    __shared__ uint32_t s_wave[kPartThreads / kWave];
    const uint32_t tid = threadIdx.x;
    uint32_t all;
    const uint32_t base = part_scan(tid < NB ? total[tid] : 0u, s_wave, &all);
    if (blockIdx.x == 0 && tid < NB) {
        starts[tid] = base;
        if (tid == 0) starts[NB] = (uint32_t)m;
    }
    if (tid < NB) s_cnt[tid] = 0;
    B.build(split, NB);
    K x[kPartPer];
    auto load = [&](uint32_t tile) {
        const uint64_t t0 = (uint64_t)tile * kPartTile;
#pragma unroll
        for (int u = 0; u < kPartPer; ++u) {
            const uint64_t i = t0 + (uint32_t)u * kPartThreads + tid;
            x[u] = i < m ? q[i] : K(0);
        }
    };
    uint32_t it = blockIdx.x;
    uint32_t tile = it < iters ? (uint32_t)tile_of(it, tiles, 1) : tiles;
    if (tile < tiles) load(tile);
    while (it < iters) {
        const uint32_t next = it + gridDim.x;
        const uint32_t next_tile = next < iters ? (uint32_t)tile_of(next, tiles, 1) : tiles;
        if (tile < tiles) {  // workgroup-uniform
            const uint64_t t0 = (uint64_t)tile * kPartTile;
            const uint32_t cnt = m - t0 < kPartTile ? (uint32_t)(m - t0) : kPartTile;
            const uint32_t before = tid < NB ? hist[(uint64_t)tid * tiles + tile] : 0u;
            uint32_t at[kPartPer];  // bucket << 16 | turn, then place in the tile
#pragma unroll
            for (int u = 0; u < kPartPer; ++u) {
                at[u] = 0;
                if ((uint32_t)u * kPartThreads + tid < cnt) {
                    const uint32_t b = B.of(x[u]);
                    at[u] = (b << 16) | atomicAdd(&s_cnt[b], 1u);
                }
            }
            __syncthreads();
            const uint32_t start = part_scan(tid < NB ? s_cnt[tid] : 0u, s_wave, &all);
            if (tid < NB) {
                s_start[tid] = start;
                s_off[tid] = base + before - start;
                s_cnt[tid] = 0;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kPartPer; ++u) {
                const uint32_t j = (uint32_t)u * kPartThreads + tid;
                if (j >= cnt) continue;
                const uint32_t b = at[u] >> 16, pos = s_start[b] + (at[u] & 0xFFFFu);
                s_q[pos] = x[u];
                s_run[pos] = (uint16_t)b;
                place[t0 + j] = (uint16_t)pos;
                at[u] = pos;
            }
            if constexpr (RANGE) {
#pragma unroll
                for (int u = 0; u < kPartPer; ++u) {
                    const uint32_t j = (uint32_t)u * kPartThreads + tid;
                    x[u] = j < cnt ? q_hi[t0 + j] : K(0);
                }
            } else if (next_tile < tiles) {
                load(next_tile);
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kPartPer; ++u) {
                const uint32_t j = (uint32_t)u * kPartThreads + tid;
                if (j < cnt) q2[s_off[s_run[j]] + j] = s_q[j];
            }
            __syncthreads();
            if constexpr (RANGE) {
#pragma unroll
                for (int u = 0; u < kPartPer; ++u)
                    if ((uint32_t)u * kPartThreads + tid < cnt) s_q[at[u]] = x[u];
                if (next_tile < tiles) load(next_tile);
                __syncthreads();
#pragma unroll
                for (int u = 0; u < kPartPer; ++u) {
                    const uint32_t j = (uint32_t)u * kPartThreads + tid;
                    if (j < cnt) q2_hi[s_off[s_run[j]] + j] = s_q[j];
                }
                __syncthreads();
            }
        } else if (next_tile < tiles) {
            load(next_tile);
        }
        it = next;
        tile = next_tile;
    }
}

// 6. A tile's answers sit in one piece per bucket: they are read piece by piece,
// consecutive threads on consecutive answers, into LDS in bucket order, and
// out[i] = the tile's answer place[i].  Tiles are walked XCD by XCD like the
// scatter's, so that the lines two tiles' pieces share are read once.  Bound by
// memory: 0.38 ms per 2^27 answers of 4 bytes from 512 buckets, 0.61 from 910
// (a read per answer at its 32-bit place in the whole batch, as many L2
// requests, took 0.55 and 0.61).
template <typename T>
__global__ __launch_bounds__(kPartThreads) void k_part_gather(const T *__restrict__ ans,
                                                              const uint16_t *__restrict__ place, uint64_t m,
                                                              uint32_t NB, uint32_t tiles, uint32_t iters,
                                                              const uint32_t *__restrict__ hist,
                                                              const uint32_t *__restrict__ total,
                                                              const uint32_t *__restrict__ starts,
                                                              T *__restrict__ out) {
    __shared__ T s_ans[kPartTile];
    __shared__ __align__(16) uint16_t s_run[kPartTile];  // bucket of every place, eight to a 16-byte word
    __shared__ uint32_t s_off[kMaxBuckets];  // place in ans minus place in the tile
    __shared__ uint32_t s_wave[kPartThreads / kWave];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const uint32_t mine = tid < NB ? starts[tid] : 0u, in_all = tid < NB ? total[tid] : 0u;
    uint32_t first = 0, count = 0;  // the tile's answers in bucket tid
    uint16_t at[kPartPer];
    auto load = [&](uint32_t tile) {
        if (tid < NB) {
            const uint32_t *row = hist + (uint64_t)tid * tiles + tile;
            first = row[0];
            count = (tile + 1 < tiles ? row[1] : in_all) - first;
        }
        const uint64_t t0 = (uint64_t)tile * kPartTile;
#pragma unroll
        for (int u = 0; u < kPartPer; ++u) {
            const uint64_t i = t0 + (uint32_t)u * kPartThreads + tid;
            at[u] = i < m ? __builtin_nontemporal_load(place + i) : (uint16_t)0;
        }
    };
    static_assert(kPartPer == 8, "a thread's places are one 16-byte word of s_run");
    uint32_t it = blockIdx.x;
    uint32_t tile = it < iters ? (uint32_t)tile_of(it, tiles, 1) : tiles;
    if (tile < tiles) load(tile);
    while (it < iters) {
        const uint32_t next = it + gridDim.x;
        const uint32_t next_tile = next < iters ? (uint32_t)tile_of(next, tiles, 1) : tiles;
        if (tile < tiles) {  // workgroup-uniform
            const uint64_t t0 = (uint64_t)tile * kPartTile;
            const uint32_t cnt = m - t0 < kPartTile ? (uint32_t)(m - t0) : kPartTile;
            ((uint4 *)s_run)[tid] = make_uint4(0, 0, 0, 0);
            uint32_t all;
            const uint32_t start = part_scan(count, s_wave, &all);
            if (count) {
                s_run[start] = (uint16_t)tid;
                s_off[tid] = mine + first - start;
            }
            __syncthreads();
            // every place's bucket: the largest marked at or before it
            uint32_t b[kPartPer], last = 0;
            const uint4 w = ((const uint4 *)s_run)[tid];
            const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < kPartPer; ++j) {
                const uint32_t v = (ww[j / 2] >> (16 * (j & 1))) & 0xFFFFu;
                last = v > last ? v : last;
                b[j] = last;
            }
            uint32_t before = last;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t o = (uint32_t)__shfl_up((int)before, off, kWave);
                if (lane >= (uint32_t)off) before = o > before ? o : before;
            }
            if (lane == kWave - 1) s_wave[wave] = before;
            before = (uint32_t)__shfl_up((int)before, 1, kWave);
            if (lane == 0) before = 0;
            __syncthreads();
            for (uint32_t v = 0; v < wave; ++v) before = s_wave[v] > before ? s_wave[v] : before;
            uint32_t packed[4];
#pragma unroll
            for (int j = 0; j < kPartPer; ++j) b[j] = b[j] > before ? b[j] : before;
#pragma unroll
            for (int j = 0; j < 4; ++j) packed[j] = b[2 * j] | (b[2 * j + 1] << 16);
            ((uint4 *)s_run)[tid] = make_uint4(packed[0], packed[1], packed[2], packed[3]);
            __syncthreads();
            T v[kPartPer];
#pragma unroll
            for (int u = 0; u < kPartPer; ++u) {
                const uint32_t j = (uint32_t)u * kPartThreads + tid;
                if (j < cnt) v[u] = ans[s_off[s_run[j]] + j];
            }
            uint16_t from[kPartPer];
#pragma unroll
            for (int u = 0; u < kPartPer; ++u) from[u] = at[u];
            if (next_tile < tiles) load(next_tile);
#pragma unroll
            for (int u = 0; u < kPartPer; ++u) {
                const uint32_t j = (uint32_t)u * kPartThreads + tid;
                if (j < cnt) s_ans[j] = v[u];
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kPartPer; ++u) {
                const uint32_t j = (uint32_t)u * kPartThreads + tid;
                if (j < cnt) __builtin_nontemporal_store(s_ans[from[u]], out + t0 + j);
            }
        } else if (next_tile < tiles) {
            load(next_tile);
        }
        it = next;
        tile = next_tile;
    }
}

// ------------------------------------------------------------------ lookups

// A workgroup takes a span of the partitioned batch, bucket by bucket: it
// copies the bucket's table to LDS, 2^L entries in heap order (entry v's
// children are 2v and 2v + 1, which keeps a wave's reads of one level on
// different banks), and each lane walks R queries down it in lockstep, then
// down the rest of the bucket in memory, which its XCD's L2 holds.
//
// Bound by L2 requests: 128 channels serve about 270 G/s, and with 8192
// queries in flight per compute unit no line stays in the 32 KiB L1 between
// two dependent probes, so every probe is one.  On the sorted array, per 2^27
// lookups at n = 2^26: 11 probes and a short-window scan from the bucket's
// rank interval 4.74 ms; 12 levels in LDS and 5 probes 3.92 ms (7 requests a
// lookup); 13 levels in LDS, then the one line that holds the lower bound,
// read by eight lanes with one load, 1.55 ms (2.1 requests a lookup; half of the
// waves' time is waiting: two workgroups a compute unit, 64 KiB of LDS each,
// overlap the table's copy, the walk and the lines only so far).
constexpr uint32_t kLookThreads = 1024;
constexpr int kLookPer = 4;        // queries per lane at once
constexpr uint32_t kSpan = kLookThreads * kLookPer;  // queries per workgroup: two workgroups per compute unit keep
                                                     // the queries an XCD has in flight within a bucket or two
                                                     // (twice the span: its L2 thrashed, 4.89 ms)
constexpr uint32_t kMaxLevels1 = 13;  // levels in LDS: 64 KiB of 64-bit keys, two workgroups per compute unit
constexpr uint32_t kMinLevels = 6;

// The last step of a search reads a run of keys with kRunLanes lanes, 16 bytes
// each, one request: a whole line.  (Half a line halves the lanes' work, 1.53
// against 1.67 ms per 2^27 lookups when tried, but needs twice the buckets at n = 2^26,
// and the count, scatter and gather lose 0.26 ms to their shorter pieces.)
constexpr uint32_t kRunLanes = 8;

template <typename K>
constexpr uint32_t run_log() {  // log2 of the keys of a run
    return (kRunLanes == 4 ? 2u : 3u) + (sizeof(K) == 8 ? 1u : 2u);
}

// Tables of the sorted array: entry i in key order is the key at rank
// b * step + (i + 1) 2^D - 1, i < 2^L - 1 (heap entry 0 is unused).  With c
// entries below x, bucket b's x has its lower bound in the 2^D ranks from
// b * step + c 2^D.  Ranks past the array count as above everything.  Written once per call, so that the many workgroups of
// one bucket copy it with consecutive loads.
template <typename K, bool AOS>
__global__ __launch_bounds__(256) void k_part_tables(Load<K, AOS> A, uint64_t n, PartGeo P, K *__restrict__ tab) {
    const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const uint32_t b = (uint32_t)(t >> P.L), v = (uint32_t)(t & ((1u << P.L) - 1u));
    if (b >= P.NB || v == 0) return;
    const uint32_t l = 31u - (uint32_t)__clz((int)v);
    const uint64_t i = ((2ull * (v - (1u << l)) + 1) << (P.L - 1 - l)) - 1;
    const uint64_t at = b * P.step + ((i + 1) << P.D) - 1;
    tab[t] = at < n ? A.key(at) : key_max_v<K>();
}

// Tables of the k-ary Eytzinger layout: entry i in key order is the key after
// the bucket's i-th node, in the same heap order; rows has their row IDs.  With
// c entries below x, the descent goes on at node c, and entry c is the only one
// that can equal x.
template <typename K>
__global__ __launch_bounds__(256) void k_part_tables_eks(Load<K, false> A, Geo G, PartGeo P, K *__restrict__ tab,
                                                         uint32_t *__restrict__ rows) {
    const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const uint32_t b = (uint32_t)(t >> P.L), v = (uint32_t)(t & ((1u << P.L) - 1u));
    if (b >= P.NB || v == 0) return;
    const uint32_t lv = 31u - (uint32_t)__clz((int)v);
    const uint32_t i = ((2u * (v - (1u << lv)) + 1) << (P.L - 1 - lv)) - 1;
    uint32_t cut, j0, j1;
    bucket_nodes(P, b, cut, j0, j1);
    const bool real = i < j1 - j0 && j0 + i < G.start[cut];  // (no key follows the level's last node)
    const uint64_t at = real ? key_slot(G, j0 + i, cut) : 0ull;
    tab[t] = real ? A.key(at) : key_max_v<K>();
    rows[t] = real ? A.row(at) : kMiss;
}

template <typename K>
__device__ __forceinline__ void fill_table(const K *__restrict__ tab, uint32_t b, uint32_t L, K *s_tab) {
    const uint4 *src = (const uint4 *)(tab + ((uint64_t)b << L));
    const uint32_t chunks = (uint32_t)(sizeof(K) << L) / 16;  // L >= kMinLevels
    for (uint32_t v = threadIdx.x; v < chunks; v += kLookThreads) ((uint4 *)s_tab)[v] = src[v];
}

// Table entries below each x.
template <typename K, int R>
__device__ __forceinline__ void table_count(const K *s_tab, uint32_t L, const K (&x)[R], uint32_t (&c)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) c[r] = 1;
    for (uint32_t l = 0; l < L; ++l) {
#pragma unroll
        for (int r = 0; r < R; ++r) c[r] = 2 * c[r] + (s_tab[c[r]] < x[r] ? 1u : 0u);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) c[r] -= 1u << L;
}

// Start rank (relative to the bucket) of the 2^D ranks that hold each x.
template <typename K, int R>
__device__ __forceinline__ void table_find(const K *s_tab, const PartGeo &P, const K (&x)[R], uint32_t (&rel)[R]) {
    table_count<K, R>(s_tab, P.L, x, rel);
#pragma unroll
    for (int r = 0; r < R; ++r) rel[r] <<= P.D;
}

// Value of lane k of each group of NL lanes.
template <uint32_t NL, int k>
__device__ __forceinline__ uint32_t run_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (0x20 - (int)NL) | (k << 5));
}
template <uint32_t NL, int k>
__device__ __forceinline__ uint64_t run_lane(uint64_t v) {
    return ((uint64_t)run_lane<NL, k>((uint32_t)(v >> 32)) << 32) | run_lane<NL, k>((uint32_t)v);
}

// Sum of v over each group of NL lanes, in all of them.
template <uint32_t NL>
__device__ __forceinline__ uint32_t run_sum(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);  // lane ^ 1
    if constexpr (NL >= 4) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);   // lane ^ 2
    if constexpr (NL >= 8) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);  // 7 - lane
    return v;
}

// Every lane's run (from rank `run` of the bucket, a multiple of the run's
// keys) is read by its group of NL lanes, 16 bytes a lane: keys below x into
// below, and whether one equals x.  FULL: no run ends past `have` ranks; what
// lies there is anything.  The lanes' counts of a group's queries are summed
// as bytes, four queries to a word (a run has at most 32 keys): 171 vector
// instructions per 64 lookups of k_part_bs with 64-bit keys, where counting bits
// of ballots took 277; 1.55 ms per 2^27 either way, 1.42 against 1.70 with 32-bit
// keys.
template <typename K, uint32_t NL, bool FULL>
__device__ __forceinline__ void run_all(const K *__restrict__ keys, uint32_t have, uint32_t run, K x, uint32_t &below,
                                        bool &equal) {
    constexpr int V = 16 / sizeof(K), W = (NL + 3) / 4, U = NL < 4 || sizeof(K) == 8 ? 2 : 4;
    const uint32_t sub = threadIdx.x & (NL - 1);
    uint32_t lt[W] = {}, eq[W] = {};
    auto some = [&]<int k0>(std::integral_constant<int, k0>) {  // U queries from k0 on, loaded together
        uint32_t at[U];
        uint4 w[U];
        at[0] = run_lane<NL, k0>(run) + sub * V;
        at[1] = run_lane<NL, k0 + 1>(run) + sub * V;
        if constexpr (U == 4) {
            at[2] = run_lane<NL, k0 + 2>(run) + sub * V;
            at[3] = run_lane<NL, k0 + 3>(run) + sub * V;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = *(const uint4 *)((const char *)keys + at[u] * (uint32_t)sizeof(K));
        K xs[U];
        xs[0] = run_lane<NL, k0>(x);
        xs[1] = run_lane<NL, k0 + 1>(x);
        if constexpr (U == 4) {
            xs[2] = run_lane<NL, k0 + 2>(x);
            xs[3] = run_lane<NL, k0 + 3>(x);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            K kk[V];
            if constexpr (sizeof(K) == 8) {
                kk[0] = ((uint64_t)w[u].y << 32) | w[u].x;
                kk[1] = ((uint64_t)w[u].w << 32) | w[u].z;
            } else {
                kk[0] = w[u].x;
                kk[1] = w[u].y;
                kk[2] = w[u].z;
                kk[3] = w[u].w;
            }
            uint32_t c = 0;
            bool e = false;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const bool in = FULL || at[u] + v < have;
                c += in && kk[v] < xs[u] ? 1u : 0u;
                e |= in && kk[v] == xs[u];
            }
            lt[k0 / 4] += c << (8 * (k0 % 4 + u));
            eq[k0 / 4] += e ? 1u << (8 * (k0 % 4 + u)) : 0u;
        }
    };
    some(std::integral_constant<int, 0>{});
    if constexpr (U == 2 && NL >= 4) some(std::integral_constant<int, 2>{});
    if constexpr (NL == 8) some(std::integral_constant<int, 4>{});
    if constexpr (U == 2 && NL == 8) some(std::integral_constant<int, 6>{});
#pragma unroll
    for (int j = 0; j < W; ++j) {
        lt[j] = run_sum<NL>(lt[j]);
        eq[j] = run_sum<NL>(eq[j]);
    }
    const uint32_t l = W == 2 && sub >= 4 ? lt[W - 1] : lt[0], q = W == 2 && sub >= 4 ? eq[W - 1] : eq[0];
    below = (l >> (8 * (sub & 3u))) & 0xFFu;
    equal = ((q >> (8 * (sub & 3u))) & 0xFFu) != 0;
}

// Lower bounds of x[R] from rank `base` on: rel[r] comes as the start of the
// 2^D ranks that hold it (a multiple of a run's keys; base + rel <= n) and
// leaves as the lower bound.  All lanes of the wave call this together.  hit:
// the key there equals x.
template <typename K, bool AOS, int R>
__device__ __forceinline__ void settle(const Load<K, AOS> &A, uint64_t n, uint64_t base, const PartGeo &P,
                                       const K (&x)[R], uint32_t (&rel)[R], bool (&hit)[R]) {
    constexpr uint32_t last = AOS ? 0u : run_log<K>();  // keys and row IDs interleaved: probes to the end
    const uint32_t have = n - base < 0xFFFFFFFFull ? (uint32_t)(n - base) : 0xFFFFFFFFu;
    for (uint32_t e = P.D; e-- > last;) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t at = rel[r] + (1u << e) - 1;
            rel[r] += (at < have && A.key(base + at) < x[r]) ? 1u << e : 0u;
        }
    }
    if constexpr (AOS) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const K k = rel[r] < have ? A.key(base + rel[r]) : key_max_v<K>();
            hit[r] = rel[r] < have && k == x[r];
            rel[r] += rel[r] < have && k < x[r] ? 1u : 0u;  // the bucket's last key is below x
        }
    } else {
        const K *keys = A.k + base;
        auto runs = [&](auto full) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                uint32_t below;
                run_all<K, kRunLanes, decltype(full)::value>(keys, have, rel[r], x[r], below, hit[r]);
                rel[r] += below;
            }
        };
        if (have >= P.step) runs(std::true_type{});  // workgroup-uniform
        else runs(std::false_type{});
    }
}

// The bucket of partitioned position p: the last b with starts[b] <= p.
__device__ __forceinline__ uint32_t bucket_at(const uint32_t *__restrict__ starts, uint32_t NB, uint32_t p) {
    uint32_t lo = 0, hi = NB;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (starts[mid] <= p) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Calls body(b, p0, p1) for the pieces [p0, p1) of this workgroup's span, one
// bucket each (workgroup-uniform).
template <typename Body>
__device__ __forceinline__ void for_pieces(uint64_t m, const uint32_t *__restrict__ starts, uint32_t NB, uint64_t spans,
                                           Body &&body) {
    const uint64_t sp = tile_of(blockIdx.x, spans, 1);
    if (sp >= spans) return;
    uint32_t p0 = (uint32_t)(sp * kSpan);
    const uint32_t end = m - sp * kSpan < kSpan ? (uint32_t)m : p0 + kSpan;
    uint32_t b = bucket_at(starts, NB, p0);
    while (p0 < end) {
        while (starts[b + 1] <= p0) ++b;
        const uint32_t p1 = starts[b + 1] < end ? starts[b + 1] : end;
        body(b, p0, p1);
        p0 = p1;
    }
}

template <typename K, bool AOS>
__global__ __launch_bounds__(kLookThreads, 8) void k_part_bs(Load<K, AOS> A, uint64_t n, const K *__restrict__ q,
                                                             uint64_t m, const uint32_t *__restrict__ starts,
                                                             PartGeo P, const K *__restrict__ tab, uint64_t spans,
                                                             uint32_t *__restrict__ ans) {
    extern __shared__ __align__(16) char smem[];
    K *s_tab = (K *)smem;
    constexpr int R = kLookPer;
    for_pieces(m, starts, P.NB, spans, [&](uint32_t b, uint32_t p0, uint32_t p1) {
        K x[R];  // a piece is at most one round of the workgroup's queries
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t i = p0 + (uint32_t)r * kLookThreads + threadIdx.x;
            x[r] = q[i < p1 ? i : p0];
        }
        fill_table(tab, b, P.L, s_tab);
        __syncthreads();
        uint32_t rel[R];
        table_find<K, R>(s_tab, P, x, rel);
        bool hit[R];
        const uint64_t base = b * P.step;
        settle<K, AOS, R>(A, n, base, P, x, rel, hit);
        uint32_t res[R];
#pragma unroll
        for (int r = 0; r < R; ++r) res[r] = hit[r] ? A.row(base + rel[r]) : kMiss;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t i = p0 + (uint32_t)r * kLookThreads + threadIdx.x;
            if (i < p1) ans[i] = res[r];
        }
        __syncthreads();
    });
}

// Binary Eytzinger layout: bucket b is the subtree of slot NB + b (1-based),
// whose next L full levels are the table; the descent goes on from there.
template <typename K, bool AOS>
__global__ __launch_bounds__(kLookThreads) void k_part_ebs(Load<K, AOS> A, uint64_t n, uint32_t m_full,
                                                           const K *__restrict__ q, uint64_t m,
                                                           const uint32_t *__restrict__ starts, PartGeo P,
                                                           uint64_t spans, uint32_t *__restrict__ ans) {
    extern __shared__ __align__(16) char smem[];
    K *s_tab = (K *)smem;
    const uint32_t L = P.L;
    for_pieces(m, starts, P.NB, spans, [&](uint32_t b, uint32_t p0, uint32_t p1) {
        const uint64_t root = (uint64_t)P.NB + b;
        for (uint32_t v = 1 + threadIdx.x; v < (1u << L); v += kLookThreads) {
            const uint32_t l = 31u - (uint32_t)__clz((int)v);
            s_tab[v] = A.key((root << l) + (v - (1u << l)));
        }
        __syncthreads();
        for (uint32_t t = p0 + threadIdx.x; t < p1; t += kLookThreads * kLookPer) {
            K x[kLookPer], ck[kLookPer];
            uint64_t i[kLookPer];
            {
                uint32_t v[kLookPer];
#pragma unroll
                for (int r = 0; r < kLookPer; ++r) {
                    const uint32_t at = t + (uint32_t)r * kLookThreads;
                    x[r] = q[at < p1 ? at : t];
                    v[r] = 1;
                    ck[r] = key_max_v<K>();
                }
                for (uint32_t l = 0; l < L; ++l) {
#pragma unroll
                    for (int r = 0; r < kLookPer; ++r) {
                        const K k = s_tab[v[r]];
                        const bool right = k < x[r];
                        ck[r] = right ? ck[r] : k;
                        v[r] = 2 * v[r] + (right ? 1u : 0u);
                    }
                }
#pragma unroll
                for (int r = 0; r < kLookPer; ++r) i[r] = (root << L) + (v[r] - (1u << L));
            }
            for (uint32_t l = P.top + L; l < m_full; ++l) {
#pragma unroll
                for (int r = 0; r < kLookPer; ++r) {
                    const K k = A.key(i[r]);
                    const bool right = k < x[r];
                    ck[r] = right ? ck[r] : k;
                    i[r] = 2 * i[r] + (right ? 1 : 0);
                }
            }
            uint32_t res[kLookPer];
#pragma unroll
            for (int r = 0; r < kLookPer; ++r) {
                if (i[r] <= n) {
                    const K k = A.key(i[r]);
                    const bool right = k < x[r];
                    ck[r] = right ? ck[r] : k;
                    i[r] = 2 * i[r] + (right ? 1 : 0);
                }
                const uint64_t j = i[r] >> (__builtin_ctzll(~i[r]) + 1);
                if (j != 0 && j < P.NB) ck[r] = A.key(j);  // the lower bound lies above the bucket
                res[r] = (j != 0 && ck[r] == x[r]) ? A.row(j) : kMiss;
            }
#pragma unroll
            for (int r = 0; r < kLookPer; ++r) {
                const uint32_t at = t + (uint32_t)r * kLookThreads;
                if (at < p1) ans[at] = res[r];
            }
        }
        __syncthreads();
    });
}

// k-ary Eytzinger layout of nodes of 16 * NL bytes: the bucket's table, then the
// nodes below it (one, unless the tree is too large for that), each read by NL
// lanes with one load.  Bound by L2 requests and vector work like k_part_bs.
// Per 2^27 lookups at n = 2^26, k = 9, 64-bit keys: 1.53 ms (with whole subtrees
// for buckets, the left ones larger than the L2 and two nodes below the table,
// 2.48), 3.3 ms with the partition; a walk over all levels of the batch as it
// comes takes 9.3.
template <typename K, uint32_t NL>
__global__ __launch_bounds__(kLookThreads, 8) void k_part_eks(Load<K, false> A, Geo G, const K *__restrict__ q,
                                                              uint64_t m, const uint32_t *__restrict__ starts,
                                                              PartGeo P, const K *__restrict__ tab,
                                                              const uint32_t *__restrict__ rows, uint64_t spans,
                                                              uint32_t *__restrict__ ans) {
    extern __shared__ __align__(16) char smem[];
    K *s_tab = (K *)smem;
    constexpr int R = kLookPer;
    constexpr uint32_t g = NL * 16 / sizeof(K);
    for_pieces(m, starts, P.NB, spans, [&](uint32_t b, uint32_t p0, uint32_t p1) {
        K x[R];  // a piece is at most one round of the workgroup's queries
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t i = p0 + (uint32_t)r * kLookThreads + threadIdx.x;
            x[r] = q[i < p1 ? i : p0];
        }
        fill_table(tab, b, P.L, s_tab);
        __syncthreads();
        uint32_t cut, j0, j1;
        bucket_nodes(P, b, cut, j0, j1);
        uint32_t c[R], res[R];  // node on the level, counted from the bucket's first; answer
        table_count<K, R>(s_tab, P.L, x, c);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t e = (uint32_t)__builtin_ctz(c[r] + 1), v = (1u << (P.L - 1 - e)) + (c[r] >> (e + 1));
            const bool real = j0 + c[r] < G.start[cut];  // (c < j1 - j0: the splitter is not below x)
            res[r] = kMiss;
            if (real && s_tab[v] == x[r]) res[r] = rows[(b << P.L) + v];  // NB << L < 2^24
        }
        uint64_t first = (uint64_t)j0 * g, width = (uint64_t)(j1 - j0) * g;  // the bucket's keys on the level
        for (uint32_t l = cut; l < G.levels; ++l, first *= G.k, width *= G.k) {
            const uint64_t base = G.start[l] + first;
            if (base >= G.n) break;  // workgroup-uniform
            const uint32_t have = G.n - base < width ? (uint32_t)(G.n - base) : (uint32_t)width;
            const K *keys = A.k + base;
            const uint32_t *ids = A.r + base;
            auto nodes = [&](auto full) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const bool in = c[r] < (have + g - 1) / g;
                    const uint32_t at = in ? c[r] * g : 0u;
                    uint32_t below;
                    bool equal;
                    run_all<K, NL, decltype(full)::value>(keys, have, at, x[r], below, equal);
                    if (in && equal) res[r] = ids[at + below];
                    c[r] = in ? c[r] * G.k + below : ~0u;
                }
            };
            if (have == width) nodes(std::true_type{});  // workgroup-uniform
            else nodes(std::false_type{});
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t i = p0 + (uint32_t)r * kLookThreads + threadIdx.x;
            if (i < p1) ans[i] = res[r];
        }
        __syncthreads();
    });
}

// Both ranks of every range on the sorted array, as one packed word (first
// rank << 32 | count) in partitioned order.  The range's lower bound names
// the bucket; an upper bound past the bucket is searched in the rest of the
// array.
template <typename K, bool AOS>
__global__ __launch_bounds__(kLookThreads, 8) void k_part_range_bs(Load<K, AOS> A, uint64_t n,
                                                                   const K *__restrict__ q, const K *__restrict__ q_hi,
                                                                   uint64_t m, const uint32_t *__restrict__ starts,
                                                                   PartGeo P, const K *__restrict__ tab, uint64_t spans,
                                                                   uint64_t *__restrict__ packed) {
    extern __shared__ __align__(16) char smem[];
    K *s_tab = (K *)smem;
    constexpr int R = 4;  // bounds: two ranges per lane at once
    for_pieces(m, starts, P.NB, spans, [&](uint32_t b, uint32_t p0, uint32_t p1) {
        fill_table(tab, b, P.L, s_tab);
        __syncthreads();
        const uint64_t base = b * P.step;
        for (uint32_t t0 = p0; t0 < p1; t0 += kLookThreads * (R / 2)) {
            K x[R];
            bool empty[R / 2], all[R / 2];
#pragma unroll
            for (int r = 0; r < R / 2; ++r) {
                const uint32_t i = t0 + (uint32_t)r * kLookThreads + threadIdx.x, at = i < p1 ? i : p0;
                const K l = q[at], u = q_hi[at];
                empty[r] = l > u;
                all[r] = u == key_max_v<K>();  // nothing is above u
                x[2 * r] = l;
                x[2 * r + 1] = all[r] ? u : (K)(u + 1);
            }
            uint32_t rel[R];
            table_find<K, R>(s_tab, P, x, rel);
            bool hit[R];
            settle<K, AOS, R>(A, n, base, P, x, rel, hit);
#pragma unroll
            for (int r = 0; r < R / 2; ++r) {
                const uint32_t i = t0 + (uint32_t)r * kLookThreads + threadIdx.x;
                uint64_t r1 = base + rel[2 * r + 1];
                if (rel[2 * r + 1] == P.step && !empty[r] && !all[r]) {  // past the bucket
                    uint64_t len = n - r1;
                    while (len) {
                        const uint64_t half = len >> 1;
                        if (A.key(r1 + half) < x[2 * r + 1]) {
                            r1 += half + 1;
                            len -= half + 1;
                        } else {
                            len = half;
                        }
                    }
                }
                if (all[r]) r1 = n;
                const uint64_t r0 = base + rel[2 * r];
                if (i < p1) packed[i] = empty[r] ? 0ull : (r0 << 32) | (r1 > r0 ? r1 - r0 : 0ull);
            }
        }
        __syncthreads();
    });
}

// Buckets of the k-ary Eytzinger layout.  Cut just above the last level: the
// nodes of the partial level, then those of the last full one past it, 2^13 - 1
// to a bucket, leave one node to read below the table.  When that makes more
// than kMaxBuckets, or few queries per bucket or table entry, the cut goes up,
// level by level.
void eks_geo(const Geo &G, uint64_t m, PartGeo &P) {
    P.NB = 1;
    if (G.m < 2) return;
    uint64_t gaps[kMaxLevels];  // k^c, the nodes of full level c
    gaps[0] = 1;
    for (uint32_t c = 1; c < G.m; ++c) gaps[c] = gaps[c - 1] * G.k;
    const uint64_t nodes = (G.b + G.g - 1) / G.g;  // of the partial level
    auto plan = [&](uint32_t cr, bool two, uint32_t L) -> uint64_t {
        const uint64_t E = (1ull << L) - 1, over = two ? (nodes + G.k - 1) / G.k : 0;
        P.L = L;
        P.entries = (uint32_t)E;
        P.cut_l = cr + 1;
        P.cut_r = cr;
        P.gaps = (uint32_t)gaps[cr];
        P.right = (uint32_t)over;
        P.left = (uint32_t)(over * G.k);
        P.NB_l = (uint32_t)((over * G.k + E - 1) / E);
        return P.NB_l + (gaps[cr] - over + E - 1) / E;
    };
    uint32_t cr = G.m - 1;
    bool two = nodes > 0;
    uint64_t NB;
    for (;;) {
        const uint64_t all = gaps[cr] + (two ? nodes : 0);  // table entries in all
        NB = all < (1ull << 32) ? plan(cr, two, kMaxLevels1) : ~0ull;
        if (NB <= kMaxBuckets && NB * kBucketQueries <= m && all <= 8 * m) break;
        if (two) two = false;
        else if (cr > 1) --cr;
        else return;
    }
    while (NB < 8 && P.L > kMinLevels) NB = plan(cr, two, P.L - 1);
    P.NB = (uint32_t)NB;
}

// The buckets of a batch of m queries: at most kMaxBuckets, no fewer than
// kBucketQueries queries each on average (they share the cost of the
// bucket's table), and otherwise as small as a table of up to 13 levels over
// whole lines makes them: 1.5 MiB of 64-bit keys and row IDs, 2 MiB of 32-bit
// ones (an XCD's L2 holds the one or two in flight).  Small sets get shorter
// tables, for eight buckets or more.
PartGeo bucket_geo(const idx_index *h, uint64_t m) {
    PartGeo P{};
    P.NB = 1;
    if (h->n < 4) return P;
    if (h->layout == IDX_BS) {
        P.L = kMaxLevels1;
        P.D = h->u64 ? run_log<uint64_t>() : run_log<uint32_t>();
        auto buckets = [&] { return (h->n + (1ull << (P.L + P.D)) - 1) >> (P.L + P.D); };
        while (P.L > kMinLevels && buckets() < 8) --P.L;
        // (few queries: larger buckets, of 2^26 ranks at most, whose byte offsets fit 32 bits)
        while (buckets() > kMaxBuckets || (buckets() > 2 && buckets() * kBucketQueries > m && P.L + P.D < 26)) ++P.D;
        while (P.L > kMinLevels && (1ull << P.L) * buckets() > 8 * m) {  // few queries per bucket: shorter tables
            --P.L;
            ++P.D;
        }
        P.step = 1ull << (P.L + P.D);
        P.NB = (uint32_t)buckets();
        return P;
    }
    if (h->layout == IDX_EKS) {
        eks_geo(h->geo, m, P);
        return P;
    }
    const uint64_t bytes = h->n * ((h->u64 ? 8 : 4) + 4);
    uint32_t want = 2;
    while (want < kMaxBuckets && want * kBucketBytes < bytes) want <<= 1;
    while (want > 2 && (want * kBucketQueries > m || want > h->n / 2)) want >>= 1;
    while (P.top < h->geo.m && P.NB * h->geo.k <= want) {
        P.NB *= h->geo.k;
        ++P.top;
    }
    P.L = kMaxLevels1;
    while (P.L > kMinLevels && (1ull << P.L) * P.NB > 8 * m) --P.L;
    if (P.L > h->geo.m - P.top) P.L = h->geo.m - P.top;
    return P;
}

PartGeo part_geo(const idx_index *h, uint64_t m, Search search) {
    PartGeo P = bucket_geo(h, m);
    if (search == Search::sorted_tables || search == Search::node_tables) P.tab = (uint64_t)P.NB << P.L;
    return P;
}

size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

uint64_t part_tiles(uint64_t m) { return (m + kPartTile - 1) / kPartTile; }

// Scratch of one chunk of m queries (256-byte aligned regions).
struct PartBufs {
    void *q2, *q2_hi;   // queries (and upper bounds) in partitioned order
    uint16_t *place;    // place of every query within its tile, in bucket order
    void *ans;          // answers in partitioned order: u32, or u64 for ranges
    uint32_t *hist;     // NB x tiles
    uint32_t *total;    // NB
    uint32_t *starts;   // NB + 1
    void *split;        // NB keys
    void *tab;          // the buckets' tables, if any: NB << L keys
    uint32_t *rows;     // their row IDs (k-ary Eytzinger layout)
};

// Row IDs of the tables' entries (k-ary Eytzinger layout).
size_t row_entries(const PartGeo &P) { return P.entries ? P.tab : 0; }

size_t part_bytes(uint64_t m, size_t kb, const PartGeo &P, bool range) {
    const uint32_t NB = P.NB;
    return up256(m * kb) * (range ? 2 : 1) + up256(m * 2) + up256(m * (range ? 8 : 4)) +
           up256((size_t)NB * part_tiles(m) * 4) + up256((size_t)NB * 4) + up256(((size_t)NB + 1) * 4) +
           up256((size_t)NB * kb) + up256(P.tab * kb) + up256(row_entries(P) * 4);
}

PartBufs carve(char *t, uint64_t m, size_t kb, const PartGeo &P, bool range) {
    const uint32_t NB = P.NB;
    PartBufs p{};
    auto take = [&](size_t b) {
        char *r = t;
        t += up256(b);
        return r;
    };
    p.q2 = take(m * kb);
    p.q2_hi = range ? take(m * kb) : nullptr;
    p.place = (uint16_t *)take(m * 2);
    p.ans = take(m * (range ? 8 : 4));
    p.hist = (uint32_t *)take((size_t)NB * part_tiles(m) * 4);
    p.total = (uint32_t *)take((size_t)NB * 4);
    p.starts = (uint32_t *)take(((size_t)NB + 1) * 4);
    p.split = take((size_t)NB * kb);
    p.tab = take(P.tab * kb);
    p.rows = (uint32_t *)take(row_entries(P) * 4);
    return p;
}

// Steps 1-4.
template <typename K, bool AOS>
int partition_t(idx_index *h, const K *q, const K *q_hi, uint64_t m, const PartGeo &P, const PartBufs &B,
                hipStream_t s) {
    const Load<K, AOS> A = make_load<K, AOS>(h);
    const uint32_t NB = P.NB;
    if (h->layout == IDX_BS)
        hipLaunchKernelGGL((k_split_sorted<K, AOS>), dim3((NB + 255) / 256), dim3(256), 0, s, A, P.step, NB,
                           (K *)B.split);
    else
        hipLaunchKernelGGL((k_split_eyt<K, AOS>), dim3((NB + 255) / 256), dim3(256), 0, s, A, h->geo,
                           (uint64_t)(h->layout == IDX_EBS ? 1 : 0), P, (K *)B.split);
    IDX_LAUNCH_CHECK();
    const uint32_t tiles = (uint32_t)part_tiles(m);
    const uint32_t iters = (tiles + kXcds - 1) / kXcds * kXcds;
    const uint32_t cus = (uint32_t)h->cu_count / kXcds * kXcds;  // a multiple of the XCDs: workgroups keep their share
    const uint32_t one = cus ? cus : kXcds, two = 2 * one;
    hipLaunchKernelGGL((k_part_count<K>), dim3(iters < two ? iters : two), dim3(kPartThreads),
                       (size_t)NB * (sizeof(K) + 4) + kCellBytes, s, q, m, (const K *)B.split, NB, tiles, iters, B.hist);
    IDX_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_part_scan, dim3(NB), dim3(kScanThreads), 0, s, B.hist, tiles, B.total);
    IDX_LAUNCH_CHECK();
    const size_t lds = scatter_lds_bytes<K>(NB);
    const dim3 grid(iters < one ? iters : one);
    if (q_hi)
        hipLaunchKernelGGL((k_part_scatter<K, true>), grid, dim3(kPartThreads), lds, s, q, q_hi, m, (const K *)B.split,
                           NB, tiles, iters, B.hist, B.total, (K *)B.q2, (K *)B.q2_hi, B.place, B.starts);
    else
        hipLaunchKernelGGL((k_part_scatter<K, false>), grid, dim3(kPartThreads), lds, s, q, (const K *)nullptr, m,
                           (const K *)B.split, NB, tiles, iters, B.hist, B.total, (K *)B.q2, (K *)nullptr, B.place,
                           B.starts);
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

template <typename K, bool AOS>
int build_tables(const idx_index *h, const PartGeo &P, const PartBufs &B, hipStream_t s) {
    hipLaunchKernelGGL((k_part_tables<K, AOS>), dim3((uint32_t)((P.tab + 255) / 256)), dim3(256), 0, s,
                       make_load<K, AOS>(h), h->n, P, (K *)B.tab);
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

// Step 6.
template <typename T>
int gather(const idx_index *h, const PartBufs &B, uint64_t m, uint32_t NB, const T *ans, T *out, hipStream_t s) {
    const uint32_t tiles = (uint32_t)part_tiles(m), iters = (tiles + kXcds - 1) / kXcds * kXcds;
    const uint32_t cus = (uint32_t)h->cu_count / kXcds * kXcds, two = 2 * (cus ? cus : kXcds);
    hipLaunchKernelGGL(k_part_gather<T>, dim3(iters < two ? iters : two), dim3(kPartThreads), 0, s, ans,
                       (const uint16_t *)B.place, m, NB, tiles, iters, (const uint32_t *)B.hist,
                       (const uint32_t *)B.total, (const uint32_t *)B.starts, out);
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

uint64_t spans_of(uint64_t m) { return (m + kSpan - 1) / kSpan; }
dim3 span_grid(uint64_t spans) { return dim3((uint32_t)((spans + kXcds - 1) / kXcds * kXcds)); }

template <typename K, bool AOS>
int chunk_t(idx_index *h, const K *q, uint64_t m, uint32_t *out, const PartGeo &P, const PartBufs &B, hipStream_t s) {
    int rc = partition_t<K, AOS>(h, q, (const K *)nullptr, m, P, B, s);
    if (rc != IDX_OK) return rc;
    const uint64_t spans = spans_of(m);
    const Search search = point_search(h);
    uint32_t *ans = (uint32_t *)B.ans;
    if (search == Search::sorted_tables) {
        rc = build_tables<K, AOS>(h, P, B, s);
        if (rc != IDX_OK) return rc;
        hipLaunchKernelGGL((k_part_bs<K, AOS>), span_grid(spans), dim3(kLookThreads), sizeof(K) << P.L, s,
                           make_load<K, AOS>(h), h->n, (const K *)B.q2, m, B.starts, P, (const K *)B.tab, spans, ans);
        IDX_LAUNCH_CHECK();
    } else if (search == Search::subtrees) {
        hipLaunchKernelGGL((k_part_ebs<K, AOS>), span_grid(spans), dim3(kLookThreads), sizeof(K) << P.L, s,
                           make_load<K, AOS>(h), h->n, h->geo.m, (const K *)B.q2, m, B.starts, P, spans, ans);
        IDX_LAUNCH_CHECK();
    } else if (search == Search::node_tables) {  // (keys and row IDs apart)
        const Load<K, false> A = make_load<K, false>(h);
        hipLaunchKernelGGL(k_part_tables_eks<K>, dim3((uint32_t)((P.tab + 255) / 256)), dim3(256), 0, s, A, h->geo, P,
                           (K *)B.tab, B.rows);
        IDX_LAUNCH_CHECK();
        auto look = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, span_grid(spans), dim3(kLookThreads), sizeof(K) << P.L, s, A, h->geo,
                               (const K *)B.q2, m, B.starts, P, (const K *)B.tab, (const uint32_t *)B.rows, spans, ans);
        };
        switch (h->geo.g * sizeof(K)) {
            case 32: look(k_part_eks<K, 2>); break;
            case 64: look(k_part_eks<K, 4>); break;
            default: look(k_part_eks<K, 8>); break;
        }
        IDX_LAUNCH_CHECK();
    } else {  // the handle's own lookup kernel over the partitioned batch
        rc = point_run(h, PointIO{B.q2, m, ans, false, true}, s);
        if (rc != IDX_OK) return rc;
    }
    return gather(h, B, m, P.NB, (const uint32_t *)ans, out, s);
}

template <typename K, bool AOS>
int range_chunk_t(idx_index *h, const K *lo, const K *hi, uint64_t m, const PartGeo &P, char *scratch, RangePart *out,
                  hipStream_t s) {
    const PartBufs B = carve(scratch, m, sizeof(K), P, true);
    int rc = partition_t<K, AOS>(h, lo, hi, m, P, B, s);
    if (rc != IDX_OK) return rc;
    out->lo = B.q2;
    out->hi = B.q2_hi;
    out->packed = (uint64_t *)B.ans;
    out->counted = range_search(h) == Search::sorted_tables;
    if (!out->counted) return IDX_OK;
    rc = build_tables<K, AOS>(h, P, B, s);
    if (rc != IDX_OK) return rc;
    const uint64_t spans = spans_of(m);
    hipLaunchKernelGGL((k_part_range_bs<K, AOS>), span_grid(spans), dim3(kLookThreads), sizeof(K) << P.L, s,
                       make_load<K, AOS>(h), h->n, (const K *)B.q2, (const K *)B.q2_hi, m, B.starts, P,
                       (const K *)B.tab, spans, out->packed);
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

}  // namespace

// ---- the partition for range counts
bool range_partition_pays(const idx_index *h, uint64_t m) {
    return m >= range_part_min(h) && part_geo(h, m, range_search(h)).NB > 1;
}

size_t range_partition_bytes(const idx_index *h, uint64_t m) {
    return part_bytes(m, h->u64 ? 8 : 4, part_geo(h, m, range_search(h)), true);
}

int range_partition(idx_index *h, const void *lo, const void *hi, uint64_t m, void *scratch, RangePart *out,
                    hipStream_t s) {
    if (m == 0 || m > kPartChunk) return IDX_ERR_ARG;
    const PartGeo P = part_geo(h, m, range_search(h));
    char *t = (char *)scratch;
    if (h->u64)
        return h->aos ? range_chunk_t<uint64_t, true>(h, (const uint64_t *)lo, (const uint64_t *)hi, m, P, t, out, s)
                      : range_chunk_t<uint64_t, false>(h, (const uint64_t *)lo, (const uint64_t *)hi, m, P, t, out, s);
    return h->aos ? range_chunk_t<uint32_t, true>(h, (const uint32_t *)lo, (const uint32_t *)hi, m, P, t, out, s)
                  : range_chunk_t<uint32_t, false>(h, (const uint32_t *)lo, (const uint32_t *)hi, m, P, t, out, s);
}

int range_partition_back(const idx_index *h, const RangePart &v, void *scratch, uint64_t m, uint64_t *packed,
                         hipStream_t s) {
    const PartGeo P = part_geo(h, m, range_search(h));
    const PartBufs B = carve((char *)scratch, m, h->u64 ? 8 : 4, P, true);
    return gather(h, B, m, P.NB, (const uint64_t *)v.packed, packed, s);
}

int point_partitioned(idx_index *h, const void *q, uint64_t m, uint32_t *out, hipStream_t s) {
    const uint64_t chunk = m < kPartChunk ? m : kPartChunk;
    const PartGeo P = part_geo(h, chunk, point_search(h));
    if (m < part_min(h) || P.NB == 1) return point_run(h, PointIO{q, m, out, false, false}, s);
    const size_t kb = h->u64 ? 8 : 4;
    char *tmp = (char *)h->alloc.get(part_bytes(chunk, kb, P, false), s);
    if (!tmp) return point_run(h, PointIO{q, m, out, false, false}, s);  // the same answers, without scratch
    int rc = IDX_OK;
    for (uint64_t c0 = 0; c0 < m && rc == IDX_OK; c0 += chunk) {
        const uint64_t mc = (m - c0) < chunk ? (m - c0) : chunk;
        const PartBufs B = carve(tmp, mc, kb, P, false);
        // places of this chunk are relative to its own start
        if (h->u64)
            rc = h->aos ? chunk_t<uint64_t, true>(h, (const uint64_t *)q + c0, mc, out + c0, P, B, s)
                        : chunk_t<uint64_t, false>(h, (const uint64_t *)q + c0, mc, out + c0, P, B, s);
        else
            rc = h->aos ? chunk_t<uint32_t, true>(h, (const uint32_t *)q + c0, mc, out + c0, P, B, s)
                        : chunk_t<uint32_t, false>(h, (const uint32_t *)q + c0, mc, out + c0, P, B, s);
    }
    h->alloc.put(tmp, s);
    return rc;
}

}  // namespace idx
