// Stable sort of (key, rowid) pairs by key -- the build step of the
// sorted-array index (Section 3: BS is a key-value sort; Section 8.5: the
// sort dominates build time).  gfx950, wave64.
//
// Two forms, chosen by the keys' distribution:
//
//  buckets  The pairs are first ordered by their top hb <= 16 varying bits
//           with one or two stable radix passes, into buckets of about 1 K
//           pairs; then each workgroup takes a few whole buckets into LDS and
//           finishes them there (k_bucket_sort).  Every pair moves three
//           times instead of once per key byte.  Buckets are cut from the key
//           itself or, when a sample spreads better that way (clustered,
//           lognormal-like keys), from a float-like code of it.  An exact
//           histogram of the buckets decides: a set with a bucket too large
//           for LDS (few distinct or very skewed keys) takes the other form.
//  LSD      One stable pass per 8-bit digit that varies.
//
// A radix pass is three kernels (reduce-then-scan; no inter-workgroup waiting
// anywhere):
//   1. tile histogram: each workgroup counts the digits of its 4096-key tile;
//   2. digit scan: one workgroup per digit turns the per-tile counts into
//      exclusive offsets and a digit total;
//   3. scatter: each workgroup ranks its tile stably (wave-level ballot
//      "peer" masks, items taken in index order), stages the tile in LDS in
//      digit order and writes every digit run out contiguously.
// What bounds it: memory.  2^26 64-bit keys move 88 B each through the
// bucket form (histogram 8, two passes of 8 + 24, buckets 24) against 256 B
// through eight LSD passes.
#include "internal.hpp"
#include "learned_model.hpp"

namespace idx {
namespace {

constexpr int RS_BITS = 8;
constexpr int RS_BINS = 1 << RS_BITS;
constexpr int RS_THREADS = 256;
constexpr int RS_WAVES = RS_THREADS / kWave;
constexpr int RS_ITEMS = 16;
constexpr int RS_TILE = RS_THREADS * RS_ITEMS;  // 4096 keys
constexpr int RS_SCAN_ITEMS = 16;
constexpr uint32_t RS_XCDS = 8;  // workgroups are dealt round-robin over the 8 XCDs

// The tile that workgroup b scatters: XCD x (b % 8) takes a contiguous share
// of the tiles, in order.  A digit's runs from consecutive tiles are adjacent
// in the output, so the partial 128 B lines at their ends are completed in
// one XCD's L2 instead of being written back in pieces from several.
// A bijection of [0, tiles): XCD x holds tiles/8 + (x < tiles%8) workgroups.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t tiles) {
    const uint32_t per = tiles / RS_XCDS, rem = tiles % RS_XCDS;
    const uint32_t x = b % RS_XCDS, i = b / RS_XCDS;
    return x * per + (x < rem ? x : rem) + i;
}

static_assert(RS_THREADS == RS_BINS, "one thread per digit value in the scan phases");

// Exclusive scan of one value per thread across a 256-thread workgroup.
// Returns the exclusive prefix; *total receives the workgroup sum.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *s_wave, uint32_t *total) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = threadIdx.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, kWave);
        if (lane >= (uint32_t)off) incl += t;
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) {
        const uint32_t c = s_wave[w];
        before += (w < (int)wave) ? c : 0;
        sum += c;
    }
    __syncthreads();
    *total = sum;
    return before + incl - v;
}

template <typename K>
__global__ __launch_bounds__(RS_THREADS) void k_global_hist(const K *__restrict__ keys, uint64_t n, int passes,
                                                            uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[8 * RS_BINS];
    for (int i = threadIdx.x; i < passes * RS_BINS; i += RS_THREADS) h[i] = 0;
    __syncthreads();
    for (uint64_t i = (uint64_t)blockIdx.x * RS_THREADS + threadIdx.x; i < n; i += (uint64_t)gridDim.x * RS_THREADS) {
        const K key = keys[i];
        for (int p = 0; p < passes; ++p) atomicAdd(&h[p * RS_BINS + ((key >> (p * RS_BITS)) & (RS_BINS - 1))], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < passes * RS_BINS; i += RS_THREADS)
        if (h[i]) atomicAdd(&hist[i], h[i]);
}

// The code whose bits the passes sort by: the key, or (LOG) floor(log2 key)
// in bits 58-63 and the 58 bits below the key's leading one.  Both are
// non-decreasing in the key; the first is the key itself.
template <bool LOG, typename K>
__device__ __forceinline__ uint64_t sort_code(K key) {
    if constexpr (LOG) return bin_feature((uint64_t)key, IDX_FEATURE_LOG);
    else return (uint64_t)key;
}

template <bool LOG, typename K>
__device__ __forceinline__ uint32_t digit_of(K key, int shift, uint32_t mask) {
    if constexpr (LOG) return (uint32_t)(sort_code<true>(key) >> shift) & mask;
    else return (uint32_t)(key >> shift) & mask;
}

template <typename K, bool LOG>
__global__ __launch_bounds__(RS_THREADS) void k_tile_hist(const K *__restrict__ keys, uint64_t n, int shift,
                                                          uint32_t mask, uint32_t *__restrict__ tile_hist,
                                                          uint32_t tiles) {
    __shared__ uint32_t h[RS_WAVES][RS_BINS];
    const uint32_t wave = threadIdx.x / kWave;
    for (int w = 0; w < RS_WAVES; ++w) h[w][threadIdx.x] = 0;
    __syncthreads();
    // XCD-contiguous tiles, as in the scatter: the per-digit counts of
    // neighbouring tiles share lines of tile_hist.
    const uint32_t tile = xcd_tile(blockIdx.x, tiles);
    const uint64_t base = (uint64_t)tile * RS_TILE;
    // all of a thread's keys are loaded before the first LDS atomic, so the
    // 16 loads are in flight together
    K kk[RS_ITEMS];
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const uint64_t i = base + (uint64_t)j * RS_THREADS + threadIdx.x;
        kk[j] = i < n ? keys[i] : K(0);
    }
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const uint64_t i = base + (uint64_t)j * RS_THREADS + threadIdx.x;
        if (i < n) atomicAdd(&h[wave][digit_of<LOG>(kk[j], shift, mask)], 1u);
    }
    __syncthreads();
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) c += h[w][threadIdx.x];
    tile_hist[(uint64_t)threadIdx.x * tiles + tile] = c;
}

// One workgroup per digit: exclusive scan of that digit's per-tile counts
// (in place) and the digit's total.
__global__ __launch_bounds__(RS_THREADS) void k_digit_scan(uint32_t *__restrict__ tile_hist, uint32_t tiles,
                                                           uint32_t *__restrict__ digit_total) {
    __shared__ uint32_t s_wave[RS_WAVES];
    uint32_t *row = tile_hist + (uint64_t)blockIdx.x * tiles;
    uint32_t running = 0;
    for (uint32_t chunk = 0; chunk < tiles; chunk += RS_THREADS * RS_SCAN_ITEMS) {
        uint32_t v[RS_SCAN_ITEMS];
        uint32_t sum = 0;
        const uint32_t first = chunk + threadIdx.x * RS_SCAN_ITEMS;
#pragma unroll
        for (int j = 0; j < RS_SCAN_ITEMS; ++j) {
            v[j] = (first + j < tiles) ? row[first + j] : 0u;
            sum += v[j];
        }
        uint32_t total;
        uint32_t acc = running + block_exclusive_scan(sum, s_wave, &total);
#pragma unroll
        for (int j = 0; j < RS_SCAN_ITEMS; ++j) {
            if (first + j < tiles) row[first + j] = acc;
            acc += v[j];
        }
        running += total;
    }
    if (threadIdx.x == 0) digit_total[blockIdx.x] = running;
}

template <typename K>
struct ScatterSmem {
    K keys[RS_TILE];
    uint32_t rows[RS_TILE];
    uint32_t wave_cnt[RS_WAVES][RS_BINS];
    uint32_t digit_start[RS_BINS];
    uint32_t global_base[RS_BINS];
    uint32_t scan_tmp[RS_WAVES];
};

template <typename K, bool LOG>
__global__ __launch_bounds__(RS_THREADS) void k_scatter(const K *__restrict__ keys_in,
                                                        const uint32_t *__restrict__ rows_in,
                                                        K *__restrict__ keys_out, uint32_t *__restrict__ rows_out,
                                                        uint64_t n, int shift, uint32_t mask,
                                                        const uint32_t *__restrict__ tile_hist, uint32_t tiles,
                                                        const uint32_t *__restrict__ digit_total) {
    __shared__ ScatterSmem<K> sm;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = threadIdx.x / kWave;
    const uint64_t lt_mask = (1ull << lane) - 1ull;

    for (int w = 0; w < RS_WAVES; ++w) sm.wave_cnt[w][threadIdx.x] = 0;

    // Items of a wave are consecutive keys: item j of lane l is key
    // base + j*64 + l, so taking items j = 0, 1, ... with lanes in order
    // visits the wave's keys in index order (stability).
    const uint32_t tile = xcd_tile(blockIdx.x, tiles);
    const uint64_t tile_base = (uint64_t)tile * RS_TILE;
    const uint64_t wave_base = tile_base + (uint64_t)wave * (RS_ITEMS * kWave);
    K key[RS_ITEMS];
    uint32_t row[RS_ITEMS];
    uint32_t rank[RS_ITEMS];
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const uint64_t i = wave_base + (uint64_t)j * kWave + lane;
        const bool valid = i < n;
        key[j] = valid ? keys_in[i] : K(0);
        row[j] = valid ? rows_in[i] : 0u;
    }
    __syncthreads();

#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const uint64_t i = wave_base + (uint64_t)j * kWave + lane;
        const bool valid = i < n;
        const uint32_t d = digit_of<LOG>(key[j], shift, mask);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < RS_BITS; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
        const uint32_t before = sm.wave_cnt[wave][d];
        rank[j] = before + below;
        wave_lds_order();
        if (valid && below == 0) sm.wave_cnt[wave][d] = before + (uint32_t)__popcll(peers);
        wave_lds_order();
    }
    __syncthreads();

    // Per digit (thread = digit): offsets of each wave inside the tile's run
    // of that digit, then the digit runs' starts inside the tile.
    {
        const uint32_t d = threadIdx.x;
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) {
            const uint32_t c = sm.wave_cnt[w][d];
            sm.wave_cnt[w][d] = sum;
            sum += c;
        }
        uint32_t tile_total;
        const uint32_t start = block_exclusive_scan(sum, sm.scan_tmp, &tile_total);
        sm.digit_start[d] = start;
        uint32_t dig_total_all;
        const uint32_t dbase = block_exclusive_scan(digit_total[d], sm.scan_tmp, &dig_total_all);
        sm.global_base[d] = dbase + tile_hist[(uint64_t)d * tiles + tile];
    }
    __syncthreads();

#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const uint64_t i = wave_base + (uint64_t)j * kWave + lane;
        if (i < n) {
            const uint32_t d = digit_of<LOG>(key[j], shift, mask);
            const uint32_t pos = sm.digit_start[d] + sm.wave_cnt[wave][d] + rank[j];
            sm.keys[pos] = key[j];
            sm.rows[pos] = row[j];
        }
    }
    __syncthreads();

    const uint32_t valid_in_tile = (uint32_t)((n - tile_base) < (uint64_t)RS_TILE ? (n - tile_base) : RS_TILE);
#pragma unroll 4
    for (uint32_t p = threadIdx.x; p < valid_in_tile; p += RS_THREADS) {
        const K kk = sm.keys[p];
        const uint32_t d = digit_of<LOG>(kk, shift, mask);
        const uint64_t o = (uint64_t)sm.global_base[d] + (p - sm.digit_start[d]);
        keys_out[o] = kk;
        rows_out[o] = sm.rows[p];
    }
}

// ------------------------------------------------------------- bucket form

constexpr uint32_t BK_BITS = 16;       // at most 2^16 buckets: their 16-bit counters fill 128 KiB of LDS
constexpr uint32_t BK_AVG = 1024;      // pairs per bucket aimed at
constexpr uint32_t BK_HIST_THREADS = 1024;
constexpr uint32_t BK_HIST_GRID = 256; // one counting workgroup per compute unit
constexpr int BK_ITEMS = 8;            // pairs per thread of k_bucket_sort
constexpr uint32_t BK_SMALL = 512, BK_LARGE = 1024;  // its workgroup sizes: 4096 or 8192 pairs in LDS
constexpr uint32_t BK_BIN_MAX = 24;    // bins of more pairs are left to the radix passes in LDS

// What the bucket histogram found; read once by the host.
struct SortInfo {
    unsigned long long ors;  // OR of every key's code ^ the first key's
    uint32_t bits;           // code bits [0, bits) vary (as the sample has it)
    uint32_t log;            // buckets are cut from the float-like code
    uint32_t bad;            // a 16-bit counter overflowed
    uint32_t max_bucket;
};

__device__ __forceinline__ uint32_t bits_of(uint64_t v) { return v ? 64u - (uint32_t)__builtin_clzll(v) : 0u; }

// Bits of the code that name the bucket, of the `bits` that vary.
__host__ __device__ __forceinline__ uint32_t bucket_bits(uint32_t want, uint32_t bits) {
    return want < bits ? want : bits;
}

// Sample of 1024 keys: which code spreads them better over 256 buckets, and
// its varying bits.
template <typename K>
__global__ __launch_bounds__(RS_BINS) void k_sort_sample(const K *__restrict__ keys, uint64_t n, SortInfo *info) {
    __shared__ unsigned long long s_or[2];
    __shared__ uint32_t s_hist[2][RS_BINS], s_max[2];
    if (threadIdx.x < 2) {
        s_or[threadIdx.x] = 0;
        s_max[threadIdx.x] = 0;
    }
    s_hist[0][threadIdx.x] = s_hist[1][threadIdx.x] = 0;
    __syncthreads();
    const K k0 = keys[0];
    K k[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) k[u] = keys[(n * (threadIdx.x * 4 + u)) >> 10];  // n < 2^32
    uint64_t o0 = 0, o1 = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        o0 |= sort_code<false>(k[u]) ^ sort_code<false>(k0);
        o1 |= sort_code<true>(k[u]) ^ sort_code<true>(k0);
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        o0 |= (uint64_t)__shfl_xor((unsigned long long)o0, off, kWave);
        o1 |= (uint64_t)__shfl_xor((unsigned long long)o1, off, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicOr(&s_or[0], (unsigned long long)o0);
        atomicOr(&s_or[1], (unsigned long long)o1);
    }
    __syncthreads();
    const uint32_t b0 = bits_of(s_or[0]), b1 = bits_of(s_or[1]);
    const uint32_t sh0 = b0 > 8 ? b0 - 8 : 0, sh1 = b1 > 8 ? b1 - 8 : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        atomicAdd(&s_hist[0][(sort_code<false>(k[u]) >> sh0) & (RS_BINS - 1)], 1u);
        atomicAdd(&s_hist[1][(sort_code<true>(k[u]) >> sh1) & (RS_BINS - 1)], 1u);
    }
    __syncthreads();
    uint32_t m0 = s_hist[0][threadIdx.x], m1 = s_hist[1][threadIdx.x];
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        m0 = max(m0, (uint32_t)__shfl_xor(m0, off, kWave));
        m1 = max(m1, (uint32_t)__shfl_xor(m1, off, kWave));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicMax(&s_max[0], m0);
        atomicMax(&s_max[1], m1);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const bool log = 2 * s_max[1] < s_max[0];
        info->ors = 0;
        info->bits = log ? b1 : b0;
        info->log = log ? 1u : 0u;
        info->bad = 0;
        info->max_bucket = 0;
    }
}

// Bucket counts of a workgroup's share of the keys, two 16-bit counters per
// word, to its row of `partial` (2^want / 2 words).  A counter that overflows
// carries into its neighbour, which shows as a count sum short of the keys.
template <typename K, bool LOG>
__device__ __forceinline__ void bucket_hist(const K *__restrict__ keys, uint64_t n, uint32_t bits, uint32_t hb,
                                            uint32_t *s_bin, uint64_t &ors, uint32_t &mine) {
    constexpr int U = 8;
    const uint32_t shift = bits - hb, mask = (1u << hb) - 1u;
    const uint64_t c0 = sort_code<LOG>(keys[0]);
    constexpr uint64_t step = (uint64_t)BK_HIST_THREADS * U;
    for (uint64_t t0 = (uint64_t)blockIdx.x * step; t0 < n; t0 += (uint64_t)gridDim.x * step) {
        K k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = t0 + (uint64_t)u * BK_HIST_THREADS + threadIdx.x;
            k[u] = i < n ? keys[i] : K(0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = t0 + (uint64_t)u * BK_HIST_THREADS + threadIdx.x;
            if (i >= n) continue;
            const uint64_t c = sort_code<LOG>(k[u]);
            const uint32_t b = (uint32_t)(c >> shift) & mask;
            ors |= c ^ c0;
            ++mine;
            atomicAdd(&s_bin[b >> 1], 1u << (16 * (b & 1)));
        }
    }
}

template <typename K>
__global__ __launch_bounds__(BK_HIST_THREADS) void k_sort_hist(const K *__restrict__ keys, uint64_t n, uint32_t want,
                                                               uint32_t *__restrict__ partial, SortInfo *info) {
    extern __shared__ __align__(16) char smem[];
    uint32_t *s_bin = (uint32_t *)smem;
    __shared__ unsigned long long s_or;
    __shared__ uint32_t s_keys, s_counts;
    const uint32_t words = (1u << want) / 2;
    for (uint32_t i = threadIdx.x; i < words; i += BK_HIST_THREADS) s_bin[i] = 0;
    if (threadIdx.x == 0) {
        s_or = 0;
        s_keys = 0;
        s_counts = 0;
    }
    __syncthreads();
    const uint32_t bits = info->bits, hb = bucket_bits(want, bits);
    uint64_t ors = 0;
    uint32_t mine = 0;
    if (info->log) bucket_hist<K, true>(keys, n, bits, hb, s_bin, ors, mine);
    else bucket_hist<K, false>(keys, n, bits, hb, s_bin, ors, mine);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        ors |= (uint64_t)__shfl_xor((unsigned long long)ors, off, kWave);
        mine += __shfl_xor(mine, off, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicOr(&s_or, (unsigned long long)ors);
        atomicAdd(&s_keys, mine);
    }
    __syncthreads();
    uint32_t sum = 0;
    for (uint32_t i = threadIdx.x; i < words; i += BK_HIST_THREADS) {
        const uint32_t w = s_bin[i];
        sum += (w & 0xFFFFu) + (w >> 16);
        partial[(uint64_t)blockIdx.x * words + i] = w;
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&s_counts, sum);
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicOr(&info->ors, s_or);
        if (s_counts != s_keys) atomicOr(&info->bad, 1u);
    }
}

// Bucket counts summed over the histogram's workgroups (BK_SUM_WORDS words per
// workgroup here, the rows split over its waves), scanned within the
// workgroup: starts without the counts of earlier workgroups, which go to
// block[]; and the largest bucket.
constexpr uint32_t BK_SUM_WORDS = 64, BK_SUM_ROWS = 16;

__global__ __launch_bounds__(BK_SUM_WORDS * BK_SUM_ROWS) void k_sort_hist_sum(const uint32_t *__restrict__ partial,
                                                                              uint32_t rows, uint32_t words,
                                                                              uint32_t *__restrict__ starts,
                                                                              uint32_t *__restrict__ block,
                                                                              SortInfo *info) {
    __shared__ uint32_t s_lo[BK_SUM_ROWS][BK_SUM_WORDS], s_hi[BK_SUM_ROWS][BK_SUM_WORDS];
    const uint32_t x = threadIdx.x % BK_SUM_WORDS, y = threadIdx.x / BK_SUM_WORDS;  // y: the wave
    const uint32_t i = blockIdx.x * BK_SUM_WORDS + x;
    uint32_t lo = 0, hi = 0;
#pragma unroll 4
    for (uint32_t r = y; r < rows; r += BK_SUM_ROWS) {
        const uint32_t w = i < words ? partial[(uint64_t)r * words + i] : 0u;
        lo += w & 0xFFFFu;
        hi += w >> 16;
    }
    s_lo[y][x] = lo;
    s_hi[y][x] = hi;
    __syncthreads();
    if (y != 0) return;
    for (uint32_t r = 1; r < BK_SUM_ROWS; ++r) {
        lo += s_lo[r][x];
        hi += s_hi[r][x];
    }
    uint32_t incl = lo + hi, mx = lo > hi ? lo : hi;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, kWave);
        if (x >= (uint32_t)off) incl += t;
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const uint32_t t = __shfl_xor(mx, off, kWave);
        mx = t > mx ? t : mx;
    }
    if (i < words) {
        starts[2 * i] = incl - lo - hi;
        starts[2 * i + 1] = incl - hi;
    }
    if (x == kWave - 1) {
        block[blockIdx.x] = incl;
        atomicMax(&info->max_bucket, mx);
    }
}

// Exclusive scan of one value per thread over the workgroup (any multiple of
// 64 threads); s_wave holds one entry per wave.  Barriers on both sides.
__device__ __forceinline__ uint32_t wg_exclusive_scan(uint32_t v, uint32_t *s_wave) {
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, kWave);
        if (lane >= (uint32_t)off) incl += t;
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < wave; ++w) before += s_wave[w];
    __syncthreads();
    return before + incl - v;
}

// Adds the counts of earlier workgroups of k_sort_hist_sum (at most 512) to
// their starts, 128 per workgroup as there; starts[bins] = n.
__global__ __launch_bounds__(2 * BK_SUM_WORDS) void k_sort_hist_starts(const uint32_t *__restrict__ block,
                                                                       uint32_t bins, uint64_t n,
                                                                       uint32_t *__restrict__ starts) {
    __shared__ uint32_t s_sum;
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t b = threadIdx.x; b < blockIdx.x; b += 2 * BK_SUM_WORDS) before += block[b];
    if (before) atomicAdd(&s_sum, before);
    __syncthreads();
    const uint32_t i = blockIdx.x * 2 * BK_SUM_WORDS + threadIdx.x;
    if (i < bins) starts[i] += s_sum;
    if (i == 0) starts[bins] = (uint32_t)n;
}

// First bucket of every tile of k_bucket_sort: tile t takes the buckets that
// start in [t * tile, (t + 1) * tile).
__global__ __launch_bounds__(256) void k_sort_tiles(const uint32_t *__restrict__ starts, uint32_t bins, uint32_t tile,
                                                    uint32_t tiles, uint32_t *__restrict__ first,
                                                    uint32_t *__restrict__ todo) {
    const uint32_t t = blockIdx.x * 256 + threadIdx.x;
    if (t == 0) todo[0] = 0;
    if (t > tiles) return;
    const uint64_t at = (uint64_t)t * tile;
    uint32_t lo = 0, len = bins;  // first bucket with start >= at (bins: none)
    while (len) {
        const uint32_t half = len >> 1;
        if (starts[lo + half] < at) {
            lo += half + 1;
            len -= half + 1;
        } else {
            len = half;
        }
    }
    first[t] = lo;
}

// LDS of k_bucket_sort: the pairs' keys (their bins first), the pairs' row IDs
// (a word of each first), and a pad past the last bin's words.
template <typename K>
constexpr size_t bucket_lds_bytes(uint32_t threads) {
    return (size_t)threads * BK_ITEMS * (sizeof(K) + 4) + 4 * (BK_BIN_MAX + 8);
}

// One stable radix pass of the (key, input position) pairs in LDS by the 8
// bits at `shift` (k_scatter's ranking).  Every thread takes part.
template <typename K, int THREADS>
__device__ __forceinline__ void lds_radix_pass(K *s_key, uint16_t *s_idx, uint32_t *s_cnt, uint32_t *s_start,
                                               uint32_t *s_wave, uint32_t cnt, int shift) {
    constexpr int WAVES = THREADS / kWave;
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    for (uint32_t i = threadIdx.x; i < WAVES * RS_BINS; i += THREADS) s_cnt[i] = 0;
    K key[BK_ITEMS];
    uint32_t rank[BK_ITEMS];  // input position << 16 | rank
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j) {
        const uint32_t i = wave * (BK_ITEMS * kWave) + j * kWave + lane;
        key[j] = i < cnt ? s_key[i] : K(0);
        rank[j] = i < cnt ? (uint32_t)s_idx[i] << 16 : 0u;
    }
    __syncthreads();
    uint32_t *mine = s_cnt + wave * RS_BINS;
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j) {
        const bool valid = wave * (BK_ITEMS * kWave) + j * kWave + lane < cnt;
        const uint32_t d = (uint32_t)(key[j] >> shift) & (RS_BINS - 1);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < RS_BITS; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
        const uint32_t before = mine[d];
        rank[j] |= before + below;
        wave_lds_order();
        if (valid && below == 0) mine[d] = before + (uint32_t)__popcll(peers);
        wave_lds_order();
        __builtin_amdgcn_sched_barrier(0);  // one pair's ballots at a time: together they spill registers
    }
    __syncthreads();
    uint32_t sum = 0;
    if (threadIdx.x < RS_BINS) {
        for (int w = 0; w < WAVES; ++w) {
            const uint32_t c = s_cnt[w * RS_BINS + threadIdx.x];
            s_cnt[w * RS_BINS + threadIdx.x] = sum;
            sum += c;
        }
    }
    const uint32_t start = wg_exclusive_scan(sum, s_wave);
    if (threadIdx.x < RS_BINS) s_start[threadIdx.x] = start;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j) {
        if (wave * (BK_ITEMS * kWave) + j * kWave + lane >= cnt) continue;
        const uint32_t d = (uint32_t)(key[j] >> shift) & (RS_BINS - 1);
        const uint32_t pos = s_start[d] + mine[d] + (rank[j] & 0xFFFFu);
        s_key[pos] = key[j];
        s_idx[pos] = (uint16_t)(rank[j] >> 16);
    }
    __syncthreads();
}

// Writes a tile's pairs (ranks from p0 on) from LDS; flags as k_bucket_sort.
// PLACE: to their slots of a level-order layout, whose lowest level takes runs of
// k - 1 consecutive ranks, so that the separate pass from the sorted arrays (285
// us for 2^26 64-bit keys, k = 9) is saved for 60 us more here.
template <typename K, int THREADS, bool PLACE>
__device__ __forceinline__ void tile_out(const K *s_key, const uint32_t *s_row, uint32_t cnt, uint64_t p0, K *ko,
                                         uint32_t *ro, const SortPlace &place, uint32_t *flags) {
    bool dup = false, miss = false;
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j) {
        const uint32_t i = (uint32_t)j * THREADS + threadIdx.x;
        if (i >= cnt) continue;
        const K k = s_key[i];
        const uint32_t r = s_row[i];
        dup |= i > 0 && s_key[i - 1] == k;  // the previous tile's keys lie in other buckets
        miss |= r == kMiss;
        uint64_t at = p0 + i;
        if constexpr (PLACE)
            at = place.G.k == 2 ? rank_slot_binary(place.G, at) + place.off
                                : rank_slot_general(place.G, (uint32_t)at, place.kinv);
        ko[at] = k;
        ro[at] = r;
    }
    if (flags) {
        if (__any(dup) && (threadIdx.x & (kWave - 1)) == 0 && flags[0] == 0) atomicOr(&flags[0], 1u);
        if (__any(miss) && (threadIdx.x & (kWave - 1)) == 0) atomicOr(&flags[1], 1u);
    }
}

// Sorts whole buckets in LDS: workgroup t takes the pairs [starts[first[t]],
// starts[first[t + 1]]), which are in bucket order, and writes them in key
// order to the same positions (the input may be the output).  starts =
// nullptr: one bucket of all n pairs.
//
// The pairs are counted into one bin per pair, each bucket's bins spread
// evenly over the code range below its bucket bits, so that a bin holds one
// pair on average when the keys spread evenly there.  A pair's place is its
// bin's start plus the bin's pairs before it, which it counts itself from one
// 32-bit word per pair: 19 bits of the key's offset inside the bin, then the
// input position, so that words order by (key, position).  Two words of a bin
// that differ in the position alone may stand for different keys: then the
// tile's pairs are counted again by their keys.  If a bin holds more than
// BK_BIN_MAX pairs (keys clustered inside the bucket, many duplicates) the
// tile is left to k_bucket_radix: todo[0] counts such tiles (zeroed by
// k_sort_tiles), their numbers follow.
//
// Bound by LDS work and VALU between its barriers: 2^26 64-bit pairs take
// 0.44 ms where copying them takes 0.33 ms (1.72 ms with each bin put in order
// by one thread's insertions, 1.37 ms with whole keys compared).  48 KiB of
// LDS per 4096 64-bit pairs let three workgroups share a compute unit.
// flags (when given): [0] |= 1 for two equal adjacent keys, [1] |= 1 for a
// row ID equal to IDX_MISS.
template <typename K, int THREADS, bool LOG, bool PLACE>
__global__ __launch_bounds__(THREADS, THREADS == 512 ? 6 : 4) void k_bucket_sort(
    const K *keys_in, const uint32_t *rows_in, K *keys_out, uint32_t *rows_out, uint64_t n,
    const uint32_t *__restrict__ starts, const uint32_t *__restrict__ first, uint32_t tiles, uint32_t bits, uint32_t hb,
    uint32_t *__restrict__ todo, SortPlace place, uint32_t *flags) {
    constexpr uint32_t CAP = THREADS * BK_ITEMS;
    constexpr uint32_t POS = 0x1FFF;  // positions, starts: 13 bits
    static_assert(BK_ITEMS == 8 && CAP <= POS + 1, "two 16-byte reads of bins per thread; 13-bit positions");
    extern __shared__ __align__(16) char smem[];
    K *s_key = (K *)smem;
    uint32_t *s_row = (uint32_t *)(s_key + CAP);
    uint32_t *s_bin = (uint32_t *)smem;  // CAP counters, then start | count << 13; before the keys are placed
    uint32_t *s_word = s_row;            // before the row IDs are placed
    __shared__ uint32_t s_wave[THREADS / kWave];
    __shared__ unsigned long long s_or;
    __shared__ uint32_t s_long, s_tie;
    const uint32_t t = starts ? xcd_tile(blockIdx.x, tiles) : 0;
    uint64_t p0 = 0;
    uint32_t cnt = (uint32_t)n;
    if (starts) {
        p0 = starts[first[t]];
        cnt = starts[first[t + 1]] - (uint32_t)p0;
    }
    if (cnt == 0) return;  // workgroup-uniform
    const K *kp = keys_in + p0;
    const uint32_t *rp = rows_in + p0;
    if (threadIdx.x == 0) {
        s_or = 0;
        s_long = 0;
        s_tie = 0;
    }
    ((uint4 *)s_bin)[threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
    ((uint4 *)s_bin)[threadIdx.x + THREADS] = make_uint4(0u, 0u, 0u, 0u);
    // Straight-line code over the thread's pairs in every phase (a pair past
    // cnt stands for pair 0 and adds nothing), so that their loads, atomics
    // and LDS reads are in flight together.
    K key[BK_ITEMS];
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j) {
        const uint32_t i = (uint32_t)j * THREADS + threadIdx.x;
        key[j] = kp[i < cnt ? i : 0];
    }
    __syncthreads();
    if (!starts) {  // one bucket: its varying bits are the tile's
        const K k0 = kp[0];
        uint64_t o = 0;
#pragma unroll
        for (int j = 0; j < BK_ITEMS; ++j) o |= (uint64_t)(key[j] ^ k0);
        if (o) atomicOr(&s_or, (unsigned long long)o);
        __syncthreads();
        bits = bits_of(s_or);
        hb = 0;
    }
    const uint32_t low = bits - hb;  // code bits below the bucket's
    uint32_t at[BK_ITEMS];           // bin, then start | bin's pairs << 13 | turn << 18 | pairs before << 23
    uint32_t word[BK_ITEMS];
    {
        const uint64_t low_mask = low >= 64 ? ~0ull : (1ull << low) - 1ull;
        const uint32_t bmask = (uint32_t)((1ull << hb) - 1ull);
        uint32_t b0[BK_ITEMS], b1[BK_ITEMS];
#pragma unroll
        for (int j = 0; j < BK_ITEMS; ++j) {
            b0[j] = 0;
            b1[j] = cnt;
            if (starts) {
                const uint32_t b = low >= 64 ? 0u : (uint32_t)(sort_code<LOG>(key[j]) >> low) & bmask;
                b0[j] = starts[b];
                b1[j] = starts[b + 1];
            }
        }
#pragma unroll
        for (int j = 0; j < BK_ITEMS; ++j) {
            const uint32_t i = (uint32_t)j * THREADS + threadIdx.x;
            const uint64_t v = sort_code<LOG>(key[j]) & low_mask;
            const uint32_t frac = low >= 32 ? (uint32_t)(v >> (low - 32)) : (uint32_t)(v << (32 - low));
            const uint64_t prod = (uint64_t)frac * (b1[j] - b0[j]);
            at[j] = b0[j] - (uint32_t)p0 + (uint32_t)(prod >> 32);
            word[j] = ((uint32_t)prod & ~POS) | i;
        }
    }
    uint32_t turn[BK_ITEMS];
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j)
        turn[j] = atomicAdd(&s_bin[at[j]], (uint32_t)j * THREADS + threadIdx.x < cnt ? 1u : 0u);
    __syncthreads();
    {  // bin starts: each thread scans its 8 bins
        const uint4 w0 = ((const uint4 *)s_bin)[2 * threadIdx.x], w1 = ((const uint4 *)s_bin)[2 * threadIdx.x + 1];
        uint32_t c[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
        uint32_t sum = 0, mx = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            sum += c[i];
            mx = c[i] > mx ? c[i] : mx;
        }
        if (mx > BK_BIN_MAX) s_long = 1;
        uint32_t run = wg_exclusive_scan(sum, s_wave);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t here = c[i];
            c[i] = run | (here << 13);
            run += here;
        }
        ((uint4 *)s_bin)[2 * threadIdx.x] = make_uint4(c[0], c[1], c[2], c[3]);
        ((uint4 *)s_bin)[2 * threadIdx.x + 1] = make_uint4(c[4], c[5], c[6], c[7]);
    }
    __syncthreads();
    if (!starts && threadIdx.x == 0) todo[0] = s_long;
    if (s_long) {  // workgroup-uniform: left to k_bucket_radix
        if (threadIdx.x == 0) todo[starts ? 1 + atomicAdd(&todo[0], 1u) : 1] = t;
        return;
    }
    uint32_t cmax = 0;
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j) at[j] = s_bin[at[j]];
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j) {
        if ((uint32_t)j * THREADS + threadIdx.x < cnt) {
            s_word[(at[j] & POS) + turn[j]] = word[j];
            cmax = max(cmax, at[j] >> 13);
            at[j] |= turn[j] << 18;
        } else {
            at[j] = 0;
        }
    }
    uint32_t row[BK_ITEMS];
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j) {
        const uint32_t i = (uint32_t)j * THREADS + threadIdx.x;
        row[j] = rp[i < cnt ? i : 0];
    }
    __syncthreads();
    bool tie = false;
    if (cmax > 1)
        for (uint32_t e = 0; e < cmax; e += 2) {
            uint32_t w[BK_ITEMS][2];
#pragma unroll
            for (int j = 0; j < BK_ITEMS; ++j) {  // at most BK_BIN_MAX words past the tile's: within s_word and its pad
                w[j][0] = s_word[(at[j] & POS) + e];
                w[j][1] = s_word[(at[j] & POS) + e + 1];
            }
#pragma unroll
            for (int j = 0; j < BK_ITEMS; ++j) {
#pragma unroll
                for (uint32_t f = 0; f < 2; ++f) {
                    const bool in = e + f < ((at[j] >> 13) & 31u);
                    at[j] += (in && w[j][f] < word[j]) ? 1u << 23 : 0u;
                    const uint32_t x = w[j][f] ^ word[j];
                    tie |= in && x != 0 && x <= POS;
                }
            }
        }
    if (tie) s_tie = 1;
    __syncthreads();
    if (s_tie) {  // workgroup-uniform
#pragma unroll
        for (int j = 0; j < BK_ITEMS; ++j)
            if ((uint32_t)j * THREADS + threadIdx.x < cnt) s_key[(at[j] & POS) + ((at[j] >> 18) & 31u)] = key[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < BK_ITEMS; ++j) {
            const uint32_t s0 = at[j] & POS, c = (at[j] >> 13) & 31u;
            uint32_t before = 0;
            for (uint32_t e = 0; e < c; ++e) {
                const K k = s_key[s0 + e];
                before += (k < key[j] || (k == key[j] && (s_word[s0 + e] & POS) < (word[j] & POS))) ? 1u : 0u;
            }
            at[j] = (at[j] & 0x7FFFFFu) | (before << 23);
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < BK_ITEMS; ++j) {
        const uint32_t pos = (at[j] & POS) + (at[j] >> 23);
        if ((uint32_t)j * THREADS + threadIdx.x < cnt) {
            s_key[pos] = key[j];
            s_row[pos] = row[j];
        }
    }
    __syncthreads();
    tile_out<K, THREADS, PLACE>(s_key, s_row, cnt, p0, keys_out, rows_out, place, flags);
}

// The tiles that k_bucket_sort left (todo), by radix passes in LDS.
// The row IDs are read by input position once the keys are in order, all of
// them before any is written.
template <typename K, int THREADS, bool PLACE>
__global__ __launch_bounds__(THREADS) void k_bucket_radix(const K *keys_in, const uint32_t *rows_in, K *keys_out,
                                                          uint32_t *rows_out, uint64_t n,
                                                          const uint32_t *__restrict__ starts,
                                                          const uint32_t *__restrict__ first,
                                                          const uint32_t *__restrict__ todo, SortPlace place,
                                                          uint32_t *flags) {
    constexpr uint32_t CAP = THREADS * BK_ITEMS;
    extern __shared__ __align__(16) char smem[];
    K *s_key = (K *)smem;
    uint32_t *s_row = (uint32_t *)(s_key + CAP);
    uint16_t *s_idx = (uint16_t *)s_row;
    uint32_t *s_cnt = s_row + CAP / 2;
    __shared__ uint32_t s_wave[THREADS / kWave], s_start[RS_BINS];
    __shared__ unsigned long long s_or;
    const uint32_t listed = todo[0];
    for (uint32_t l = blockIdx.x; l < listed; l += gridDim.x) {
        const uint32_t t = todo[1 + l];
        const uint64_t p0 = starts ? starts[first[t]] : 0;
        const uint32_t cnt = starts ? starts[first[t + 1]] - (uint32_t)p0 : (uint32_t)n;
        const K *kp = keys_in + p0;
        if (threadIdx.x == 0) s_or = 0;
        __syncthreads();
        const K k0 = kp[0];
        uint64_t o = 0;
        for (uint32_t i = threadIdx.x; i < cnt; i += THREADS) {
            const K k = kp[i];
            s_key[i] = k;
            s_idx[i] = (uint16_t)i;
            o |= (uint64_t)(k ^ k0);
        }
        if (o) atomicOr(&s_or, (unsigned long long)o);
        __syncthreads();
        const uint64_t ors = s_or;
        for (int shift = 0; shift < (int)sizeof(K) * 8; shift += RS_BITS)
            if ((ors >> shift) & (RS_BINS - 1))
                lds_radix_pass<K, THREADS>(s_key, s_idx, s_cnt, s_start, s_wave, cnt, shift);
        uint32_t row[BK_ITEMS];
#pragma unroll
        for (int j = 0; j < BK_ITEMS; ++j) {
            const uint32_t i = (uint32_t)j * THREADS + threadIdx.x;
            row[j] = i < cnt ? rows_in[p0 + s_idx[i]] : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < BK_ITEMS; ++j) {
            const uint32_t i = (uint32_t)j * THREADS + threadIdx.x;
            if (i < cnt) s_row[i] = row[j];
        }
        __syncthreads();
        tile_out<K, THREADS, PLACE>(s_key, s_row, cnt, p0, keys_out, rows_out, place, flags);
        __syncthreads();  // before the next tile is staged
    }
}

struct TempLayout {
    size_t keys_off, rows_off, tile_off, total_off, ghist_off, info_off, block_off, starts_off, first_off, todo_off, bytes;
    uint32_t tiles;
    uint32_t want;       // bucket bits asked for (0: n fits one workgroup)
    uint32_t hist_grid;  // workgroups of the bucket histogram
};

TempLayout temp_layout(uint64_t n, bool u64) {
    auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    TempLayout t{};
    t.tiles = (uint32_t)((n + RS_TILE - 1) / RS_TILE);
    if (t.tiles == 0) t.tiles = 1;
    if (n > BK_LARGE * BK_ITEMS)
        while (t.want < BK_BITS && (n >> t.want) > BK_AVG) ++t.want;
    const uint64_t share = (n + 8191) / 8192;  // one round of its loads each
    t.hist_grid = share < BK_HIST_GRID ? (uint32_t)(share ? share : 1) : BK_HIST_GRID;
    size_t off = 0;
    t.keys_off = off;
    off += up(n * (u64 ? 8 : 4));
    t.rows_off = off;
    off += up(n * 4);
    t.tile_off = off;
    off += up((size_t)t.tiles * RS_BINS * 4);
    t.total_off = off;
    off += up(RS_BINS * 4);
    t.ghist_off = off;
    off += up(8 * RS_BINS * 4);
    t.info_off = off;
    off += up(sizeof(SortInfo));
    t.block_off = off;
    off += up((((size_t)1 << t.want) / (2 * BK_SUM_WORDS) + 1) * 4);
    t.starts_off = off;
    off += up((((size_t)1 << t.want) + 1) * 4);
    t.first_off = off;
    off += up((size_t)(n / 1024 + 3) * 4);  // tiles hold 1536 pairs or more
    t.todo_off = off;
    off += up((size_t)(n / 1024 + 4) * 4);
    t.bytes = off;
    return t;
}

// One stable radix pass by the digit (code >> shift) & mask.
template <typename K, bool LOG>
int radix_pass(const TempLayout &tl, char *tb, const K *src_k, const uint32_t *src_r, K *dst_k, uint32_t *dst_r,
               uint64_t n, int shift, uint32_t mask, hipStream_t s) {
    uint32_t *tile_hist = (uint32_t *)(tb + tl.tile_off);
    uint32_t *digit_total = (uint32_t *)(tb + tl.total_off);
    hipLaunchKernelGGL((k_tile_hist<K, LOG>), dim3(tl.tiles), dim3(RS_THREADS), 0, s, src_k, n, shift, mask, tile_hist,
                       tl.tiles);
    IDX_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_digit_scan, dim3(RS_BINS), dim3(RS_THREADS), 0, s, tile_hist, tl.tiles, digit_total);
    IDX_LAUNCH_CHECK();
    hipLaunchKernelGGL((k_scatter<K, LOG>), dim3(tl.tiles), dim3(RS_THREADS), 0, s, src_k, src_r, dst_k, dst_r, n,
                       shift, mask, tile_hist, tl.tiles, digit_total);
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

// LSD passes over the digits that vary.
template <typename K>
int sort_lsd(const TempLayout &tl, char *tb, const K *keys_in, const uint32_t *rows_in, uint64_t n, K *keys_out,
             uint32_t *rows_out, hipStream_t s) {
    constexpr int passes_max = (int)sizeof(K);
    K *tkeys = (K *)(tb + tl.keys_off);
    uint32_t *trows = (uint32_t *)(tb + tl.rows_off);
    uint32_t *ghist = (uint32_t *)(tb + tl.ghist_off);
    IDX_HIP(hipMemsetAsync(ghist, 0, 8 * RS_BINS * 4, s));
    {
        uint64_t blocks = (n + RS_THREADS * 16 - 1) / (RS_THREADS * 16);
        if (blocks > 2048) blocks = 2048;
        hipLaunchKernelGGL(k_global_hist<K>, dim3((uint32_t)blocks), dim3(RS_THREADS), 0, s, keys_in, n, passes_max,
                           ghist);
        IDX_LAUNCH_CHECK();
    }
    uint32_t hh[8 * RS_BINS];
    IDX_HIP(hipMemcpyAsync(hh, ghist, sizeof(uint32_t) * passes_max * RS_BINS, hipMemcpyDeviceToHost, s));
    IDX_HIP(hipStreamSynchronize(s));
    int run[8], nrun = 0;
    for (int p = 0; p < passes_max; ++p) {
        bool trivial = false;
        for (int d = 0; d < RS_BINS; ++d)
            if (hh[p * RS_BINS + d] == n) trivial = true;
        if (!trivial) run[nrun++] = p;
    }
    if (nrun == 0) {
        IDX_HIP(hipMemcpyAsync(keys_out, keys_in, n * sizeof(K), hipMemcpyDeviceToDevice, s));
        IDX_HIP(hipMemcpyAsync(rows_out, rows_in, n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
        return IDX_OK;
    }
    // Ping-pong so that the last pass writes keys_out / rows_out.
    const K *src_k = keys_in;
    const uint32_t *src_r = rows_in;
    for (int r = 0; r < nrun; ++r) {
        const bool to_out = ((nrun - 1 - r) % 2) == 0;
        K *dst_k = to_out ? keys_out : tkeys;
        uint32_t *dst_r = to_out ? rows_out : trows;
        const int rc = radix_pass<K, false>(tl, tb, src_k, src_r, dst_k, dst_r, n, run[r] * RS_BITS, RS_BINS - 1, s);
        if (rc != IDX_OK) return rc;
        src_k = dst_k;
        src_r = dst_r;
    }
    return IDX_OK;
}

template <typename K, int THREADS, bool LOG, bool PLACE>
int bucket_sort(const K *ki, const uint32_t *ri, K *ko, uint32_t *ro, uint64_t n, const uint32_t *starts,
                const uint32_t *first, uint32_t tiles, uint32_t bits, uint32_t hb, uint32_t *todo,
                const SortPlace &place, uint32_t *flags, hipStream_t s) {
    hipLaunchKernelGGL((k_bucket_sort<K, THREADS, LOG, PLACE>), dim3(tiles), dim3(THREADS),
                       bucket_lds_bytes<K>(THREADS), s, ki, ri, ko, ro, n, starts, first, tiles, bits, hb, todo, place,
                       flags);
    IDX_LAUNCH_CHECK();
    hipLaunchKernelGGL((k_bucket_radix<K, THREADS, PLACE>), dim3(tiles < 512 ? tiles : 512), dim3(THREADS),
                       bucket_lds_bytes<K>(THREADS), s, ki, ri, ko, ro, n, starts, first, (const uint32_t *)todo,
                       place, flags);
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

// The same to the sorted arrays ko, ro, or (place) to the layout's.
template <typename K, int THREADS, bool LOG>
int bucket_sort_to(const K *ki, const uint32_t *ri, K *ko, uint32_t *ro, uint64_t n, const uint32_t *starts,
                   const uint32_t *first, uint32_t tiles, uint32_t bits, uint32_t hb, uint32_t *todo, SortPlace *place,
                   uint32_t *flags, hipStream_t s) {
    if (!place)
        return bucket_sort<K, THREADS, LOG, false>(ki, ri, ko, ro, n, starts, first, tiles, bits, hb, todo, SortPlace{},
                                                   flags, s);
    place->done = true;
    return bucket_sort<K, THREADS, LOG, true>(ki, ri, (K *)place->keys, place->rows, n, starts, first, tiles, bits, hb,
                                              todo, *place, flags, s);
}

// The radix passes over the bucket bits [bits - hb, bits), then the buckets.
template <typename K, bool LOG>
int sort_buckets(const TempLayout &tl, char *tb, const K *keys_in, const uint32_t *rows_in, uint64_t n, K *keys_out,
                 uint32_t *rows_out, const SortInfo &info, uint32_t hb, SortPlace *place, uint32_t *flags, hipStream_t s) {
    const uint32_t lo = hb > RS_BITS ? hb / 2 : 0, hi = hb - lo;  // bits of the passes (lo first, when there are two)
    const int base = (int)(info.bits - hb);
    K *tkeys = (K *)(tb + tl.keys_off);
    uint32_t *trows = (uint32_t *)(tb + tl.rows_off);
    int rc;
    if (lo) {
        rc = radix_pass<K, LOG>(tl, tb, keys_in, rows_in, tkeys, trows, n, base, (1u << lo) - 1u, s);
        if (rc != IDX_OK) return rc;
    }
    rc = radix_pass<K, LOG>(tl, tb, lo ? (const K *)tkeys : keys_in, lo ? (const uint32_t *)trows : rows_in, keys_out,
                            rows_out, n, base + (int)lo, (1u << hi) - 1u, s);
    if (rc != IDX_OK) return rc;
    if (hb == info.bits && !LOG)  // every varying bit is sorted by
        return flags ? check_sorted(keys_out, rows_out, n, sizeof(K) == 8, flags, s) : IDX_OK;
    const uint32_t *starts = (const uint32_t *)(tb + tl.starts_off);
    uint32_t *first = (uint32_t *)(tb + tl.first_off), *todo = (uint32_t *)(tb + tl.todo_off);
    // A tile is the buckets that start in `tile` consecutive positions: at
    // most tile + max_bucket - 1 pairs, which fit the workgroup's LDS.
    const bool small = info.max_bucket <= 2560;
    const uint32_t cap = (small ? BK_SMALL : BK_LARGE) * BK_ITEMS;
    const uint32_t tile = cap - info.max_bucket;
    const uint32_t tiles = (uint32_t)((n + tile - 1) / tile);
    hipLaunchKernelGGL(k_sort_tiles, dim3(tiles / 256 + 1), dim3(256), 0, s, starts, 1u << tl.want, tile, tiles, first, todo);
    IDX_LAUNCH_CHECK();
    return small ? bucket_sort_to<K, BK_SMALL, LOG>(keys_out, rows_out, keys_out, rows_out, n, starts, first, tiles,
                                                 info.bits, hb, todo, place, flags, s)
                 : bucket_sort_to<K, BK_LARGE, LOG>(keys_out, rows_out, keys_out, rows_out, n, starts, first, tiles,
                                                 info.bits, hb, todo, place, flags, s);
}

template <typename K>
int sort_impl(const K *keys_in, const uint32_t *rows_in, uint64_t n, K *keys_out, uint32_t *rows_out, void *temp,
              SortPlace *place, uint32_t *flags, hipStream_t s) {
    if (n == 0) return IDX_OK;
    const TempLayout tl = temp_layout(n, sizeof(K) == 8);
    char *tb = (char *)temp;
    uint32_t *todo = (uint32_t *)(tb + tl.todo_off);
    // one workgroup takes it all: no histogram, nothing for the host to read
    if (n <= BK_SMALL * BK_ITEMS)
        return bucket_sort_to<K, BK_SMALL, false>(keys_in, rows_in, keys_out, rows_out, n, nullptr, nullptr, 1, 0, 0,
                                               todo, place, flags, s);
    if (n <= BK_LARGE * BK_ITEMS)
        return bucket_sort_to<K, BK_LARGE, false>(keys_in, rows_in, keys_out, rows_out, n, nullptr, nullptr, 1, 0, 0,
                                               todo, place, flags, s);
    SortInfo *dinfo = (SortInfo *)(tb + tl.info_off);
    uint32_t *partial = (uint32_t *)(tb + tl.keys_off);  // hist_grid * 2^want / 2 words <= n words; free until the passes
    uint32_t *block = (uint32_t *)(tb + tl.block_off);
    uint32_t *starts = (uint32_t *)(tb + tl.starts_off);
    const uint32_t bins = 1u << tl.want, words = bins / 2;
    SortInfo info{};
    hipLaunchKernelGGL(k_sort_sample<K>, dim3(1), dim3(RS_BINS), 0, s, keys_in, n, dinfo);
    IDX_LAUNCH_CHECK();
    bool known = false;
    for (int attempt = 0; attempt < 2 && !known; ++attempt) {
        hipLaunchKernelGGL(k_sort_hist<K>, dim3(tl.hist_grid), dim3(BK_HIST_THREADS), (size_t)words * 4, s, keys_in, n,
                           tl.want, partial, dinfo);
        IDX_LAUNCH_CHECK();
        const uint32_t blocks = (words + BK_SUM_WORDS - 1) / BK_SUM_WORDS;
        hipLaunchKernelGGL(k_sort_hist_sum, dim3(blocks), dim3(BK_SUM_WORDS * BK_SUM_ROWS), 0, s, partial,
                           tl.hist_grid, words, starts, block, dinfo);
        IDX_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_sort_hist_starts, dim3(blocks), dim3(2 * BK_SUM_WORDS), 0, s, block, bins, n, starts);
        IDX_LAUNCH_CHECK();
        IDX_HIP(hipMemcpyAsync(&info, dinfo, sizeof(info), hipMemcpyDeviceToHost, s));
        IDX_HIP(hipStreamSynchronize(s));
        known = (info.ors >> 1) >> (info.bits ? info.bits - 1 : 0) == 0 && !(info.bits == 0 && info.ors);
        if (!known) {  // bits above the sample's vary: count again with the true ones
            info.bits = 64u - (uint32_t)__builtin_clzll(info.ors);
            info.ors = 0;
            info.bad = 0;
            info.max_bucket = 0;
            IDX_HIP(hipMemcpyAsync(dinfo, &info, sizeof(info), hipMemcpyHostToDevice, s));
        }
    }
    const uint32_t hb = bucket_bits(tl.want, info.bits);
    const bool all_bits = hb == info.bits && !info.log;
    if (known && info.bits > 0 && (all_bits || (!info.bad && info.max_bucket <= 6144)))
        return info.log ? sort_buckets<K, true>(tl, tb, keys_in, rows_in, n, keys_out, rows_out, info, hb, place, flags, s)
                        : sort_buckets<K, false>(tl, tb, keys_in, rows_in, n, keys_out, rows_out, info, hb, place, flags, s);
    const int rc = sort_lsd<K>(tl, tb, keys_in, rows_in, n, keys_out, rows_out, s);
    if (rc != IDX_OK || !flags) return rc;
    return check_sorted(keys_out, rows_out, n, sizeof(K) == 8, flags, s);
}

}  // namespace

size_t sort_temp_bytes(uint64_t n, bool u64) { return temp_layout(n, u64).bytes; }

int sort_pairs(const void *keys_in, const uint32_t *rows_in, uint64_t n, bool u64, void *keys_out,
               uint32_t *rows_out, void *temp, SortPlace *place, uint32_t *flags, hipStream_t s) {
    if (u64)
        return sort_impl<uint64_t>((const uint64_t *)keys_in, rows_in, n, (uint64_t *)keys_out, rows_out, temp, place,
                                   flags, s);
    return sort_impl<uint32_t>((const uint32_t *)keys_in, rows_in, n, (uint32_t *)keys_out, rows_out, temp, place,
                               flags, s);
}

}  // namespace idx
