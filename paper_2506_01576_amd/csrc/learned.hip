// Learned rank model on a sorted-array index (BS layout): a two-stage FP32
// model -- a linear root over a monotone key feature selects one of L leaves,
// each leaf a line over the leaf-local key offset -- trained on the GPU on the
// index's own (key, rank) pairs, then used to narrow every lookup to a window
// bounded by the leaf's measured error (the window-then-search idea of the
// PGM index the paper compares with, Section 8; the last-mile search is the
// expensive step, Section 9).
//
// Exactness does not depend on the model.  The root is non-decreasing in the
// key (non-negative slope over a non-decreasing feature, round-to-nearest
// arithmetic without contraction), so the keys of a leaf form one contiguous
// rank interval [base, base + size) and every key that maps to a leaf has its
// lower bound inside that interval (or at its end).  Inside a leaf the
// prediction is non-decreasing too, and the error bounds are measured with the
// same device function over all of the leaf's keys; a window
// [pred + elo, pred + ehi + 1] clamped to the leaf interval therefore contains
// the lower bound of any query, member or not.
//
// Training (per stage, `epochs` times): a forward/backward kernel evaluates
// the FP32 prediction and accumulates, in FP64, the loss sum, the gradient
// sums (residual * feature, residual) and the Hessian sums (feature^2,
// feature, count); an update kernel takes the Newton step
// theta -= H^-1 g, which for this quadratic loss reaches the least-squares
// fit in one step from zero, the second step correcting FP32 rounding.
#include <climits>
#include <cstddef>

#include <new>

#include "internal.hpp"
#include "access.hpp"
#include "learned_model.hpp"
#include "qio.hpp"

namespace idx {

namespace {

constexpr int LT = 256;  // threads per block in the training kernels
constexpr int CHUNK = 32;  // consecutive keys per thread in the per-leaf passes

// Root candidates of one training, by index: linear roots over the LINEAR and
// LOG feature, spline roots with LINEAR and LOG bins.
constexpr int kRoots = 4;
constexpr int kSpline0 = 2;  // the first spline candidate

// What a root pass sums for the linear candidates (accumulator layout at
// NACC): the feature sums depend on the keys alone, so that the first pass
// takes them for all steps, and the loss is wanted once.
constexpr uint32_t kSumX = 1, kSumGrad = 2, kSumLoss = 4;

// Sums of every candidate in `mask` over all keys, in one read of them (a
// spline root has no parameters to fit: only its loss).  Bound by vector
// instructions (conversions and FP64), so each pass leaves out the sums it
// does not need: 2^26 64-bit keys in 126, 108 and 275 us for the first, second
// and last pass of the four candidates, where each candidate took 136 us a
// pass and the training eight passes.
template <typename K, bool AOS, uint32_t SUMS, bool SPLINES>
__global__ __launch_bounds__(LT) void k_root_accum(Load<K, AOS> keys, uint64_t n, const RootRec *__restrict__ roots,
                                                   uint32_t mask, double *__restrict__ acc) {
    __shared__ double s[LT / kWave][kRoots][NACC];
    double a[kRoots][NACC] = {};
    const double scale = (double)roots[__builtin_ctz(mask)].L / (double)n;
    const RootRec R0 = roots[0], R1 = roots[1], R2 = roots[2], R3 = roots[3];
    constexpr int U = 2;  // keys loaded together
    const uint64_t step = (uint64_t)gridDim.x * LT;
    for (uint64_t i0 = (uint64_t)blockIdx.x * LT + threadIdx.x; i0 < n; i0 += U * step) {
        uint64_t kk[U];
#pragma unroll
        for (int u = 0; u < U; ++u) kk[u] = i0 + u * step < n ? (uint64_t)keys.key(i0 + u * step) : 0ull;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t i = i0 + u * step, key = kk[u];
            if (i >= n) continue;
            const float t = (float)((double)(uint32_t)i * scale);
            auto linear = [&](const RootRec &R, double (&v)[NACC]) {
                const float x = key_feature(key, R.mode);
                const float r = __fsub_rn(__fadd_rn(__fmul_rn(R.a1, x), R.a0), t);  // forward residual
                if constexpr (SUMS & kSumX) {
                    v[1] += x;
                    v[2] += (double)x * x;
                }
                if constexpr (SUMS & kSumGrad) {
                    v[3] += r;
                    v[4] += (double)r * x;
                }
                if constexpr (SUMS & kSumLoss) v[5] += (double)r * r;
            };
            auto spline = [&](const RootRec &R, double (&v)[NACC]) {
                float pred;
                (void)spline_leaf(R, key, &pred);
                const float r = __fsub_rn(pred, t);
                v[5] += (double)r * r;
            };
            if (mask & 1u) linear(R0, a[0]);
            if (mask & 2u) linear(R1, a[1]);
            if constexpr (SPLINES) {
                spline(R2, a[2]);
                spline(R3, a[3]);
            }
        }
    }
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
    for (int c = 0; c < kRoots; ++c) {
        if (!((mask >> c) & 1u)) continue;
#pragma unroll
        for (int j = 1; j < NACC; ++j) {
            const double v = wave_sum(a[c][j]);
            if (lane == 0) s[wave][c][j] = v;
        }
    }
    __syncthreads();
    if (threadIdx.x < kRoots * NACC && ((mask >> (threadIdx.x / NACC)) & 1u)) {
        const int c = threadIdx.x / NACC, j = threadIdx.x % NACC;
        if (j == 0) {
            if (blockIdx.x == 0) acc[threadIdx.x] = (double)n;
        } else {
            double v = 0;
            for (int w = 0; w < LT / kWave; ++w) v += s[w][c][j];
            if (v != 0.0) atomicAdd(&acc[threadIdx.x], v);
        }
    }
}

// The Newton step of the linear candidates in `mask`; their residual sums
// start over.
__global__ void k_root_update(RootRec *roots, uint32_t mask, double *acc) {
    const uint32_t c = threadIdx.x;
    if (c >= (uint32_t)kSpline0 || !((mask >> c) & 1u)) return;
    newton_linear(acc + c * NACC, roots[c].a0, roots[c].a1);
    acc[c * NACC + 3] = acc[c * NACC + 4] = 0.0;
}

// First rank of every leaf, base[0, L], base[L] = n.  The root is
// non-decreasing along the keys, so leaf l starts at the first rank whose
// leaf is l or more: the rank where the leaf rises past it writes it, with no
// counts, atomics or scan (0.53 ms for those and the leaf records of 2^24
// leaves, 0.10 to 0.15 ms for this).  Runs of more than kGapInline empty leaves go to a
// list in pieces, filled by k_leaf_gaps.  A linear root given with a negative
// slope (learn_eval only) is non-increasing: its leaves are counted from the
// last key down, so that base[l] is still the number of keys below leaf l.
constexpr uint32_t kGapInline = 64, kGapPiece = 4096;

struct Gap {
    uint32_t first, last, value;  // base[first..last] = value
};

// Gap pieces that L leaves can make.
inline size_t gap_capacity(uint32_t L) { return (size_t)L / kGapInline + L / kGapPiece + 4; }

template <typename K, bool AOS>
__global__ __launch_bounds__(LT) void k_leaf_bounds(Load<K, AOS> keys, uint64_t n, const RootRec *Rp,
                                                    uint32_t *__restrict__ base, Gap *__restrict__ gaps,
                                                    uint32_t *__restrict__ ngaps) {
    const RootRec R = *Rp;
    const bool down = R.mode != IDX_FEATURE_SPLINE && R.a1 < 0.f;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    auto key_at = [&](uint64_t i) { return (uint64_t)keys.key(down ? n - 1 - i : i); };
    constexpr int U = 8;  // steps of 64 keys per wave, loaded together
    const uint64_t b = ((uint64_t)blockIdx.x * LT + (threadIdx.x & ~(uint32_t)(kWave - 1))) * U;
    auto set = [&](uint32_t first, uint32_t last, uint32_t value) {
        if (last - first < kGapInline) {
            for (uint32_t l = first; l <= last; ++l) base[l] = value;
            return;
        }
        const uint32_t pieces = (last - first) / kGapPiece + 1;
        uint32_t g = atomicAdd(ngaps, pieces);
        for (uint32_t p = 0; p < pieces; ++p, ++g) {
            const uint32_t f = first + p * kGapPiece;
            gaps[g] = Gap{f, last - f < kGapPiece ? last : f + kGapPiece - 1, value};
        }
    };
    uint64_t kk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t i = b + (uint64_t)u * kWave + lane;
        kk[u] = i < n ? key_at(i) : 0ull;
    }
    uint32_t carry = ~0u;  // leaf of the rank before the wave's step; none before rank 0
    if (b > 0 && b < n) carry = leaf_of(R, key_at(b - 1));
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t i = b + (uint64_t)u * kWave + lane;
        const uint32_t l = leaf_of(R, kk[u]);
        const uint32_t before = __shfl_up(l, 1);
        const uint32_t prev = lane == 0 ? carry : before;
        carry = __shfl(l, kWave - 1);
        if (i >= n) continue;
        if (l + 1 > prev + 1) set(prev + 1, l, (uint32_t)i);
        if (i == n - 1) set(l + 1, R.L, (uint32_t)n);
    }
}

__global__ __launch_bounds__(256) void k_leaf_gaps(const Gap *__restrict__ gaps, const uint32_t *__restrict__ ngaps,
                                                   uint32_t *__restrict__ base) {
    const uint32_t count = *ngaps;
    for (uint32_t g = blockIdx.x; g < count; g += gridDim.x) {
        const Gap p = gaps[g];
        for (uint32_t l = p.first + threadIdx.x; l <= p.last; l += 256) base[l] = p.value;
    }
}

// The keys of the workgroup's leaves [l0, l1) into LDS (false: too many).
template <typename K, bool AOS>
__device__ __forceinline__ bool stage_leaf_keys(Load<K, AOS> keys, uint64_t kb, uint64_t ke, K *s_key, uint32_t cap) {
    if (ke - kb > cap) return false;  // workgroup-uniform
    stage_keys<K>([&](uint64_t i) { return keys.key(i); }, kb, ke, s_key);
    return true;
}

// A leaf's record before its fit.
template <typename K, bool AOS>
__device__ __forceinline__ LeafRec new_leaf(Load<K, AOS> keys, uint32_t base, uint32_t end) {
    LeafRec r{};
    r.base = base;
    r.size = end - base;
    r.kmin = r.size ? (uint64_t)keys.key(base) : 0ull;
    r.elo = 0;
    r.ehi = -1;
    return r;
}

// Fit and error bounds of one leaf of at most kFitSlots keys: its features are
// converted once and stay in registers, the feature sums are taken once, and
// each step sums only what depends on the parameters.  The sums run in the
// order of leaf_sums_thread and every product is exact in FP64, so that the
// parameters come out the same.
constexpr int kFitSlots = 12;

template <typename KeyAt>
__device__ __forceinline__ void fit_leaf_short(const KeyAt &key, LeafRec &r, uint32_t epochs, double &loss) {
    float x[kFitSlots];
    double a[NACC] = {(double)r.size, 0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < kFitSlots; ++j) {
        if ((uint32_t)j >= r.size) continue;
        x[j] = local_feature(r, key((uint64_t)r.base + j));
        a[1] += x[j];
        a[2] += (double)x[j] * x[j];
    }
    auto residual = [&](int j) {  // forward residual, as leaf_terms rounds it
        return __fsub_rn(__fadd_rn(__fmul_rn(r.b1, x[j]), r.b0), (float)j);
    };
    for (uint32_t ep = 0; ep < epochs; ++ep) {
        a[3] = a[4] = 0.0;
#pragma unroll
        for (int j = 0; j < kFitSlots; ++j) {
            if ((uint32_t)j >= r.size) continue;
            const float e = residual(j);
            a[3] += e;
            a[4] += (double)e * x[j];
        }
        newton_linear(a, r.b0, r.b1);
    }
    int32_t lo = INT_MAX, hi = INT_MIN;
#pragma unroll
    for (int j = 0; j < kFitSlots; ++j) {
        if ((uint32_t)j >= r.size) continue;
        const float p = __fadd_rn(__fmul_rn(r.b1, x[j]), r.b0);  // as pred_local
        const int32_t pl = !(p > 0.f) ? 0 : p >= (float)r.size ? (int32_t)r.size : (int32_t)p;
        lo = j - pl < lo ? j - pl : lo;
        hi = j - pl > hi ? j - pl : hi;
        const float e = __fsub_rn(p, (float)j);
        loss += (double)e * e;
    }
    r.elo = lo;
    r.ehi = hi;
}

// A thread walks its leaf key by key, so a leaf of 1000 keys among leaves of 4
// (the last bin of a spline root holds such ones) kept one lane busy for 300 us
// after the others were done.  Leaves of more than kWaveLeaf keys are trained
// by a wave each (k_leaf_train_wave); up to there a leaf takes about 25 us.
constexpr uint32_t kWaveLeaf = 128;

// The leaves trained in one pass, one thread per leaf of at most kWaveLeaf
// keys: `epochs` Newton steps from its sums in registers, then its error
// bounds and squared residuals, the workgroup's keys staged in LDS once
// (`cap` keys of dynamic LDS, stage_cap) for all of them.  The workgroup's
// leaves are dealt to its threads by size, largest first, so that the lanes of
// a wave walk leaves of about the same size (a wave of 64 leaves of 4 keys on
// average holds one of 11).  part[3 * blockIdx.x] receives the workgroup's
// window sum, largest window and loss.  A larger leaf gets its record here and
// goes to the list todo[0..*ntodo); one of more than kLeafCap keys gets zero
// sums and *big = 1, and the *_big kernels train it.
// Bound by vector instructions (conversions and FP64): 2^24 leaves of 2^26
// keys in 385 us, where a pass over the keys for each step, the bounds and the
// statistics took 1.32 ms.
template <typename K, bool AOS>
__global__ __launch_bounds__(kLeafBlock) void k_leaf_train(Load<K, AOS> keys, const uint32_t *__restrict__ base,
                                                           uint32_t L, uint32_t epochs, LeafRec *__restrict__ leaves,
                                                           double *__restrict__ acc, uint32_t *big,
                                                           uint32_t *__restrict__ todo, uint32_t *__restrict__ ntodo,
                                                           uint32_t cap, double *__restrict__ part) {
    extern __shared__ __align__(16) char smem_stage[];
    K *s_key = (K *)smem_stage;
    __shared__ double s_part[kLeafBlock / kWave][3];
    __shared__ uint32_t s_bin[kFitSlots + 2], s_base[kLeafBlock + 1];
    __shared__ uint8_t s_leaf[kLeafBlock];
    const uint32_t l0 = blockIdx.x * kLeafBlock, l1 = l0 + kLeafBlock < L ? l0 + kLeafBlock : L, nl = l1 - l0;
    if (threadIdx.x < kFitSlots + 2) s_bin[threadIdx.x] = 0;
    for (uint32_t t = threadIdx.x; t <= nl; t += kLeafBlock) s_base[t] = base[l0 + t];
    __syncthreads();
    const uint64_t kb = s_base[0];
    // places by size: bin 0 the leaves of more than kFitSlots keys, then
    // kFitSlots keys, and so on down to none
    uint32_t bin = 0, place = 0;
    if (threadIdx.x < nl) {
        const uint32_t size = s_base[threadIdx.x + 1] - s_base[threadIdx.x];
        bin = size > (uint32_t)kFitSlots ? 0u : kFitSlots + 1 - size;
        place = atomicAdd(&s_bin[bin], 1u);
    }
    const bool staged = s_base[nl] - s_base[0] <= cap;  // workgroup-uniform
    if (staged) stage_keys<K>([&](uint64_t i) { return keys.key(i); }, kb, (uint64_t)s_base[nl], s_key);
    else __syncthreads();
    if (threadIdx.x < nl) {
        for (uint32_t b = 0; b < bin; ++b) place += s_bin[b];
        s_leaf[place] = (uint8_t)threadIdx.x;
    }
    __syncthreads();
    double ws = 0.0, wmax = 0.0, ls = 0.0;
    if (threadIdx.x < nl) {
        const uint32_t o = s_leaf[threadIdx.x], l = l0 + o;
        LeafRec r{};
        r.base = s_base[o];
        r.size = s_base[o + 1] - r.base;
        r.elo = 0;
        r.ehi = -1;
        auto train = [&](auto &&key) {
            r.kmin = key(r.base);
            if (r.size > kLeafCap) {
                *big = 1u;
                r.elo = INT_MAX;
                r.ehi = INT_MIN;
                for (int j = 0; j < NACC; ++j) acc[(uint64_t)l * NACC + j] = 0.0;
                return;
            }
            if (r.size > kWaveLeaf) {
                todo[atomicAdd(ntodo, 1u)] = l;
                return;
            }
            if (r.size <= (uint32_t)kFitSlots) {
                fit_leaf_short(key, r, epochs, ls);
            } else {
                for (uint32_t ep = 0; ep < epochs; ++ep) {
                    double a[NACC];
                    leaf_sums_thread(key, r, a);
                    newton_linear(a, r.b0, r.b1);
                }
                long long lo, hi;
                leaf_errs_thread(key, r, lo, hi, &ls);
                r.elo = (int32_t)lo;
                r.ehi = (int32_t)hi;
            }
            wmax = (double)r.ehi - (double)r.elo + 2.0;  // window slots incl. one past
            ws = wmax * r.size;
        };
        if (r.size == 0) {
        } else if (staged) {
            train([&](uint64_t i) { return (uint64_t)s_key[i - kb]; });
        } else {
            train([&](uint64_t i) { return (uint64_t)keys.key(i); });
        }
        leaves[l] = r;
    }
    ws = wave_sum(ws);
    ls = wave_sum(ls);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const double o = __shfl_xor(wmax, off, kWave);
        wmax = o > wmax ? o : wmax;
    }
    const uint32_t wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_part[wave][0] = ws;
        s_part[wave][1] = wmax;
        s_part[wave][2] = ls;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t w = 1; w < kLeafBlock / kWave; ++w) {
            ws += s_part[w][0];
            wmax = s_part[w][1] > wmax ? s_part[w][1] : wmax;
            ls += s_part[w][2];
        }
        double *p = part + 3 * (uint64_t)blockIdx.x;
        p[0] = ws;
        p[1] = wmax;
        p[2] = ls;
    }
}

__device__ __forceinline__ void atomic_max_pos(double *p, double v) {  // values >= 0 order like their bit patterns
    atomicMax((unsigned long long *)p, (unsigned long long)__double_as_longlong(v));
}

// The leaves of the list, a wave each.  A step of 64 keys: the lanes compute
// their keys' terms side by side into LDS, then lanes 0-3 add one column each
// in key order.  The sums are those of leaf_sums_thread, addition by addition,
// at the latency of one FP64 addition a key where the walk of one thread takes
// about 40 instructions.  part[3 * blockIdx.x] as in k_leaf_train: statistics
// added by every leaf to one place cost 13 ns an addition, 2.7 ms for 67108
// leaves of 1000 64-bit keys that take 1.17 ms so (a thread a leaf, a pass over
// the keys for each step and the bounds: 1.86 ms).
template <typename K, bool AOS>
__global__ __launch_bounds__(256) void k_leaf_train_wave(Load<K, AOS> keys, uint32_t epochs,
                                                         LeafRec *__restrict__ leaves,
                                                         const uint32_t *__restrict__ todo,
                                                         const uint32_t *__restrict__ ntodo,
                                                         double *__restrict__ part) {
    __shared__ double s_term[256 / kWave][kWave][4], s_part[256 / kWave][3];
    double ws = 0.0, wmax = 0.0, ls = 0.0;
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, count = *ntodo;
    double(*term)[4] = s_term[wave];
    if (count == 0) return;  // k_leaf_stats then leaves part out
    for (uint32_t t = blockIdx.x * (256 / kWave) + wave; t < count; t += gridDim.x * (256 / kWave)) {
        const uint32_t l = todo[t];
        LeafRec r = leaves[l];
        double a[NACC] = {(double)r.size, 0, 0, 0, 0, 0};
        for (uint32_t ep = 0; ep < epochs; ++ep) {
            double col = 0.0;  // lanes 0-3: sums of x, x^2, r, r x
            for (uint32_t j0 = 0; j0 < r.size; j0 += kWave) {
                const uint32_t j = j0 + lane;
                double v[4] = {0, 0, 0, 0};
                if (j < r.size) {
                    const float x = local_feature(r, (uint64_t)keys.key((uint64_t)r.base + j));
                    const float e = __fsub_rn(__fadd_rn(__fmul_rn(r.b1, x), r.b0), (float)j);
                    v[0] = x;
                    v[1] = (double)x * x;
                    v[2] = e;
                    v[3] = (double)e * x;
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) term[lane][c] = v[c];
                wave_lds_order();
                if (lane < 4) {
                    const uint32_t end = r.size - j0 < (uint32_t)kWave ? r.size - j0 : (uint32_t)kWave;
                    for (uint32_t i0 = 0; i0 < end; i0 += 16) {  // (zeros past the leaf)
#pragma unroll
                        for (uint32_t i = 0; i < 16; ++i) col += term[i0 + i][lane];
                    }
                }
                wave_lds_order();
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) a[1 + c] = __shfl(col, c, kWave);
            newton_linear(a, r.b0, r.b1);
        }
        int32_t lo = INT_MAX, hi = INT_MIN;
        double loss = 0.0;
        for (uint32_t j = lane; j < r.size; j += kWave) {
            const uint64_t i = (uint64_t)r.base + j, key = (uint64_t)keys.key(i);
            const int32_t e = (int32_t)leaf_err(r, i, key);
            lo = e < lo ? e : lo;
            hi = e > hi ? e : hi;
            loss += leaf_sq_residual(r, i, key);
        }
        loss = wave_sum(loss);
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            const int32_t ol = __shfl_xor(lo, off, kWave), oh = __shfl_xor(hi, off, kWave);
            lo = ol < lo ? ol : lo;
            hi = oh > hi ? oh : hi;
        }
        if (lane == 0) {
            r.elo = lo;
            r.ehi = hi;
            leaves[l] = r;
        }
        const double w = (double)hi - (double)lo + 2.0;
        ws += w * r.size;
        wmax = w > wmax ? w : wmax;
        ls += loss;
    }
    if (lane == 0) {
        s_part[wave][0] = ws;
        s_part[wave][1] = wmax;
        s_part[wave][2] = ls;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t w = 1; w < 256 / kWave; ++w) {
            ws += s_part[w][0];
            wmax = s_part[w][1] > wmax ? s_part[w][1] : wmax;
            ls += s_part[w][2];
        }
        double *p = part + 3 * (uint64_t)blockIdx.x;
        p[0] = ws;
        p[1] = wmax;
        p[2] = ls;
    }
}

// stats += the workgroups' window sums, largest window and losses: those of
// k_leaf_train, then (if leaves were listed) k_leaf_train_wave's.  A few
// workgroups, one atomic each.
__global__ __launch_bounds__(256) void k_leaf_stats(const double *__restrict__ part, uint32_t tblocks, uint32_t wblocks,
                                                    const uint32_t *__restrict__ ntodo, double *__restrict__ stats) {
    double ws = 0.0, wmax = 0.0, ls = 0.0;
    const uint32_t blocks = tblocks + (*ntodo ? wblocks : 0);
    for (uint32_t b = blockIdx.x * 256 + threadIdx.x; b < blocks; b += gridDim.x * 256) {
        ws += part[3 * (uint64_t)b];
        wmax = part[3 * (uint64_t)b + 1] > wmax ? part[3 * (uint64_t)b + 1] : wmax;
        ls += part[3 * (uint64_t)b + 2];
    }
    ws = wave_sum(ws);
    ls = wave_sum(ls);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const double o = __shfl_xor(wmax, off, kWave);
        wmax = o > wmax ? o : wmax;
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicAdd(&stats[0], ws);
        atomic_max_pos(&stats[1], wmax);
        atomicAdd(&stats[2], ls);
    }
}

// The windows of the leaves larger than kLeafCap (nothing to do when *big is
// 0; the others' come with their training).
__global__ __launch_bounds__(256) void k_leaf_stats_big(const LeafRec *__restrict__ leaves, uint32_t L,
                                                        const uint32_t *big, double *__restrict__ stats) {
    if (*big == 0u) return;
    for (uint32_t l = blockIdx.x * 256 + threadIdx.x; l < L; l += gridDim.x * 256) {
        const LeafRec r = leaves[l];
        if (r.size <= kLeafCap) continue;
        const double w = (double)r.ehi - (double)r.elo + 2.0;
        atomicAdd(&stats[0], w * r.size);
        atomic_max_pos(&stats[1], w);
    }
}

// Gradient evaluation: every leaf's sums at given parameters, one thread per
// leaf; a leaf of more than kLeafCap keys gets zero sums here and raises *big
// for k_leaf_accum_big.
template <typename K, bool AOS>
__global__ __launch_bounds__(kLeafBlock) void k_leaf_accum_small(Load<K, AOS> keys, const LeafRec *__restrict__ leaves,
                                                                 uint32_t L, double *__restrict__ acc, uint32_t *big,
                                                                 uint32_t cap) {
    extern __shared__ __align__(16) char smem_stage[];
    K *s_key = (K *)smem_stage;
    const uint32_t l0 = blockIdx.x * kLeafBlock, l1 = l0 + kLeafBlock < L ? l0 + kLeafBlock : L;
    const uint64_t kb = leaves[l0].base;
    const bool staged = stage_leaf_keys(keys, kb, (uint64_t)leaves[l1 - 1].base + leaves[l1 - 1].size, s_key, cap);
    const uint32_t l = l0 + threadIdx.x;
    if (l >= L) return;
    const LeafRec r = leaves[l];
    double a[NACC] = {0, 0, 0, 0, 0, 0};
    if (r.size > kLeafCap) *big = 1u;
    else if (staged) leaf_sums_thread([&](uint64_t i) { return (uint64_t)s_key[i - kb]; }, r, a);
    else leaf_sums_thread([&](uint64_t i) { return (uint64_t)keys.key(i); }, r, a);
#pragma unroll
    for (int j = 0; j < NACC; ++j) acc[(uint64_t)l * NACC + j] = a[j];
}

// The keys of leaves larger than kLeafCap: the wave walk over all keys,
// skipping every step without such a key (nothing to do when *big is 0).
template <typename K, bool AOS>
__global__ __launch_bounds__(LT) void k_leaf_accum_big(Load<K, AOS> keys, uint64_t n, const RootRec *Rp,
                                                       const LeafRec *__restrict__ leaves, double *__restrict__ acc,
                                                       const uint32_t *big) {
    if (*big == 0u) return;
    const RootRec R = *Rp;
    // this wave's CHUNK * 64 consecutive keys
    const uint64_t b = ((uint64_t)blockIdx.x * LT + (threadIdx.x & ~(uint32_t)(kWave - 1))) * CHUNK;
    const uint64_t e = b + (uint64_t)kWave * CHUNK < n ? b + (uint64_t)kWave * CHUNK : n;
    wave_leaf_sums<NACC>(
        b, e,
        [&](uint64_t i, uint32_t &l, double *a) {
            const uint64_t key = (uint64_t)keys.key(i);
            l = leaf_of(R, key);
            const LeafRec L = leaves[l];
            if (L.size <= kLeafCap) return false;
            leaf_terms(L, i, key, a);
            return true;
        },
        [&](uint32_t l, const double *v) {
#pragma unroll
            for (int j = 0; j < NACC; ++j) atomicAdd(&acc[(uint64_t)l * NACC + j], v[j]);
        });
}

// The Newton step of the leaves larger than kLeafCap (nothing to do when
// *big is 0; the others stepped in k_leaf_train or k_leaf_train_wave); their sums start over.
__global__ void k_leaf_update_big(LeafRec *__restrict__ leaves, double *__restrict__ acc, uint32_t L,
                                  const uint32_t *big) {
    if (*big == 0u) return;
    for (uint32_t l = blockIdx.x * blockDim.x + threadIdx.x; l < L; l += gridDim.x * blockDim.x) {
        LeafRec r = leaves[l];
        if (r.size <= kLeafCap) continue;
        newton_linear(acc + (uint64_t)l * NACC, r.b0, r.b1);
        leaves[l].b0 = r.b0;
        leaves[l].b1 = r.b1;
        for (int j = 0; j < NACC; ++j) acc[(uint64_t)l * NACC + j] = 0.0;
    }
}

// Error bounds of the leaves larger than kLeafCap (the wave walk).
template <typename K, bool AOS>
__global__ __launch_bounds__(LT) void k_leaf_errors_big(Load<K, AOS> keys, uint64_t n, const RootRec *Rp,
                                                        LeafRec *__restrict__ leaves, const uint32_t *big,
                                                        double *__restrict__ loss) {
    if (*big == 0u) return;
    const RootRec R = *Rp;
    const uint64_t b = ((uint64_t)blockIdx.x * LT + (threadIdx.x & ~(uint32_t)(kWave - 1))) * CHUNK;
    const uint64_t e = b + (uint64_t)kWave * CHUNK < n ? b + (uint64_t)kWave * CHUNK : n;
    double ls = 0.0;  // this lane's squared residuals over the large leaves' keys
    wave_leaf_maxes(
        b, e,
        [&](uint64_t i, uint32_t &l, long long *a) {
            const uint64_t key = (uint64_t)keys.key(i);
            l = leaf_of(R, key);
            const LeafRec L = leaves[l];
            if (L.size <= kLeafCap) return false;
            const long long err = leaf_err(L, i, key);
            a[0] = -err;
            a[1] = err;
            ls += leaf_sq_residual(L, i, key);
            return true;
        },
        [&](uint32_t l, const long long *v) {
            atomicMin(&leaves[l].elo, (int32_t)(-v[0]));
            atomicMax(&leaves[l].ehi, (int32_t)v[1]);
        });
    ls = wave_sum(ls);
    if ((threadIdx.x & (kWave - 1)) == 0 && ls != 0.0) atomicAdd(loss, ls);
}

// Geometry of the spline candidates in `mask` from the smallest and largest
// build key.
template <typename K, bool AOS>
__global__ void k_spline_geometry(Load<K, AOS> keys, uint64_t n, RootRec *roots, uint32_t mask) {
    const uint32_t c = threadIdx.x;
    if (c < (uint32_t)kRoots && ((mask >> c) & 1u))
        spline_geometry(roots[c], (uint64_t)keys.key(0), (uint64_t)keys.key(n - 1), n);
}

// Their bins, one thread per bin (blockIdx.y: the candidate).
template <typename K, bool AOS>
__global__ void k_spline_bins(Load<K, AOS> keys, uint64_t n, const RootRec *__restrict__ roots, uint32_t first) {
    const RootRec R = roots[first + blockIdx.y];
    const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= R.nb) return;
    ((SplineBin *)R.bins)[b] = spline_bin([&](uint64_t i) { return (uint64_t)keys.key(i); }, n, R, b);
}

uint32_t grid_for(uint64_t threads, uint32_t block) {
    uint64_t b = (threads + block - 1) / block;
    if (b == 0) b = 1;
    if (b > 0x7FFFFFFFull) b = 0x7FFFFFFFull;
    return (uint32_t)b;
}

size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

// Bytes of the first ranks of L leaves and their gap list.
size_t bounds_bytes(uint32_t L) { return up256(((size_t)L + 1) * 4) + up256(gap_capacity(L) * sizeof(Gap)); }

// First ranks of the leaves under *d_root; *ngaps comes zeroed.
template <typename K, bool AOS>
int leaf_bounds(Load<K, AOS> keys, uint64_t n, const RootRec *d_root, uint32_t L, char *tmp, uint32_t *ngaps,
                hipStream_t s) {
    uint32_t *base = (uint32_t *)tmp;
    Gap *gaps = (Gap *)(tmp + up256(((size_t)L + 1) * 4));
    hipLaunchKernelGGL((k_leaf_bounds<K, AOS>), dim3(grid_for((n + 7) / 8, LT)), dim3(LT), 0, s, keys, n, d_root, base,
                       gaps, ngaps);
    hipLaunchKernelGGL(k_leaf_gaps, dim3(512), dim3(256), 0, s, gaps, ngaps, base);
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

// What the device keeps of one training; zeroed, then the roots are set.
struct TrainCtl {
    RootRec roots[kRoots];
    double acc[kRoots][NACC];
    double stats[2][4];   // per root family: sum of window * size, max window, leaf loss
    uint32_t big[2];      // a leaf larger than kLeafCap exists
    uint32_t ngaps[2];
    uint32_t ntodo[2];    // leaves of the wave kernel
};

uint32_t root_blocks(uint64_t n) {
    const uint64_t b = (n + LT * 8 - 1) / (LT * 8);
    return b > 2048 ? 2048u : (uint32_t)b;
}

template <typename K, bool AOS>
int train_t(idx_index *h, uint32_t L, uint32_t epochs, uint32_t feature, hipStream_t s) {
    const uint64_t n = h->n;
    const Load<K, AOS> keys = make_load<K, AOS>(h);
    LearnedModel *M = h->learned;
    const bool want_lin = feature != IDX_FEATURE_SPLINE, want_sp = feature == IDX_FEATURE_AUTO ||
                                                                   feature == IDX_FEATURE_SPLINE;
    const bool both = want_lin && want_sp;
    // device scratch: control block, first ranks and gaps, the large leaves'
    // sums and the workgroups' statistics; (both root families) a second leaf
    // table and (splines) the second candidate's bins, which take the place of
    // the model's when they win
    const uint32_t tblocks = grid_for(L, kLeafBlock);
    const size_t ctl_b = up256(sizeof(TrainCtl)), bounds_b = bounds_bytes(L);
    const uint64_t todo_n = n / (kWaveLeaf + 1) + 1;  // leaves of more than kWaveLeaf keys at most
    const uint32_t wblocks = grid_for(todo_n, 4) < 2048 ? grid_for(todo_n, 4) : 2048;
    const size_t acc_b = up256((size_t)L * NACC * sizeof(double));
    const size_t part_b = up256(((size_t)tblocks + wblocks) * 3 * sizeof(double));
    char *tmp = (char *)h->alloc.get(ctl_b + bounds_b + acc_b + part_b + up256(todo_n * 4), s);
    LeafRec *alt = tmp && both ? (LeafRec *)h->alloc.get((size_t)L * sizeof(LeafRec), s) : nullptr;
    SplineBin *bins2 = tmp && want_sp ? (SplineBin *)h->alloc.get((size_t)spline_bins(n) * sizeof(SplineBin), s)
                                      : nullptr;
    auto give_back = [&] {
        if (bins2) h->alloc.put(bins2, s);
        if (alt) h->alloc.put(alt, s);
        if (tmp) h->alloc.put(tmp, s);
    };
    if (!tmp || (both && !alt) || (want_sp && !bins2)) {
        give_back();
        return IDX_ERR_NOMEM;
    }
    TrainCtl *ctl = (TrainCtl *)tmp;
    char *bounds = tmp + ctl_b;
    double *leaf_acc = (double *)(bounds + bounds_b), *part = (double *)((char *)leaf_acc + acc_b);
    uint32_t *todo = (uint32_t *)((char *)part + part_b);
    const uint32_t cblocks = grid_for((n + CHUNK - 1) / CHUNK, LT);
    const uint32_t lblocks = grid_for(L, 256) < 1024 ? grid_for(L, 256) : 1024;  // passes over large leaves alone
    const uint32_t cap = stage_cap(n, L);  // keys staged per workgroup of the leaf pass

    // Leaves under candidate c into `leaves`: first ranks, Newton steps, error
    // bounds and statistics of family f.
    auto leaves_for = [&](int c, int f, LeafRec *leaves) -> int {
        const RootRec *d_root = &ctl->roots[c];
        uint32_t *big = &ctl->big[f];
        int rc = leaf_bounds<K, AOS>(keys, n, d_root, L, bounds, &ctl->ngaps[f], s);
        if (rc != IDX_OK) return rc;
        hipLaunchKernelGGL((k_leaf_train<K, AOS>), dim3(tblocks), dim3(kLeafBlock), (size_t)cap * sizeof(K), s, keys,
                           (const uint32_t *)bounds, L, epochs, leaves, leaf_acc, big, todo, &ctl->ntodo[f], cap, part);
        hipLaunchKernelGGL((k_leaf_train_wave<K, AOS>), dim3(wblocks), dim3(256), 0, s, keys, epochs, leaves, todo,
                           &ctl->ntodo[f], part + 3 * (size_t)tblocks);
        for (uint32_t ep = 0; ep < epochs; ++ep) {
            hipLaunchKernelGGL((k_leaf_accum_big<K, AOS>), dim3(cblocks), dim3(LT), 0, s, keys, n, d_root, leaves,
                               leaf_acc, big);
            hipLaunchKernelGGL(k_leaf_update_big, dim3(lblocks), dim3(256), 0, s, leaves, leaf_acc, L, big);
        }
        hipLaunchKernelGGL((k_leaf_errors_big<K, AOS>), dim3(cblocks), dim3(LT), 0, s, keys, n, d_root, leaves, big,
                           &ctl->stats[f][2]);
        hipLaunchKernelGGL(k_leaf_stats_big, dim3(lblocks), dim3(256), 0, s, leaves, L, big, ctl->stats[f]);
        const uint32_t sblocks = grid_for(tblocks + wblocks, 256);
        hipLaunchKernelGGL(k_leaf_stats, dim3(sblocks < 64 ? sblocks : 64), dim3(256), 0, s, part, tblocks, wblocks,
                           &ctl->ntodo[f], ctl->stats[f]);
        IDX_LAUNCH_CHECK();
        return IDX_OK;
    };

    int rc = IDX_OK;
    do {
        // ---- stage 1: roots.  A linear root takes `epochs` Newton steps over
        // either key feature; a spline root is built from the keys' ranks over
        // either bin feature.  Within each family the lower loss wins.
        TrainCtl hc{};
        uint32_t lin_mask = 0, sp_mask = 0;
        for (uint32_t f = 0; f < 2; ++f) {
            RootRec R{};
            R.L = L;
            R.mode = IDX_FEATURE_LINEAR + f;
            hc.roots[f] = R;
            if (want_lin && (feature == IDX_FEATURE_AUTO || feature == IDX_FEATURE_LINEAR + f)) lin_mask |= 1u << f;
            R.mode = IDX_FEATURE_SPLINE;
            R.bins = f == 0 ? M->spline : bins2;
            R.bfeat = IDX_FEATURE_LINEAR + f;
            hc.roots[kSpline0 + f] = R;
            if (want_sp) sp_mask |= 1u << (kSpline0 + f);
        }
        if (hipMemcpyAsync(ctl, &hc, sizeof(hc), hipMemcpyHostToDevice, s) != hipSuccess) {
            rc = IDX_ERR_HIP;
            break;
        }
        if (want_sp) {
            hipLaunchKernelGGL((k_spline_geometry<K, AOS>), dim3(1), dim3(64), 0, s, keys, n, ctl->roots, sp_mask);
            hipLaunchKernelGGL((k_spline_bins<K, AOS>), dim3(grid_for(spline_bins(n), 256), 2), dim3(256), 0, s, keys,
                               n, ctl->roots, (uint32_t)kSpline0);
        }
        // the spline losses come with the linear roots' last pass
        auto root_sums = [&](auto kernel, uint32_t mask) {
            hipLaunchKernelGGL(kernel, dim3(root_blocks(n)), dim3(LT), 0, s, keys, n, ctl->roots, mask,
                               &ctl->acc[0][0]);
        };
        for (uint32_t ep = lin_mask ? 0 : epochs; ep <= epochs; ++ep) {
            if (ep == 0) root_sums(k_root_accum<K, AOS, kSumX | kSumGrad, false>, lin_mask);
            else if (ep < epochs) root_sums(k_root_accum<K, AOS, kSumGrad, false>, lin_mask);
            else if (want_sp) root_sums(k_root_accum<K, AOS, kSumLoss, true>, lin_mask | sp_mask);
            else root_sums(k_root_accum<K, AOS, kSumLoss, false>, lin_mask);
            if (ep < epochs)
                hipLaunchKernelGGL(k_root_update, dim3(1), dim3(64), 0, s, ctl->roots, lin_mask, &ctl->acc[0][0]);
        }
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(&hc, ctl, offsetof(TrainCtl, stats), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            rc = IDX_ERR_HIP;
            break;
        }
        auto pick = [&](uint32_t mask, int c0) {  // the lower loss of a family's candidates
            int best = -1;
            for (int c = c0; c < c0 + 2; ++c)
                if (((mask >> c) & 1u) && (best < 0 || hc.acc[c][5] < hc.acc[best][5])) best = c;
            return best;
        };
        const int lin = pick(lin_mask, 0), spl = pick(sp_mask, kSpline0);

        // ---- stage 2: leaves under each family's root; with both, the lower
        // estimated lookup cost wins
        const int first = want_lin ? lin : spl;
        if ((rc = leaves_for(first, 0, M->leaves)) != IDX_OK) break;
        if (both && (rc = leaves_for(spl, 1, alt)) != IDX_OK) break;
        if (hipMemcpyAsync(hc.stats, ctl->stats, sizeof(hc.stats), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            rc = IDX_ERR_HIP;
            break;
        }
        int won = first, fam = 0;
        if (both && window_cost(hc.stats[1][0] / (double)n, true) < window_cost(hc.stats[0][0] / (double)n, false)) {
            won = spl;
            fam = 1;
            std::swap(M->leaves, alt);
        }
        if (won == kSpline0 + 1) std::swap(M->spline, bins2);
        M->root = hc.roots[won];
        M->stats.root_loss = hc.acc[won][5];
        M->stats.leaf_loss = hc.stats[fam][2];
        M->stats.mean_window = n ? hc.stats[fam][0] / (double)n : 0.0;
        M->stats.max_window = hc.stats[fam][1];
    } while (0);
    give_back();
    return rc;
}

}  // namespace

int learn(idx_index *h, uint32_t L, uint32_t epochs, uint32_t feature, hipStream_t s) {
    if (h->layout != IDX_BS || h->n == 0) return IDX_ERR_ARG;
    if (L == 0 || L > (1u << 26) || epochs == 0 || epochs > 16 || feature > IDX_FEATURE_SPLINE) return IDX_ERR_ARG;
    drop_model(h, s, h->params.leaf_lines == 1);
    LearnedModel *M = new (std::nothrow) LearnedModel();
    if (!M) return IDX_ERR_NOMEM;
    M->leaves = (LeafRec *)h->alloc.get((size_t)L * sizeof(LeafRec), s);
    if (M->leaves && (feature == IDX_FEATURE_AUTO || feature == IDX_FEATURE_SPLINE)) {
        M->spline = (SplineBin *)h->alloc.get((size_t)spline_bins(h->n) * sizeof(SplineBin), s);
        if (!M->spline) {
            h->alloc.put(M->leaves, s);
            M->leaves = nullptr;
        }
    }
    if (!M->leaves) {
        delete M;
        return IDX_ERR_NOMEM;
    }
    h->learned = M;
    M->stats.leaves = L;
    M->stats.epochs = epochs;
    int rc;
    if (h->u64) rc = h->aos ? train_t<uint64_t, true>(h, L, epochs, feature, s) : train_t<uint64_t, false>(h, L, epochs, feature, s);
    else rc = h->aos ? train_t<uint32_t, true>(h, L, epochs, feature, s) : train_t<uint32_t, false>(h, L, epochs, feature, s);
    if (rc != IDX_OK) {
        drop_model(h, s);
        return rc;
    }
    M->stats.feature = M->root.mode;
    M->stats.root_a0 = M->root.a0;
    M->stats.root_a1 = M->root.a1;
    M->stats.segments = M->root.mode == IDX_FEATURE_SPLINE ? M->root.nb : 0;
    M->stats.bin_feature = M->root.mode == IDX_FEATURE_SPLINE ? M->root.bfeat : 0;
    if (M->root.mode != IDX_FEATURE_SPLINE && M->spline) {
        h->alloc.put(M->spline, s);
        M->spline = nullptr;
    }
    if (h->params.leaf_lines == 1) {
        rc = ensure_lines(h, s);
        if (rc != IDX_OK) {
            drop_model(h, s);
            return rc;
        }
    }
    return IDX_OK;
}

void drop_model(idx_index *h, hipStream_t s, bool keep_lines) {
    void *lines = h->learned ? h->learned->lines : nullptr;
    if (h->spare_lines && (!keep_lines || lines)) {
        h->alloc.put(h->spare_lines, s);
        h->spare_lines = nullptr;
        h->spare_lines_bytes = 0;
    }
    if (!h->learned) return;
    h->alloc.put(h->learned->leaves, s);
    if (h->learned->spline) h->alloc.put(h->learned->spline, s);
    if (lines && keep_lines) {
        h->spare_lines = lines;
        h->spare_lines_bytes = (size_t)h->learned->root.L * kLineBytes;
    } else if (lines) {
        h->alloc.put(lines, s);
    }
    delete h->learned;
    h->learned = nullptr;
}

int learn_stats(const idx_index *h, idx_learn_stats *out) {
    if (!h->learned) return IDX_ERR_ARG;
    *out = h->learned->stats;
    return IDX_OK;
}

int learn_export(const idx_index *h, void *leaves_out, hipStream_t s) {
    if (!h->learned) return IDX_ERR_ARG;
    if (!leaves_out) return IDX_OK;
    IDX_HIP(hipMemcpyAsync(leaves_out, h->learned->leaves, (size_t)h->learned->root.L * sizeof(LeafRec),
                           hipMemcpyDeviceToDevice, s));
    return IDX_OK;
}

// ---------------------------------------------------------------- lookups

namespace {

// Window scan on the array-of-structures sorted array (one key and its row
// ID per slot): keys of slots [b, b + len) (len <= W) below x, and the row ID
// of the first slot equal to x.  Slots are read with independent loads; the
// row ID comes with its key, so a hit costs no further line.  A 16-byte slot
// holding a 64-bit key is one 16-byte vector load.
template <typename K, int W>
__device__ __forceinline__ uint32_t count_below_slots(const Load<K, true> &L, uint64_t b, uint32_t len, K x,
                                                      bool &eq, uint32_t &row, bool two = true) {
    uint32_t cnt = 0;
    bool e = false;
    uint32_t rw = kMiss;
    if (sizeof(K) == 8 && L.stride == 16) {
        uint4 w[W];
#pragma unroll
        for (int j = 0; j < W; ++j)
            if ((uint32_t)j < len) w[j] = *(const uint4 *)(L.base + (b + j) * 16);
#pragma unroll
        for (int j = 0; j < W; ++j) {
            if ((uint32_t)j >= len) continue;
            const K k = (K)(((uint64_t)w[j].y << 32) | w[j].x);
            cnt += k < x ? 1u : 0u;
            if (!e && k == x) {
                e = true;
                rw = w[j].z;
            }
        }
    } else {
        // Two rounds: first the slots whose key lies in the 128-byte line of
        // the window's first key; the rest only when all of those are below x
        // (keys ascend, so otherwise the lower bound is already among them).
        // A window within one line costs that line alone.
        K k[W];
        bool got[W];
        const uint64_t line0 = (uint64_t)(uintptr_t)(L.base + b * (uint64_t)L.stride) >> 7;
        uint32_t n1 = 0;
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const uint64_t a = (uint64_t)(uintptr_t)(L.base + (b + j) * (uint64_t)L.stride);
            got[j] = (uint32_t)j < len && (!two || ((a + sizeof(K) - 1) >> 7) == line0);
            k[j] = got[j] ? L.key(b + j) : K(0);
            n1 += got[j] ? 1u : 0u;
        }
#pragma unroll
        for (int j = 0; j < W; ++j) cnt += (got[j] && k[j] < x) ? 1u : 0u;
        if (two && cnt == n1 && n1 < len) {
#pragma unroll
            for (int j = 0; j < W; ++j) {
                if ((uint32_t)j >= len || got[j]) continue;
                k[j] = L.key(b + j);
                got[j] = true;
                cnt += k[j] < x ? 1u : 0u;
            }
        }
#pragma unroll
        for (int j = 0; j < W; ++j) e |= got[j] && k[j] == x;
        if (e) rw = L.row(b + cnt);
    }
    eq = e;
    row = rw;
    return cnt;
}

// Window scan on the packed array of structures (64-bit key and 32-bit row
// ID per 12-byte slot): the slots [b, b + len) (len <= W) are read as aligned
// 16-byte chunks, every chunk of a round issued at once, and keys and row IDs
// are taken from the registers, so a hit needs no further load.  (Loading the
// row ID after the keys were counted often found its line evicted from L2:
// with hundreds of thousands of lookups in flight per XCD a line does not
// stay there long.)  Two rounds as in count_below_slots: first the chunks of
// the 128-byte line of the window's first chunk, the rest only when every
// slot read so far is below x.  A slot starts at word S + 3 j of the chunks,
// S = (12 b mod 16) / 4 differing from lane to lane: the loads do not depend
// on S (so no lane waits for another's), and each word is selected from the
// four candidates by S after they arrive.
template <int W>
__device__ __forceinline__ uint32_t count_below_packed(const char *__restrict__ base, uint64_t b, uint32_t len,
                                                       uint64_t x, bool &eq, uint32_t &row, bool two) {
    constexpr int NC = (3 * 4 + W * 12 + 15) / 16;  // chunks covering W slots from any word S <= 3
    const char *p0 = base + ((b * 12) & ~(uint64_t)15);
    const uint32_t S = (uint32_t)((b * 12) & 15) >> 2;
    const uint64_t line0 = (uint64_t)(uintptr_t)p0 >> 7;
    const uint32_t end_word = S + 3 * len;  // words [S, end_word) hold the window
    uint4 w[NC];
    uint32_t got = 0;  // bit c: chunk c loaded
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const bool need = (uint32_t)(4 * c) < end_word;
        const bool first = !two || ((uint64_t)(uintptr_t)(p0 + 16 * c) >> 7) == line0;
        w[c] = make_uint4(0u, 0u, 0u, 0u);
        if (need && first) {
            w[c] = *(const uint4 *)(p0 + 16 * c);
            got |= 1u << c;
        }
    }
    auto word = [&](int i) -> uint32_t {  // static i
        const uint4 &v = w[i >> 2];
        return (i & 3) == 0 ? v.x : (i & 3) == 1 ? v.y : (i & 3) == 2 ? v.z : v.w;
    };
    auto pick = [&](int i) -> uint32_t {  // word S + i
        const uint32_t a = word(i), bb = word(i + 1), c = word(i + 2), d = word(i + 3);
        return S == 0 ? a : S == 1 ? bb : S == 2 ? c : d;
    };
    auto slot_in = [&](int j) -> bool {  // all three words of slot j loaded
        const uint32_t k0 = S + 3 * (uint32_t)j;
        return ((got >> (k0 >> 2)) & 1u) && ((got >> ((k0 + 2) >> 2)) & 1u);
    };
    uint32_t cnt = 0, avail = 0;
#pragma unroll
    for (int j = 0; j < W; ++j) {
        const bool in = (uint32_t)j < len && slot_in(j);
        const uint64_t k = ((uint64_t)pick(3 * j + 1) << 32) | pick(3 * j);
        avail += in ? 1u : 0u;
        cnt += (in && k < x) ? 1u : 0u;
    }
    if (two && cnt == avail && avail < len) {
        // every slot read is below x: the lower bound lies further on
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (!((got >> c) & 1u) && (uint32_t)(4 * c) < end_word) {
                w[c] = *(const uint4 *)(p0 + 16 * c);
                got |= 1u << c;
            }
        cnt = 0;
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const uint64_t k = ((uint64_t)pick(3 * j + 1) << 32) | pick(3 * j);
            cnt += ((uint32_t)j < len && k < x) ? 1u : 0u;
        }
    }
    // the lower bound is slot cnt: a hit when its key equals x
    bool e = false;
    uint32_t rw = kMiss;
#pragma unroll
    for (int j = 0; j < W; ++j) {
        const uint64_t k = ((uint64_t)pick(3 * j + 1) << 32) | pick(3 * j);
        if ((uint32_t)j == cnt && (uint32_t)j < len && slot_in(j) && k == x) {
            e = true;
            rw = pick(3 * j + 2);
        }
    }
    eq = e;
    row = rw;
    return cnt;
}

// Windows are narrowed with binary-search steps down to STOP keys: 15 on the
// structure-of-arrays layout (its scan reads 16 keys in 9 vector loads), 7
// on the array of structures (8 slots, each with its row ID).
template <bool AOS>
constexpr uint32_t window_stop() {
    return AOS ? 7u : 15u;
}

template <typename K, int R, bool SORT, bool AOS, bool TWO>
__global__ __launch_bounds__(1024) void k_point_learned(Load<K, AOS> keys, uint64_t n, RootRec root,
                                                        const LeafRec *__restrict__ leaves, QueryIO<K> io) {
    extern __shared__ __align__(16) char smem[];
    constexpr uint32_t STOP = window_stop<AOS>();
    const uint64_t tile = (uint64_t)blockDim.x * R;
    for (uint64_t it = blockIdx.x; it < io.iters; it += gridDim.x) {
        const uint64_t tl = tile_of(it, io.ntiles, io.xcd);
        if (tl >= io.ntiles) continue;
        const uint64_t t0 = tl * tile;
        K x[R];
        uint32_t src[R];
        uint32_t b[R], len[R];  // ranks: n < 2^32
        tile_load<K, R, SORT>(io, smem, t0, x, src);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint64_t w0, wl;
            learned_window(root, leaves, (uint64_t)x[r], w0, wl);
            b[r] = (uint32_t)w0;
            len[r] = tile_valid(io.m, t0, src_of<R, SORT>(src, r)) ? (uint32_t)wl : 0u;
        }
        // The lower bound lies in [b, b + len].  Narrow wide windows with
        // binary-search steps, then read the last <= STOP keys and the key
        // after them in one round of independent loads.
        bool more = true;
        while (more) {
            more = false;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (len[r] > STOP) {
                    const uint32_t half = len[r] >> 1;
                    b[r] = keys.key(b[r] + half - 1) < x[r] ? b[r] + half : b[r];
                    len[r] -= half;
                    more |= len[r] > STOP;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t res = kMiss;
            if (tile_valid(io.m, t0, src_of<R, SORT>(src, r))) {
                const uint64_t sl = ((uint64_t)len[r] + 1) < (n - b[r]) ? ((uint64_t)len[r] + 1) : (n - b[r]);
                bool eq;
                if constexpr (AOS) {
                    uint32_t row;
                    if (sizeof(K) == 8 && keys.stride == 12)
                        (void)count_below_packed<STOP + 1>(keys.base, b[r], (uint32_t)sl, (uint64_t)x[r], eq, row, TWO);
                    else
                        (void)count_below_slots<K, STOP + 1>(keys, b[r], (uint32_t)sl, x[r], eq, row, TWO);
                    if (eq) res = row;
                } else {
                    const uint32_t c = count_below<K, 16>(keys.k, b[r], (uint32_t)sl, x[r], eq, TWO);
                    if (eq) res = keys.r[(uint64_t)b[r] + c];
                }
            }
            tile_put<K, SORT>(io, smem, t0, src_of<R, SORT>(src, r), res);
        }
        tile_flush<K, R, SORT>(io, smem, t0);
    }
}

// ------------------------------------------------------------- leaf lines

// The leaf lines (line layout at line_scan), one thread per 16-byte chunk,
// so that a wave writes eight whole lines.  A workgroup writes 256 leaves,
// which cover one contiguous rank range.  Its keys and row IDs are first
// copied to LDS with consecutive loads, all of them when they fit, else those
// of 128, 64 or 32 leaves at a time.  Bound by HBM: 2^24 lines over 2^26
// 64-bit keys (2 GiB written, 1.3 GB read) in 620 us; 32 leaves at a time
// through a chain of dependent loads and two barriers took 880.
constexpr uint32_t kLinesBlock = 256;   // threads, and leaves per workgroup
constexpr uint32_t kLinesStage = 1536;  // keys staged at most: eight workgroups per CU
template <typename K, bool AOS>
__global__ __launch_bounds__(kLinesBlock) void k_leaf_lines(Load<K, AOS> keys, const LeafRec *__restrict__ leaves,
                                                            uint32_t L, uint4 *__restrict__ lines) {
    __shared__ K s_key[kLinesStage];
    __shared__ uint32_t s_row[kLinesStage], s_base[kLinesBlock + 1];
    const uint32_t l0 = blockIdx.x * kLinesBlock, nl = L - l0 < kLinesBlock ? L - l0 : kLinesBlock;
    if (threadIdx.x < nl) {
        const uint2 bs = *(const uint2 *)&leaves[l0 + threadIdx.x].base;
        s_base[threadIdx.x] = bs.x;
        if (threadIdx.x == nl - 1) s_base[nl] = bs.x + bs.y;
    }
    __syncthreads();
    uint32_t step = kLinesBlock;  // leaves staged together
    for (uint64_t t = s_base[nl] - s_base[0]; t > kLinesStage && step > 32; t >>= 1) step >>= 1;
    for (uint32_t a = 0; a < nl; a += step) {
        const uint32_t b = a + step < nl ? a + step : nl;
        const uint32_t kb = s_base[a], count = s_base[b] - kb;
        const bool staged = count <= kLinesStage;  // workgroup-uniform
        if (a) __syncthreads();  // the keys before are written out
        if (staged) {
            constexpr int U = 4;
            for (uint32_t i0 = 0; i0 < count; i0 += U * kLinesBlock) {
                K k[U];
                uint32_t r[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t i = i0 + u * kLinesBlock + threadIdx.x;
                    if (i < count) {
                        k[u] = keys.key((uint64_t)kb + i);
                        r[u] = keys.row((uint64_t)kb + i);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t i = i0 + u * kLinesBlock + threadIdx.x;
                    if (i < count) {
                        s_key[i] = k[u];
                        s_row[i] = r[u];
                    }
                }
            }
            __syncthreads();
        }
        for (uint32_t t = a * kLineChunks + threadIdx.x; t < b * kLineChunks; t += kLinesBlock) {
            const uint32_t l = t / kLineChunks, c = t % kLineChunks;
            const uint32_t base = s_base[l], size = s_base[l + 1] - base;
            auto key_at = [&](uint32_t j) -> uint64_t {
                return staged ? (uint64_t)s_key[base + j - kb] : (uint64_t)keys.key((uint64_t)base + j);
            };
            auto row_at = [&](uint32_t j) -> uint32_t {
                return staged ? s_row[base + j - kb] : keys.row((uint64_t)base + j);
            };
            constexpr uint32_t C = line_slots<K>();
            constexpr uint32_t KW = sizeof(K) / 4;  // words per key
            uint32_t v[4];
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) {
                const uint32_t wi = 4 * c + i;
                uint32_t x = 0;
                if (wi == 0) {
                    x = base;
                } else if (wi == 1) {
                    x = size;
                } else if (wi < 2 + C * KW) {
                    const uint32_t j = (wi - 2) / KW;
                    if (j < size) {
                        const uint64_t k = key_at(j);
                        x = (KW == 2 && ((wi - 2) & 1u)) ? (uint32_t)(k >> 32) : (uint32_t)k;
                    }
                } else {
                    const uint32_t j = wi - 2 - C * KW;
                    if (j < size) x = row_at(j);
                }
                v[i] = x;
            }
            lines[(uint64_t)l0 * kLineChunks + t] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    }
}

// Answer for x in the window [b, b + len] of the sorted array: halved while
// it spans more than the scan's width, then the short-window scan.
template <typename K, bool AOS>
__device__ __forceinline__ uint32_t window_find(const Load<K, AOS> &keys, uint64_t n, uint64_t b, uint64_t len, K x,
                                                bool two) {
    constexpr uint32_t STOP = window_stop<AOS>();
    while (len > STOP) {
        const uint64_t half = len >> 1;
        b = keys.key(b + half - 1) < x ? b + half : b;
        len -= half;
    }
    const uint64_t sl = (len + 1) < (n - b) ? (len + 1) : (n - b);
    bool eq;
    if constexpr (AOS) {
        uint32_t row;
        if (sizeof(K) == 8 && keys.stride == 12)
            (void)count_below_packed<STOP + 1>(keys.base, b, (uint32_t)sl, (uint64_t)x, eq, row, two);
        else
            (void)count_below_slots<K, STOP + 1>(keys, b, (uint32_t)sl, x, eq, row, two);
        return eq ? row : kMiss;
    } else {
        const uint32_t c = count_below<K, 16>(keys.k, b, (uint32_t)sl, x, eq, two);
        return eq ? keys.r[b + c] : kMiss;
    }
}

// The same, kept out of line: called only for the few lookups that go past
// their leaf's line, so the callers' loops over their lookups stay small
// enough to unroll.
template <typename K, bool AOS>
__device__ __noinline__ uint32_t window_find_call(Load<K, AOS> keys, uint64_t n, uint64_t b, uint64_t len, K x,
                                                  bool two) {
    return window_find<K, AOS>(keys, n, b, len, x, two);
}

// Point lookups through the leaf lines, one lane per lookup (the sorted-tile
// form): the R lookups of a lane load their leaves' lines together (eight
// independent 16-byte loads of one line each), then each is answered from
// its registers; a lookup past every key of its line in a larger leaf
// searches the rest of that leaf in the sorted array.
template <typename K, int R, bool SORT, bool AOS, bool TWO>
__global__ __launch_bounds__(256) void k_point_lines(Load<K, AOS> keys, uint64_t n, RootRec root,
                                                     const uint4 *__restrict__ lines, QueryIO<K> io) {
    extern __shared__ __align__(16) char smem[];
    const uint64_t tile = (uint64_t)blockDim.x * R;
    for (uint64_t it = blockIdx.x; it < io.iters; it += gridDim.x) {
        const uint64_t tl = tile_of(it, io.ntiles, io.xcd);
        if (tl >= io.ntiles) continue;
        const uint64_t t0 = tl * tile;
        K x[R];
        uint32_t src[R];
        tile_load<K, R, SORT>(io, smem, t0, x, src);
        uint4 w[R][kLineChunks];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool v = tile_valid(io.m, t0, src_of<R, SORT>(src, r));
            const uint4 *p = lines + (uint64_t)leaf_of(root, (uint64_t)x[r]) * kLineChunks;
#pragma unroll
            for (int c = 0; c < (int)kLineChunks; ++c) w[r][c] = v ? p[c] : make_uint4(0u, 0u, 0u, 0u);
        }
        // answers from the lines first, so that no line is held while the
        // rest of a larger leaf is searched
        uint32_t res[R];
        uint64_t b[R], len[R];
        bool big[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            res[r] = kMiss;
            big[r] = false;
            b[r] = len[r] = 0;
            if (tile_valid(io.m, t0, src_of<R, SORT>(src, r))) {
                uint32_t cnt, row;
                bool eq;
                if (line_scan<K>(w[r], x[r], cnt, eq, row, b[r], len[r])) {
                    if (eq) res[r] = row;
                } else {
                    big[r] = true;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (big[r]) res[r] = window_find_call<K, AOS>(keys, n, b[r], len[r], x[r], TWO);
            tile_put<K, SORT>(io, smem, t0, src_of<R, SORT>(src, r), res[r]);
        }
        tile_flush<K, R, SORT>(io, smem, t0);
    }
}

// Point lookups through the leaf lines, two lanes per lookup: lane h of a
// pair loads the line's half h (four 16-byte loads).  A lane reading a whole
// line with eight loads makes the memory system serve far fewer random lines
// per second than lanes sharing it (measured on MI355X: 13 against 48 G
// lines/s).  Each lane counts its half's keys below x and at most x; the pair
// adds both counts with one exchange each, and a hit is a key equal to x
// (more keys at most x than below it).  The row IDs lie in the upper half, so
// its lane writes the answer; when x lies past every key of the line in a
// leaf that has more, the lower lane searches the rest of the leaf in the
// sorted array and writes.
template <typename K, int R, bool AOS, bool TWO>
__global__ __launch_bounds__(256) void k_point_lines_pair(Load<K, AOS> keys, uint64_t n, RootRec root,
                                                          const uint4 *__restrict__ lines, QueryIO<K> io) {
    constexpr uint32_t C = line_slots<K>();
    constexpr uint32_t KW = sizeof(K) / 4;  // words per key
    constexpr uint32_t R0 = 2 + C * KW;     // first row ID word (>= 16: in the upper half)
    static_assert(R0 >= 16, "row IDs in the upper half of the line");
    const uint32_t hf = threadIdx.x & 1u;
    const uint64_t pairs = blockDim.x / 2, pi = threadIdx.x / 2;
    const uint64_t tile = pairs * R;
    for (uint64_t it = blockIdx.x; it < io.iters; it += gridDim.x) {
        const uint64_t tl = tile_of(it, io.ntiles, io.xcd);
        if (tl >= io.ntiles) continue;
        const uint64_t t0 = tl * tile;
        K x[R];
        bool v[R];
        uint4 w[R][4];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t qi = t0 + (uint64_t)r * pairs + pi;
            v[r] = qi < io.m;
            x[r] = v[r] ? io.q[qi] : K(0);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint4 *p = lines + (uint64_t)leaf_of(root, (uint64_t)x[r]) * kLineChunks + 4 * hf;
#pragma unroll
            for (int c = 0; c < 4; ++c) w[r][c] = v[r] ? p[c] : make_uint4(0u, 0u, 0u, 0u);
        }
        uint32_t res[R];
        uint64_t b[R], len[R];
        bool big[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            auto word = [&](int i) -> uint32_t {  // static i: word 16 hf + i of the line
                const uint4 &c = w[r][i >> 2];
                return (i & 3) == 0 ? c.x : (i & 3) == 1 ? c.y : (i & 3) == 2 ? c.z : c.w;
            };
            res[r] = kMiss;
            b[r] = len[r] = 0;
            const uint32_t other = __shfl_xor(w[r][0].y, 1);
            const uint32_t size = hf ? other : w[r][0].y;
            uint32_t lt = 0, le = 0;
#pragma unroll
            for (int i = 0; i < 16; i += (int)KW) {
                const uint32_t wi = 16 * hf + (uint32_t)i;
                K key;
                if constexpr (KW == 2) key = ((uint64_t)word(i + 1) << 32) | word(i);
                else key = word(i);
                const bool in = wi >= 2 && wi < R0 && (wi - 2) / KW < size;
                lt += (in && key < x[r]) ? 1u : 0u;
                le += (in && key <= x[r]) ? 1u : 0u;
            }
            lt += __shfl_xor(lt, 1);
            le += __shfl_xor(le, 1);
            // past every key of the line in a leaf that has more: the rest
            // of the leaf is searched in the sorted array (by the lower lane)
            big[r] = lt == C && size > C;
            if (!big[r]) {
                if (le > lt) {
                    const uint32_t ri = R0 - 16 + lt;  // the row ID's word in the upper half
                    uint32_t row = 0;
#pragma unroll
                    for (int i = 0; i < 16; ++i) row = (uint32_t)i == ri ? word(i) : row;
                    res[r] = row;
                }
            } else if (hf == 0) {
                b[r] = (uint64_t)w[r][0].x + C;
                len[r] = size - C;
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t qi = t0 + (uint64_t)r * pairs + pi;
            if (big[r] && hf == 0) res[r] = window_find_call<K, AOS>(keys, n, b[r], len[r], x[r], TWO);
            if (v[r] && hf == (big[r] ? 0u : 1u)) io.out[qi] = res[r];
        }
    }
}

}  // namespace

// Write the model's leaf lines unless they are there; not under capture (the
// leaf records' windows then serve).
int ensure_lines(idx_index *h, hipStream_t s) {
    std::lock_guard<std::mutex> lock(h->lazy);
    LearnedModel *M = h->learned;
    if (M->lines || capturing(s)) return IDX_OK;
    const uint32_t L = M->root.L;
    const size_t bytes = (size_t)L * kLineBytes;
    uint4 *lines = nullptr;
    if (h->spare_lines && h->spare_lines_bytes == bytes) {
        lines = (uint4 *)h->spare_lines;  // every line is rewritten below
    } else {
        if (h->spare_lines) h->alloc.put(h->spare_lines, s);
        lines = (uint4 *)h->alloc.get(bytes, s);
    }
    h->spare_lines = nullptr;
    h->spare_lines_bytes = 0;
    if (!lines) return IDX_ERR_NOMEM;
    const uint32_t g = grid_for(L, kLinesBlock);
    if (h->u64) {
        if (h->aos) hipLaunchKernelGGL((k_leaf_lines<uint64_t, true>), dim3(g), dim3(256), 0, s, make_load<uint64_t, true>(h), M->leaves, L, lines);
        else hipLaunchKernelGGL((k_leaf_lines<uint64_t, false>), dim3(g), dim3(256), 0, s, make_load<uint64_t, false>(h), M->leaves, L, lines);
    } else {
        if (h->aos) hipLaunchKernelGGL((k_leaf_lines<uint32_t, true>), dim3(g), dim3(256), 0, s, make_load<uint32_t, true>(h), M->leaves, L, lines);
        else hipLaunchKernelGGL((k_leaf_lines<uint32_t, false>), dim3(g), dim3(256), 0, s, make_load<uint32_t, false>(h), M->leaves, L, lines);
    }
    // waited for once: the next lookup may come on another stream
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) {
        h->alloc.put(lines, s);
        return IDX_ERR_HIP;
    }
    M->lines = lines;
    return IDX_OK;
}

namespace {
// Query IO of a leaf-line launch over tiles of `tile` lookups, and its grid.
template <typename KT>
QueryIO<KT> lines_io(const idx_index *h, const idx_lookup_params &p, const PointIO &pio, uint64_t tile, uint32_t &grid) {
    QueryIO<KT> io{};
    io.q = (const KT *)pio.q;
    io.out = pio.out;
    io.m = pio.m;
    io.local_sort = pio.local_sort ? 1u : 0u;
    io.xcd = pio.xcd ? 1u : 0u;
    io.sort_off = 0;
    io.rounds = p.window_rounds == 1 ? 1u : 2u;
    set_tiles(io, tile);
    uint64_t g = io.iters;
    if (p.persistent) {
        uint64_t cap = (uint64_t)h->cu_count * p.persistent;
        if (io.xcd && cap >= kXcds) cap -= cap % kXcds;
        if (g > cap) g = cap;
    }
    grid = (uint32_t)(g ? (g > 0x7FFFFFFFull ? 0x7FFFFFFFull : g) : 1);
    return io;
}

template <typename KT, int RR>
void launch_lines(idx_index *h, const idx_lookup_params &p, const PointIO &pio, hipStream_t s) {
    const LearnedModel *M = h->learned;
    const uint32_t block = p.block > 256 ? 256u : p.block;
    uint32_t g;
    if (pio.local_sort) {  // one lane per lookup, at most 4 lookups per lane
        constexpr int RS = RR > 4 ? 4 : RR;
        const uint64_t tile = (uint64_t)block * RS;
        const QueryIO<KT> io = lines_io<KT>(h, p, pio, tile, g);
        const size_t smem = sort_lds_bytes((uint32_t)tile, sizeof(KT));
        if (h->aos && io.rounds == 2)
            hipLaunchKernelGGL((k_point_lines<KT, RS, true, true, true>), dim3(g), dim3(block), smem, s,
                               make_load<KT, true>(h), h->n, M->root, M->lines, io);
        else if (h->aos)
            hipLaunchKernelGGL((k_point_lines<KT, RS, true, true, false>), dim3(g), dim3(block), smem, s,
                               make_load<KT, true>(h), h->n, M->root, M->lines, io);
        else if (io.rounds == 2)
            hipLaunchKernelGGL((k_point_lines<KT, RS, true, false, true>), dim3(g), dim3(block), smem, s,
                               make_load<KT, false>(h), h->n, M->root, M->lines, io);
        else
            hipLaunchKernelGGL((k_point_lines<KT, RS, true, false, false>), dim3(g), dim3(block), smem, s,
                               make_load<KT, false>(h), h->n, M->root, M->lines, io);
        return;
    }
    const QueryIO<KT> io = lines_io<KT>(h, p, pio, (uint64_t)(block / 2) * RR, g);
    if (h->aos && io.rounds == 2)
        hipLaunchKernelGGL((k_point_lines_pair<KT, RR, true, true>), dim3(g), dim3(block), 0, s,
                           make_load<KT, true>(h), h->n, M->root, M->lines, io);
    else if (h->aos)
        hipLaunchKernelGGL((k_point_lines_pair<KT, RR, true, false>), dim3(g), dim3(block), 0, s,
                           make_load<KT, true>(h), h->n, M->root, M->lines, io);
    else if (io.rounds == 2)
        hipLaunchKernelGGL((k_point_lines_pair<KT, RR, false, true>), dim3(g), dim3(block), 0, s,
                           make_load<KT, false>(h), h->n, M->root, M->lines, io);
    else
        hipLaunchKernelGGL((k_point_lines_pair<KT, RR, false, false>), dim3(g), dim3(block), 0, s,
                           make_load<KT, false>(h), h->n, M->root, M->lines, io);
}

// Point lookups through the leaf lines: at most 256 threads per workgroup.
int point_lines(idx_index *h, const idx_lookup_params &p, const PointIO &pio, hipStream_t s) {
    const uint32_t R = p.per_lane;
    if (h->u64) {
        switch (R) {
            case 1: launch_lines<uint64_t, 1>(h, p, pio, s); break;
            case 2: launch_lines<uint64_t, 2>(h, p, pio, s); break;
            case 4: launch_lines<uint64_t, 4>(h, p, pio, s); break;
            default: launch_lines<uint64_t, 8>(h, p, pio, s); break;
        }
    } else {
        switch (R) {
            case 1: launch_lines<uint32_t, 1>(h, p, pio, s); break;
            case 2: launch_lines<uint32_t, 2>(h, p, pio, s); break;
            case 4: launch_lines<uint32_t, 4>(h, p, pio, s); break;
            default: launch_lines<uint32_t, 8>(h, p, pio, s); break;
        }
    }
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

}  // namespace

int point_learned(idx_index *h, const idx_lookup_params &p, const PointIO &pio, hipStream_t s) {
    if (p.leaf_lines == 1) {
        const int rc = ensure_lines(h, s);
        if (rc != IDX_OK) return rc;
        if (h->learned->lines) return point_lines(h, p, pio, s);
    }
    const LearnedModel *M = h->learned;
    const uint32_t block = p.block;
    const uint32_t R = p.per_lane;
    const uint64_t tile = (uint64_t)block * R;
#define IDX_LEARNED_KERNELS(KT, RR, TW)                                                                     \
    do {                                                                                                    \
        if (h->aos && io.local_sort)                                                                        \
            hipLaunchKernelGGL((k_point_learned<KT, RR, true, true, TW>), dim3(g), dim3(block), smem, s,    \
                               make_load<KT, true>(h), h->n, M->root, M->leaves, io);                       \
        else if (h->aos)                                                                                    \
            hipLaunchKernelGGL((k_point_learned<KT, RR, false, true, TW>), dim3(g), dim3(block), smem, s,   \
                               make_load<KT, true>(h), h->n, M->root, M->leaves, io);                       \
        else if (io.local_sort)                                                                             \
            hipLaunchKernelGGL((k_point_learned<KT, RR, true, false, TW>), dim3(g), dim3(block), smem, s,   \
                               make_load<KT, false>(h), h->n, M->root, M->leaves, io);                      \
        else                                                                                                \
            hipLaunchKernelGGL((k_point_learned<KT, RR, false, false, TW>), dim3(g), dim3(block), smem, s,  \
                               make_load<KT, false>(h), h->n, M->root, M->leaves, io);                      \
    } while (0)
#define IDX_LEARNED_LAUNCH(KT, RR)                                                                          \
    do {                                                                                                    \
        QueryIO<KT> io{};                                                                                   \
        io.q = (const KT *)pio.q;                                                                           \
        io.out = pio.out;                                                                                   \
        io.m = pio.m;                                                                                       \
        io.local_sort = pio.local_sort ? 1u : 0u;                                                           \
        io.xcd = pio.xcd ? 1u : 0u;                                                                         \
        io.sort_off = 0;                                                                                    \
        io.rounds = p.window_rounds == 1 ? 1u : 2u;                                                 \
        set_tiles(io, tile);                                                                                \
        uint64_t grid = io.iters;                                                                           \
        if (p.persistent) {                                                                         \
            uint64_t cap = (uint64_t)h->cu_count * p.persistent;                                    \
            if (io.xcd && cap >= kXcds) cap -= cap % kXcds;                                                 \
            if (grid > cap) grid = cap;                                                                     \
        }                                                                                                   \
        const uint32_t g = (uint32_t)(grid ? (grid > 0x7FFFFFFFull ? 0x7FFFFFFFull : grid) : 1);            \
        const size_t smem = io.local_sort ? sort_lds_bytes((uint32_t)tile, sizeof(KT)) : 0;                 \
        if (io.rounds == 2) IDX_LEARNED_KERNELS(KT, RR, true);                                              \
        else IDX_LEARNED_KERNELS(KT, RR, false);                                                            \
    } while (0)
    if (h->u64) {
        switch (R) {
            case 1: IDX_LEARNED_LAUNCH(uint64_t, 1); break;
            case 2: IDX_LEARNED_LAUNCH(uint64_t, 2); break;
            case 4: IDX_LEARNED_LAUNCH(uint64_t, 4); break;
            default: IDX_LEARNED_LAUNCH(uint64_t, 8); break;
        }
    } else {
        switch (R) {
            case 1: IDX_LEARNED_LAUNCH(uint32_t, 1); break;
            case 2: IDX_LEARNED_LAUNCH(uint32_t, 2); break;
            case 4: IDX_LEARNED_LAUNCH(uint32_t, 4); break;
            default: IDX_LEARNED_LAUNCH(uint32_t, 8); break;
        }
    }
#undef IDX_LEARNED_LAUNCH
#undef IDX_LEARNED_KERNELS
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

namespace {
// Rank of the first key >= x through the model (the window holds it).
template <typename K, bool AOS>
__device__ __forceinline__ uint64_t model_lower_rank(const Load<K, AOS> &keys, uint64_t n, const RootRec &root,
                                                     const LeafRec *__restrict__ leaves, K x) {
    if constexpr (!AOS) {
        return learned_lower_rank(keys.k, n, root, leaves, x);
    } else {
        uint64_t b, len;
        learned_window(root, leaves, (uint64_t)x, b, len);
        while (len > window_stop<true>()) {
            const uint64_t half = len >> 1;
            b = keys.key(b + half - 1) < x ? b + half : b;
            len -= half;
        }
        bool eq;
        uint32_t row;
        return b + count_below_slots<K, window_stop<true>() + 1>(keys, b, (uint32_t)len, x, eq, row);
    }
}

template <typename K, bool AOS>
__global__ __launch_bounds__(256) void k_range_count_learned(Load<K, AOS> keys, uint64_t n, RootRec root,
                                                             const LeafRec *__restrict__ leaves,
                                                             const K *__restrict__ lo, const K *__restrict__ hi,
                                                             uint64_t m, uint32_t *__restrict__ first,
                                                             uint64_t *__restrict__ count) {
    const uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= m) return;
    const K L = lo[q], U = hi[q];
    uint64_t r0 = 0, r1 = 0;
    if (L <= U) {
        r0 = model_lower_rank(keys, n, root, leaves, L);
        r1 = (U == ~K(0)) ? n : model_lower_rank(keys, n, root, leaves, (K)(U + 1));
    }
    first[q] = (uint32_t)r0;
    count[q] = r1 > r0 ? r1 - r0 : 0;
}

// Lower-bound rank of x in the window [b, b + len] of the sorted array.
template <typename K, bool AOS>
__device__ __forceinline__ uint64_t window_lower_rank(const Load<K, AOS> &keys, uint64_t b, uint64_t len, K x) {
    constexpr uint32_t STOP = window_stop<AOS>();
    while (len > STOP) {
        const uint64_t half = len >> 1;
        b = keys.key(b + half - 1) < x ? b + half : b;
        len -= half;
    }
    bool eq;
    uint32_t row;
    if constexpr (AOS) return b + count_below_slots<K, STOP + 1>(keys, b, (uint32_t)len, x, eq, row);
    else return b + count_below<K, 16>(keys.k, b, (uint32_t)len, x, eq);
}

// Lower-bound rank of x from half hf of its leaf's line (w), as two lanes of
// a pair hold it (both call this together; the lower lane gets the rank):
// the base rank plus the line's keys below x, or, when x lies past every key
// of the line in a leaf that has more, a search of the rest of the leaf by
// the lower lane.
template <typename K, bool AOS>
__device__ __forceinline__ uint64_t pair_lower_rank(const Load<K, AOS> &keys, const uint4 (&w)[4], uint32_t hf, K x) {
    constexpr uint32_t C = line_slots<K>();
    constexpr uint32_t KW = sizeof(K) / 4;
    constexpr uint32_t R0 = 2 + C * KW;
    auto word = [&](int i) -> uint32_t {  // static i
        const uint4 &c = w[i >> 2];
        return (i & 3) == 0 ? c.x : (i & 3) == 1 ? c.y : (i & 3) == 2 ? c.z : c.w;
    };
    const uint32_t other = __shfl_xor(w[0].y, 1);
    const uint32_t size = hf ? other : w[0].y;
    uint32_t lt = 0;
#pragma unroll
    for (int i = 0; i < 16; i += (int)KW) {
        const uint32_t wi = 16 * hf + (uint32_t)i;
        K key;
        if constexpr (KW == 2) key = ((uint64_t)word(i + 1) << 32) | word(i);
        else key = word(i);
        lt += (wi >= 2 && wi < R0 && (wi - 2) / KW < size && key < x) ? 1u : 0u;
    }
    lt += __shfl_xor(lt, 1);
    if (lt < C || size <= C) return (uint64_t)w[0].x + lt;
    if (hf != 0) return 0;
    return window_lower_rank<K, AOS>(keys, (uint64_t)w[0].x + C, size - C, x);
}

// Range counts through the leaf lines, two lanes per range (each loads one
// half of both bounds' lines, all eight loads together); the lower lane
// writes the range's first rank and count.
template <typename K, bool AOS>
__global__ __launch_bounds__(256) void k_range_count_lines(Load<K, AOS> keys, uint64_t n, RootRec root,
                                                           const uint4 *__restrict__ lines, const K *__restrict__ lo,
                                                           const K *__restrict__ hi, uint64_t m,
                                                           uint32_t *__restrict__ first, uint64_t *__restrict__ count) {
    const uint32_t hf = threadIdx.x & 1u;
    const uint64_t q = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 1;
    const bool live = q < m;  // the same for both lanes of a pair
    const K L = live ? lo[q] : K(0), U = live ? hi[q] : K(0);
    const bool act = live && L <= U, top = U == ~K(0);
    const K x1 = top ? U : (K)(U + 1);
    uint4 w0[4], w1[4];
    const uint4 *p0 = lines + (uint64_t)leaf_of(root, (uint64_t)L) * kLineChunks + 4 * hf;
    const uint4 *p1 = lines + (uint64_t)leaf_of(root, (uint64_t)x1) * kLineChunks + 4 * hf;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        w0[c] = act ? p0[c] : make_uint4(0u, 0u, 0u, 0u);
        w1[c] = act && !top ? p1[c] : make_uint4(0u, 0u, 0u, 0u);
    }
    const uint64_t r0 = pair_lower_rank<K, AOS>(keys, w0, hf, L);
    const uint64_t r1u = pair_lower_rank<K, AOS>(keys, w1, hf, x1);
    if (!live || hf != 0) return;
    const uint64_t r1 = !act ? 0 : top ? n : r1u;
    first[q] = act ? (uint32_t)r0 : 0u;
    count[q] = act && r1 > r0 ? r1 - r0 : 0;
}

template <typename K, bool AOS>
void launch_range_count(const idx_index *h, const void *lo, const void *hi, uint64_t m, uint32_t *first,
                        uint64_t *count, hipStream_t s) {
    const LearnedModel *M = h->learned;
    if (M->lines && h->params.leaf_lines == 1)
        hipLaunchKernelGGL((k_range_count_lines<K, AOS>), dim3(grid_for(2 * m, 256)), dim3(256), 0, s,
                           make_load<K, AOS>(h), h->n, M->root, M->lines, (const K *)lo, (const K *)hi, m, first,
                           count);
    else
        hipLaunchKernelGGL((k_range_count_learned<K, AOS>), dim3(grid_for(m, 256)), dim3(256), 0, s,
                           make_load<K, AOS>(h), h->n, M->root, M->leaves, (const K *)lo, (const K *)hi, m, first,
                           count);
}
}  // namespace

int range_count_learned(idx_index *h, const void *lo, const void *hi, uint64_t m, uint32_t *first, uint64_t *count,
                        bool may_alloc, hipStream_t s) {
    if (h->params.leaf_lines == 1 && may_alloc) {
        const int rc = ensure_lines(h, s);
        if (rc != IDX_OK) return rc;
    }
    if (h->u64) {
        if (h->aos) launch_range_count<uint64_t, true>(h, lo, hi, m, first, count, s);
        else launch_range_count<uint64_t, false>(h, lo, hi, m, first, count, s);
    } else {
        if (h->aos) launch_range_count<uint32_t, true>(h, lo, hi, m, first, count, s);
        else launch_range_count<uint32_t, false>(h, lo, hi, m, first, count, s);
    }
    IDX_LAUNCH_CHECK();
    return IDX_OK;
}

// ----------------------------------------------------- gradient evaluation

namespace {
// leaf records with parameters given as (b0, b1) pairs
template <typename K, bool AOS>
__global__ void k_set_leaf_params(Load<K, AOS> keys, const uint32_t *__restrict__ base, LeafRec *leaves,
                                  const float *ab, uint32_t L) {
    const uint32_t l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= L) return;
    LeafRec r = new_leaf(keys, base[l], base[l + 1]);
    r.b0 = ab[2 * l];
    r.b1 = ab[2 * l + 1];
    leaves[l] = r;
}

template <typename K, bool AOS>
int eval_t(idx_index *h, uint32_t mode, const float *root_ab, uint32_t L, const float *leaf_ab, double *root_acc_h,
           double *leaf_acc_d, hipStream_t s) {
    const uint64_t n = h->n;
    const Load<K, AOS> keys = make_load<K, AOS>(h);
    const size_t leaf_b = up256((size_t)L * sizeof(LeafRec)), ctl_b = up256(sizeof(TrainCtl));
    char *tmp = (char *)h->alloc.get(ctl_b + leaf_b + bounds_bytes(L), s);
    if (!tmp) return IDX_ERR_NOMEM;
    TrainCtl *ctl = (TrainCtl *)tmp;
    LeafRec *leaves = (LeafRec *)(tmp + ctl_b);
    char *bounds = tmp + ctl_b + leaf_b;
    double *racc = ctl->acc[0];
    int rc = IDX_OK;
    do {
        TrainCtl hc{};
        hc.roots[0] = RootRec{root_ab[0], root_ab[1], mode, L};
        if (hipMemcpyAsync(ctl, &hc, sizeof(hc), hipMemcpyHostToDevice, s) != hipSuccess) { rc = IDX_ERR_HIP; break; }
        hipLaunchKernelGGL((k_root_accum<K, AOS, kSumX | kSumGrad | kSumLoss, false>), dim3(root_blocks(n)), dim3(LT), 0,
                           s, keys, n, ctl->roots, 1u, racc);
        if (leaf_ab && leaf_acc_d) {
            const uint32_t cblocks = grid_for((n + CHUNK - 1) / CHUNK, LT);
            rc = leaf_bounds<K, AOS>(keys, n, ctl->roots, L, bounds, ctl->ngaps, s);
            if (rc != IDX_OK) break;
            hipLaunchKernelGGL((k_set_leaf_params<K, AOS>), dim3(grid_for(L, 256)), dim3(256), 0, s, keys,
                               (const uint32_t *)bounds, leaves, leaf_ab, L);
            const uint32_t cap = stage_cap(n, L);
            hipLaunchKernelGGL((k_leaf_accum_small<K, AOS>), dim3(grid_for(L, kLeafBlock)), dim3(kLeafBlock),
                               (size_t)cap * sizeof(K), s, keys, leaves, L, leaf_acc_d, ctl->big, cap);
            hipLaunchKernelGGL((k_leaf_accum_big<K, AOS>), dim3(cblocks), dim3(LT), 0, s, keys, n, ctl->roots, leaves,
                               leaf_acc_d, ctl->big);
        }
        if (hipGetLastError() != hipSuccess) { rc = IDX_ERR_HIP; break; }
        if (hipMemcpyAsync(root_acc_h, racc, NACC * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) { rc = IDX_ERR_HIP; break; }
    } while (0);
    h->alloc.put(tmp, s);
    return rc;
}
}  // namespace

int learn_eval(idx_index *h, uint32_t mode, const float *root_ab, uint32_t L, const float *leaf_ab, double *root_acc,
               double *leaf_acc, hipStream_t s) {
    if (h->layout != IDX_BS || h->n == 0) return IDX_ERR_ARG;
    if (mode != IDX_FEATURE_LINEAR && mode != IDX_FEATURE_LOG) return IDX_ERR_ARG;
    if (L == 0 || L > (1u << 26) || !root_ab || !root_acc) return IDX_ERR_ARG;
    if (h->u64)
        return h->aos ? eval_t<uint64_t, true>(h, mode, root_ab, L, leaf_ab, root_acc, leaf_acc, s)
                      : eval_t<uint64_t, false>(h, mode, root_ab, L, leaf_ab, root_acc, leaf_acc, s);
    return h->aos ? eval_t<uint32_t, true>(h, mode, root_ab, L, leaf_ab, root_acc, leaf_acc, s)
                  : eval_t<uint32_t, false>(h, mode, root_ab, L, leaf_ab, root_acc, leaf_acc, s);
}

}  // namespace idx
