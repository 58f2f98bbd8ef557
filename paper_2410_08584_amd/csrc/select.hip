// Adaptive count and important-token set (Eq. (7), Eq. (9); Algorithm 1 steps 3-5).
//
// The definition is "sort descending, cumulative sum, first crossing of
// tau * total, then top-k by the normalised score".  Neither step needs the
// sorted sequence itself:
//   * the first crossing of the sorted cumulative sum is found by a radix
//     descent over the 31-bit order-preserving image of the fp32 scores: per
//     digit, an LDS histogram of counts and of exact integer sums
//     (floor(x * 2^40), so the result is independent of summation order), a
//     descending scan over the bins, and the bin where the running sum crosses
//     the target; in the end the remaining candidates are equal and the count
//     follows by one integer division;
//   * the top-k set is {score > v*} plus the lowest-indexed ties at v*, where
//     v* is the k-th largest value, found by the same descent on counts;
//   * the set is written in ascending position.
// One 1024-thread workgroup per selection unit.  Up to n = 32768 the keys of both vectors stay in
// its registers (select_reg_kernel).  Longer vectors are re-read from memory per 8-bit digit and pass
// through LDS block by block for the emission (select_kernel), or, with a workspace, have their first
// digit counted by the whole chip (select_hist_kernel, select_tail_kernel).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "launch.h"
#include "select_dev.h"

namespace zipvl {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelMaxLdsKeys = 27648;      // of the long-vector kernels: 108 KiB of keys beside the 32 KiB histogram
constexpr int kSelRep = 16, kSelRepStride = 257;    // histogram replicas and their spacing in slots

struct SelShared {
    unsigned long long hist[kSelRep * kSelRepStride];   // packed (count, integer sum) slots, or plain 32-bit counts
    unsigned long long folded[256];
    uint32_t wave_cnt[kSelWaves];
    uint32_t wave_eq[kSelWaves];
    unsigned long long target;
    unsigned long long base_sum;
    uint32_t base_cnt;
    uint32_t sel_digit;
    uint32_t sel_cnt;      // elements in the selected bin
    uint32_t sole_key;     // the key of a bin's only element
    int k;
};

// Order-preserving keys of a unit's vector, read from memory by every sweep.
struct Keys {
    const float* x;
    int n;
    template <typename F>
    __device__ __forceinline__ void for_each(F&& f) const {
#pragma unroll 4
        for (int j = threadIdx.x; j < n; j += kSelThreads) f(j, orderable(x[j]));
    }
};

__device__ __forceinline__ void fill_keys(uint32_t* dst, const float* __restrict__ x, int n) {
#pragma unroll 8
    for (int j = threadIdx.x; j < n; j += kSelThreads) dst[j] = orderable(x[j]);
}

// One descent over the 31 key bits in four digits, exponent byte first (8 + 8 + 8 + 7 bits).  The
// first two digits see many elements and spread them over kRep histogram replicas chosen by the
// lane (replica r of digit v sits at slot r * 257 + v: the lanes of a wave that share a digit hit
// different banks, and a fold over the replicas reads consecutive slots); later digits only see the
// few elements that share the prefix and use one replica.  WITH_SUM: a histogram slot packs the
// element count (bits 41..63) over the integer score sum (bits 0..40, sum of a unit < 2^41), one LDS
// atomic per element, and the descent crosses on the sum (target fixed after the first digit from
// the grand total); otherwise slots are plain counts and the descent crosses on cnt_target.
constexpr int kRep = kSelRep, kRepStride = kSelRepStride;

template <bool WITH_SUM>
__device__ void radix_descent(const Keys& keys, double tau, uint32_t cnt_target,
                              SelShared& sh, uint32_t& prefix_out, uint32_t& base_cnt_out,
                              unsigned long long& base_sum_out, bool& degenerate)
{
    const int tid = threadIdx.x;
    uint32_t* cnt_hist = reinterpret_cast<uint32_t*>(sh.hist);
    uint32_t prefix = 0, mask = 0, base_cnt = 0;
    unsigned long long base_sum = 0;
    degenerate = false;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = pass < 3 ? 23 - 8 * pass : 0;
        const uint32_t dmask = pass < 3 ? 255u : 127u;
        const bool replicated = pass < 2;
        const int slots = replicated ? kRep * kRepStride : 256;
        const int rep_off = replicated ? (tid & (kRep - 1)) * kRepStride : 0;
        for (int i = tid; i < slots; i += kSelThreads) {
            if (WITH_SUM) sh.hist[i] = 0; else cnt_hist[i] = 0;
        }
        __syncthreads();
        keys.for_each([&](int, uint32_t key) {
            if ((key & mask) == prefix) {
                const int slot = rep_off + ((key >> shift) & dmask);
                if (WITH_SUM) atomicAdd(&sh.hist[slot], (1ull << kSumBits) + fixed40_of_key(key));
                else atomicAdd(&cnt_hist[slot], 1u);
            }
        });
        __syncthreads();
        if (replicated) {                                   // fold the replicas of bin `tid` into replica 0
            if (tid < 256) {
                uint32_t cc = 0;
                unsigned long long ss = 0;
#pragma unroll
                for (int r = 0; r < kRep; ++r) {
                    if (WITH_SUM) ss += sh.hist[r * kRepStride + tid];   // count and sum fields add without carry between them
                    else cc += cnt_hist[r * kRepStride + tid];
                }
                if (WITH_SUM) sh.folded[tid] = ss; else reinterpret_cast<uint32_t*>(sh.folded)[tid] = cc;
            }
            __syncthreads();
        }
        if (tid < 64) {
            // lane l owns bins 255-4l .. 252-4l (descending value order)
            const unsigned long long* h64 = replicated ? sh.folded : sh.hist;
            const uint32_t* h32 = reinterpret_cast<const uint32_t*>(h64);
            uint32_t c[4], lc = 0;
            unsigned long long s[4], ls = 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int bin = 255 - (4 * tid + t);
                if (WITH_SUM) {
                    const unsigned long long v = h64[bin];
                    c[t] = (uint32_t)(v >> kSumBits);
                    s[t] = v & ((1ull << kSumBits) - 1ull);
                } else {
                    c[t] = h32[bin];
                    s[t] = 0;
                }
                lc += c[t]; ls += s[t];
            }
            const uint32_t ic = wave_scan(lc);
            const unsigned long long is = WITH_SUM ? wave_scan(ls) : 0ull;
            unsigned long long target;
            if (WITH_SUM) {
                if (pass == 0) {
                    const unsigned long long W = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(is >> 32), 63) << 32) |
                                                 (uint32_t)__builtin_amdgcn_readlane((int)is, 63);
                    // ceil(tau * W): one IEEE double multiply, then ceil (W < 2^53)
                    const double prod = tau * (double)W;
                    target = (unsigned long long)ceil(prod);
                    if (tid == 0) sh.target = target;
                } else {
                    target = sh.target;
                }
            } else {
                target = cnt_target;
            }
            uint32_t rc = base_cnt + (ic - lc);
            unsigned long long rs = base_sum + (is - ls);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool cross = WITH_SUM ? (rs < target && target <= rs + s[t])
                                            : ((unsigned long long)rc < target && target <= (unsigned long long)rc + c[t]);
                if (cross) {
                    sh.sel_digit = 255 - (4 * tid + t);
                    sh.base_cnt = rc;
                    sh.base_sum = rs;
                    sh.sel_cnt = c[t];
                }
                rc += c[t];
                rs += s[t];
            }
        }
        __syncthreads();
        if (WITH_SUM && sh.target == 0ull) { degenerate = true; break; }   // all scores zero
        prefix |= sh.sel_digit << shift;
        mask |= dmask << shift;
        base_cnt = sh.base_cnt;
        base_sum = sh.base_sum;
        if (pass < 3 && sh.sel_cnt == 1u) {
            // One element left under this prefix: the remaining digits are its own.  One sweep fetches the key
            // (the counts and sums above it are already final) instead of a histogram pass per digit.
            keys.for_each([&](int, uint32_t key) {
                if ((key & mask) == prefix) sh.sole_key = key;
            });
            __syncthreads();
            prefix = sh.sole_key;
            break;
        }
    }
    prefix_out = prefix;
    base_cnt_out = base_cnt;
    base_sum_out = base_sum;
}

__global__ __launch_bounds__(kSelThreads) void select_kernel(
    const float* __restrict__ mass_all, const float* __restrict__ rank_all, int n, double tau,
    int32_t* __restrict__ idx_all, int32_t* __restrict__ k_out, int32_t* __restrict__ status)
{
    __shared__ SelShared sh;
    extern __shared__ uint32_t lds_keys[];             // kSelMaxLdsKeys entries
    const int u = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* mass = mass_all + (int64_t)u * n;
    const float* rank = rank_all ? rank_all + (int64_t)u * n : mass;
    int32_t* idx = idx_all + (int64_t)u * n;
    if (status) {
        const uint32_t f = input_flags<kSelThreads>(mass, rank, n, &sh.base_sum, &sh.sel_cnt);
        if (tid == 0) status[u] = (int32_t)f;
        __syncthreads();
    }

    if (tau >= 1.0) {
        if (tid == 0) k_out[u] = n;
        for (int j = tid; j < n; j += kSelThreads) idx[j] = j;
        return;
    }

    // ---- how many (Eq. (7)) ----
    Keys mk{mass, n};
    int k;
    {
        uint32_t prefix, base_cnt;
        unsigned long long base_sum;
        bool degenerate;
        radix_descent<true>(mk, tau, 0u, sh, prefix, base_cnt, base_sum, degenerate);
        if (tid == 0) {
            int kk = 1;
            if (!degenerate) {
                const unsigned long long qv = fixed40_of_key(prefix);
                const unsigned long long need = sh.target - base_sum;           // >= 1
                kk = (int)(base_cnt + (qv ? (need + qv - 1) / qv : 1ull));
            }
            sh.k = max(1, min(kk, n));
        }
        __syncthreads();
        k = sh.k;
    }
    if (tid == 0) k_out[u] = k;
    if (k >= n) {
        for (int j = tid; j < n; j += kSelThreads) idx[j] = j;
        return;
    }
    __syncthreads();

    // ---- which (Eq. (9)): k-th largest normalised score v*, ties to the lower index ----
    Keys rk{rank, n};
    uint32_t vstar, cnt_gt;
    {
        unsigned long long unused;
        bool dg;
        radix_descent<false>(rk, tau, (uint32_t)k, sh, vstar, cnt_gt, unused, dg);
    }
    const uint32_t need_eq = (uint32_t)k - cnt_gt;     // ties at v* that are kept (>= 1)

    // ---- ascending emission, one block of positions (as many as LDS holds) at a time ----
    uint32_t gt_run = 0, eq_run = 0;                   // elements above / at v* in the blocks before
    for (int b0 = 0; b0 < n; b0 += kSelMaxLdsKeys) {
        const int bn = min(kSelMaxLdsKeys, n - b0);
        __syncthreads();
        fill_keys(lds_keys, rank + b0, bn);
        __syncthreads();
        // thread t classifies positions [32 t, 32 t + 32) of the block; the rotation by the lane
        // spreads the 64 reads of a wave over the banks
        const int base = tid * 32;
        uint32_t gm = 0, em = 0;
        if (base < bn) {
            // all 32 reads are issued at once (index clamped, the mask bit predicated instead)
            uint32_t key[32];
#pragma unroll
            for (int cc = 0; cc < 32; ++cc) key[cc] = lds_keys[min(base + ((cc + lane) & 31), bn - 1)];
#pragma unroll
            for (int cc = 0; cc < 32; ++cc) {
                const int p = (cc + lane) & 31;
                const bool in = base + p < bn;
                gm |= (in && key[cc] > vstar ? 1u : 0u) << p;
                em |= (in && key[cc] == vstar ? 1u : 0u) << p;
            }
        }
        const uint32_t cg = __popc(gm), ce = __popc(em);
        const uint32_t both = wave_scan(cg | ce << 16);    // at most 64 * 32 each
        const uint32_t ig = both & 0xFFFFu, ie = both >> 16;
        if (lane == 63) { sh.wave_cnt[wave] = ig; sh.wave_eq[wave] = ie; }
        __syncthreads();
        uint32_t gt_before = gt_run + (ig - cg), eq_before = eq_run + (ie - ce), tot_g = 0, tot_e = 0;
#pragma unroll
        for (int w2 = 0; w2 < kSelWaves; ++w2) {
            const uint32_t wg = sh.wave_cnt[w2], we = sh.wave_eq[w2];
            if (w2 < wave) { gt_before += wg; eq_before += we; }
            tot_g += wg; tot_e += we;
        }
        // of this thread's ties, the lowest-indexed `allow` are kept
        const uint32_t allow = need_eq > eq_before ? need_eq - eq_before : 0u;
        uint32_t ek = em;
        if (allow < ce) {
            ek = 0;
            uint32_t rest = em;
            for (uint32_t a2 = 0; a2 < allow; ++a2) {
                const uint32_t low = rest & (0u - rest);
                ek |= low;
                rest ^= low;
            }
        }
        uint32_t km = gm | ek;
        uint32_t out = gt_before + min(eq_before, need_eq);
        while (km) {
            const int p = __builtin_ctz(km);
            km &= km - 1;
            idx[out++] = b0 + base + p;
        }
        gt_run += tot_g;
        eq_run += tot_e;
    }
}

// ---------------------------------------------------------------- one kernel, keys in registers (n <= 32768)
// One workgroup per unit; thread t holds the keys of positions t, t + 1024, ... of both vectors in registers, requested
// at once at the start.  What bounds the kernel is a chain of short phases on one CU, so it has as few as possible:
//  * the first digit is four bits of mantissa under the exponent, over the 32 octaves where scores lie (anything outside
//    falls into the end bins): the crossing bin then holds some 1 % of the elements, where an exponent byte leaves a
//    quarter.  Both vectors' histograms are built in one sweep (the rank one does not need k);
//  * the elements of the crossing bin (ballots and one LDS add per wave) make a list that one wave descends, 7 bits at a
//    time, without a workgroup barrier; a bin too full for the list is narrowed by further sweeps of all waves first;
//  * a ballot per 64 positions is the emission's count and its order.
// One call, two vectors, tau = 0.975 (us; in brackets a sweep, a fold and a scan per 8-bit digit over keys in LDS, 32
// consecutive positions per thread in the emission): 4 units x 576 5.9 (12.5), 32 x 2933 7.6 (15.5), 128 x 8192 10.6 (19.5),
// 4 x 18432 16.8 (30.5), 4 x 32768 26.3 (57.1; from memory).  From there on two vectors do not fit the registers: the
// largest form already moves 18 of them to scratch.  With the exponent byte and three bits: 128 x 8192 11.8, 4 x 18432 20.0.
constexpr uint32_t kNoKey = 0xFFFFFFFFu;                 // of positions past n: in no span, below every key as a signed number
constexpr int kRegKeys = 32;                             // keys per thread at most: two vectors fit 128 registers
constexpr int kRegBins = 512, kRegRep = 8, kRegStride = kRegBins + 1;   // first digit; its histogram's replicas, chosen by the lane
constexpr int kRegCand = 1024;                           // elements of the crossing bin that one wave descends
constexpr int kMassOctave = 96, kRankOctave = 103;       // biased exponents of the lowest of 32 octaves: 2^-31 and 2^-24
constexpr int kRegShift = 19;                            // sixteen bins per octave

struct RegShared {
    unsigned long long hm[kRegRep * kRegStride];         // packed (count, integer sum) slots of mass; replica r of bin b at r * kRegStride + b
    uint32_t hr[kRegRep * kRegStride];                   // counts of rank
    unsigned long long fm[kRegBins];                     // both, folded over the replicas
    uint32_t fr[kRegBins];
    uint32_t list[kRegCand];
    unsigned long long lhist[128];                       // one digit of the list descent
    uint32_t chunk[kRegKeys * kSelWaves];                // kept elements per 64 positions
    unsigned long long target, base_sum;
    uint32_t base_cnt, lo, hi, in_bin, listed;
    int k;
    uint32_t vstar, need_eq;
};

// Where the search stands: the crossing key lies in [lo, hi), base_cnt elements with base_sum lie at hi and above, in_bin in
// between.
struct Span { uint32_t lo, hi, base_cnt, in_bin; unsigned long long base_sum; };

__device__ __forceinline__ uint32_t from_lane(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lane); }
__device__ __forceinline__ unsigned long long from_lane(unsigned long long v, int lane) {
    return ((unsigned long long)from_lane((uint32_t)(v >> 32), lane) << 32) | from_lane((uint32_t)v, lane);
}

// One wave finds the bin where the descending cumulative sum (WITH_SUM) or count crosses: lane l owns the PER bins
// from 64 PER - 1 - PER l downwards.  first: the target is ceil(tau * sum of all bins).  Returns the bin (0 if none crosses,
// which needs a mass that sums to 2 or more) and advances base_cnt, base_sum, in_bin.
template <bool WITH_SUM, int PER, typename U>
__device__ __forceinline__ uint32_t cross_bins(const U* bins, bool first, double tau, unsigned long long& target, Span& s) {
    const int lane = threadIdx.x & 63;
    // counts and sums are scanned together, packed as the slots are (plain counts: as they are)
    U v[PER], lv = 0;
#pragma unroll
    for (int t = 0; t < PER; ++t) { v[t] = bins[64 * PER - 1 - (PER * lane + t)]; lv += v[t]; }
    const U iv = wave_scan(lv);
    auto cnt = [](U x) { return WITH_SUM ? (uint32_t)((unsigned long long)x >> kSumBits) : (uint32_t)x; };
    auto sum = [](U x) { return WITH_SUM ? (unsigned long long)x & ((1ull << kSumBits) - 1ull) : (unsigned long long)x; };
    // ceil(tau * W): one IEEE double multiply, then ceil (W < 2^53)
    if (WITH_SUM && first) target = (unsigned long long)ceil(tau * (double)sum(from_lane(iv, 63)));
    const unsigned long long want = target - (WITH_SUM ? s.base_sum : (unsigned long long)s.base_cnt);      // >= 1
    U run = iv - lv, above = 0;
    uint32_t bin = 0, at_in = 0;
    bool mine = false;
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const U next = run + v[t];
        if (sum(run) < want && want <= sum(next)) { mine = true; bin = 64 * PER - 1 - (PER * lane + t); above = run; at_in = cnt(v[t]); }
        run = next;
    }
    const unsigned long long who = __ballot(mine);
    const int src = who ? __builtin_ctzll(who) : 0;
    above = from_lane(above, src);
    s.base_cnt += cnt(above);
    if (WITH_SUM) s.base_sum += sum(above);
    s.in_bin = from_lane(at_in, src);
    return who ? from_lane(bin, src) : 0u;
}

// Set bits of a ballot below this lane.
__device__ __forceinline__ uint32_t lanes_before(unsigned long long who) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
}

// fixed40 of a key below 2^12 in eight instructions: 20 bits above the binary point of x * 2^20 and 20 below, both exact.
__device__ __forceinline__ unsigned long long fixed40_split(uint32_t key) {
    const float x = __uint_as_float(key < 0x7F800000u ? key : 0u) * 0x1p20f;
    const uint32_t hi = (uint32_t)x, lo = (uint32_t)((x - (float)hi) * 0x1p20f);
    return (unsigned long long)(hi >> 12) << 32 | (hi << 20 | lo);
}

// First digit: sixteen bins per octave above `octave`, the end bins open.
__device__ __forceinline__ uint32_t first_digit(uint32_t key, int octave) {
    return (uint32_t)min(max((int)(key >> kRegShift) - (octave << 4), 0), kRegBins - 1);
}
__device__ __forceinline__ void first_span(uint32_t bin, int octave, Span& s) {
    s.lo = bin ? ((uint32_t)octave * 16u + bin) << kRegShift : 0u;
    s.hi = bin == kRegBins - 1u ? 0x80000000u : ((uint32_t)octave * 16u + bin + 1u) << kRegShift;
}
// Shift that cuts [lo, hi) into at most 2^bits pieces, and the piece `bin`.
__device__ __forceinline__ int span_shift(const Span& s, int bits) { return max(0, 32 - __builtin_clz(s.hi - s.lo - 1u | 1u) - bits); }
__device__ __forceinline__ void narrow(uint32_t bin, int shift, Span& s) {
    s.lo += bin << shift;
    s.hi = min(s.hi, s.lo + (1u << shift));
}

// One wave, the `c` listed keys of [s.lo, s.hi): down to the key at which the sum / count crosses (returned; s then holds what
// lies above it).
template <bool WITH_SUM>
__device__ __forceinline__ uint32_t descend_list(RegShared& sh, int c, unsigned long long target, Span& s) {
    const int lane = threadIdx.x & 63;
    while (s.hi - s.lo > 1u) {
        if (s.in_bin == 1u) {                                // the only element of the span is the key
            for (int j = lane; __any(j < c); j += 64) {
                const uint32_t key = j < c ? sh.list[j] : 0u;
                const unsigned long long who = __ballot(j < c && key >= s.lo && key < s.hi);
                if (who) return from_lane(key, __builtin_ctzll(who));
            }
        }
        const int shift = span_shift(s, 7);
        sh.lhist[lane] = 0ull;
        sh.lhist[lane + 64] = 0ull;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int j = lane; j < c; j += 64) {
            const uint32_t key = sh.list[j];
            if (key >= s.lo && key < s.hi)
                atomicAdd(&sh.lhist[(key - s.lo) >> shift], WITH_SUM ? (1ull << kSumBits) + fixed40_of_key(key) : 1ull);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        narrow(cross_bins<WITH_SUM, 2>(sh.lhist, false, 0.0, target, s), shift, s);
    }
    return s.lo;
}

template <int KPT>
__global__ __launch_bounds__(kSelThreads, KPT <= 4 ? 8 : 4) void select_reg_kernel(      // two workgroups per CU while 64 registers do
    const float* __restrict__ mass_all, const float* __restrict__ rank_all, int n, double tau,
    int32_t* __restrict__ idx_all, int32_t* __restrict__ k_out, int32_t* __restrict__ status)
{
    __shared__ RegShared sh;
    const int u = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* mass = mass_all + (int64_t)u * n;
    const float* rank = rank_all ? rank_all + (int64_t)u * n : mass;
    int32_t* idx = idx_all + (int64_t)u * n;
    if (status) {
        const uint32_t f = input_flags<kSelThreads>(mass, rank, n, &sh.base_sum, &sh.in_bin);
        if (tid == 0) status[u] = (int32_t)f;
        __syncthreads();
    }
    if (tau >= 1.0) {
        if (tid == 0) k_out[u] = n;
        for (int j = tid; j < n; j += kSelThreads) idx[j] = j;
        return;
    }
    uint32_t km[KPT], kr[KPT];
#pragma unroll
    for (int q = 0; q < KPT; ++q) km[q] = __float_as_uint(mass[min(tid + q * kSelThreads, n - 1)]);
#pragma unroll
    for (int q = 0; q < KPT; ++q) kr[q] = __float_as_uint(rank[min(tid + q * kSelThreads, n - 1)]);
    for (int i = tid; i < kRegRep * kRegStride; i += kSelThreads) { sh.hm[i] = 0ull; sh.hr[i] = 0u; }
    if (tid == 0) sh.listed = 0u;
    __syncthreads();
    const int rep = (tid & (kRegRep - 1)) * kRegStride;
    // f(q) for every key of this thread.  The fences keep the compiler from working on all keys at once (and from holding on
    // to every key's digit or sum for a later sweep), for which there are no registers.
    auto each_key = [&](uint32_t (&key)[KPT], auto&& f) {
#pragma unroll
        for (int q = 0; q < KPT; ++q) {
            asm volatile("" : "+v"(key[q]));
            f(q);
            if (q % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    };
    each_key(km, [&](int q) {
        km[q] = tid + q * kSelThreads < n ? (uint32_t)max((int)km[q], 0) : kNoKey;  // sign bit set: ordered and summed as zero
        if (km[q] != kNoKey) atomicAdd(&sh.hm[rep + first_digit(km[q], kMassOctave)], (1ull << kSumBits) + fixed40_split(km[q]));
    });
    each_key(kr, [&](int q) {
        kr[q] = tid + q * kSelThreads < n ? (uint32_t)max((int)kr[q], 0) : kNoKey;
        if (kr[q] != kNoKey) atomicAdd(&sh.hr[rep + first_digit(kr[q], kRankOctave)], 1u);
    });
    __syncthreads();
    auto fold_mass = [&](int b) {
        unsigned long long v = 0;
#pragma unroll
        for (int r = 0; r < kRegRep; ++r) v += sh.hm[r * kRegStride + b];      // count and sum fields add without carry between them
        sh.fm[b] = v;
    };
    auto fold_rank = [&](int b) {
        uint32_t v = 0;
#pragma unroll
        for (int r = 0; r < kRegRep; ++r) v += sh.hr[r * kRegStride + b];
        sh.fr[b] = v;
    };
    if (tid < kRegBins) fold_mass(tid);
    else fold_rank(tid - kRegBins);
    __syncthreads();

    auto put = [&](const Span& s) {                          // one wave -> all
        if (lane == 0) { sh.lo = s.lo; sh.hi = s.hi; sh.base_cnt = s.base_cnt; sh.in_bin = s.in_bin; sh.base_sum = s.base_sum; }
    };
    auto get = [&]() { return Span{sh.lo, sh.hi, sh.base_cnt, sh.in_bin, sh.base_sum}; };
    // From the published span: more sweeps while it is too full, then the list of its keys.  Every thread takes part.
    auto collect = [&](uint32_t (&key)[KPT], auto with_sum) {
        constexpr bool WITH_SUM = decltype(with_sum)::value;
        Span s = get();
        // A bin that holds a sixteenth of the vector or more (and more than 256 keys) holds close or equal scores: one wave would
        // add 64 of them to one counter after the other, all waves do better although a list would take them.  Two vectors of
        // 1000 scores, 4 units: all equal 22.0 us -> 11.6, within 1e-3 18.0 -> 9.0; 2933 of three values 22.8 -> 13.2.
        const uint32_t most = (uint32_t)min(kRegCand, max(256, n >> 4));
        while (s.in_bin > most && s.hi - s.lo > 1u) {
            const int shift = span_shift(s, 9);
            for (int i = tid; i < kRegRep * kRegStride; i += kSelThreads) { if (WITH_SUM) sh.hm[i] = 0ull; else sh.hr[i] = 0u; }
            __syncthreads();
            each_key(key, [&](int q) {
                if (key[q] - s.lo < s.hi - s.lo) {
                    const int slot = rep + (int)((key[q] - s.lo) >> shift);
                    if (WITH_SUM) atomicAdd(&sh.hm[slot], (1ull << kSumBits) + fixed40_split(key[q]));
                    else atomicAdd(&sh.hr[slot], 1u);
                }
            });
            __syncthreads();
            if (tid < kRegBins) { if (WITH_SUM) fold_mass(tid); else fold_rank(tid); }
            __syncthreads();
            if (wave == 0) {
                unsigned long long target = WITH_SUM ? sh.target : (unsigned long long)(uint32_t)sh.k;
                uint32_t bin;
                if constexpr (WITH_SUM) bin = cross_bins<true, kRegBins / 64>(sh.fm, false, 0.0, target, s);
                else bin = cross_bins<false, kRegBins / 64>(sh.fr, false, 0.0, target, s);
                narrow(bin, shift, s);
                put(s);
            }
            __syncthreads();
            s = get();
        }
        if (s.hi - s.lo > 1u) {
            uint32_t cnt = 0;
            unsigned long long who[KPT];
            each_key(key, [&](int q) {
                who[q] = __ballot(key[q] - s.lo < s.hi - s.lo);
                cnt += __popcll(who[q]);
            });
            if (cnt) {
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&sh.listed, cnt);
                at = from_lane(at, 0);
                each_key(key, [&](int q) {
                    if (who[q]) {
                        const uint32_t pos = at + lanes_before(who[q]);
                        if (__builtin_amdgcn_inverse_ballot_w64(who[q]) && pos < (uint32_t)kRegCand) sh.list[pos] = key[q];
                        at += __popcll(who[q]);
                    }
                });
            }
        }
        __syncthreads();
    };

    // ---- how many (Eq. (7)) ----
    if (wave == 0) {
        Span s{0u, 1u, 0u, 0u, 0ull};
        unsigned long long target = 0;
        const uint32_t bin = cross_bins<true, kRegBins / 64>(sh.fm, true, tau, target, s);
        if (target) first_span(bin, kMassOctave, s);         // all scores zero otherwise
        if (lane == 0) sh.target = target;
        put(s);
    }
    __syncthreads();
    collect(km, std::true_type{});
    if (wave == 0) {
        Span s = get();
        const unsigned long long target = sh.target;
        int k = 1;
        if (target) {
            const uint32_t key = descend_list<true>(sh, (int)min(sh.listed, (uint32_t)kRegCand), target, s);
            const unsigned long long qv = fixed40_of_key(key), need = target - s.base_sum;      // >= 1
            k = (int)(s.base_cnt + (need > qv && qv ? (need + qv - 1) / qv : 1ull));           // the division is for ties
        }
        k = max(1, min(k, n));
        Span r{0u, 0u, 0u, 0u, 0ull};
        unsigned long long want = (unsigned long long)k;
        if (k < n) first_span(cross_bins<false, kRegBins / 64>(sh.fr, false, 0.0, want, r), kRankOctave, r);
        put(r);
        if (lane == 0) { sh.k = k; k_out[u] = k; sh.listed = 0u; }
    }
    __syncthreads();
    const int k = sh.k;
    if (k >= n) {
        for (int j = tid; j < n; j += kSelThreads) idx[j] = j;
        return;
    }
    // ---- which (Eq. (9)): k-th largest normalised score v*, ties to the lower index ----
    collect(kr, std::false_type{});
    if (wave == 0) {
        Span s = get();
        const uint32_t vs = descend_list<false>(sh, (int)min(sh.listed, (uint32_t)kRegCand), (unsigned long long)k, s);
        if (lane == 0) { sh.vstar = vs; sh.need_eq = (uint32_t)k - s.base_cnt; }                // ties at v* that are kept (>= 1)
    }
    __syncthreads();
    // ---- ascending emission: 64 positions per ballot ----
    const uint32_t vstar = sh.vstar, need_eq = sh.need_eq;
    unsigned long long gt[KPT], eq[KPT];
    uint32_t mine = 0;                                       // lane q: elements above v* and at v* of chunk q of this wave (n <= 32768 in all)
    each_key(kr, [&](int q) {
        gt[q] = __ballot((int)kr[q] > (int)vstar);
        eq[q] = __ballot(kr[q] == vstar);
        if (lane == q) mine = (uint32_t)__popcll(gt[q]) | (uint32_t)__popcll(eq[q]) << 16;
    });
    if (lane < KPT) sh.chunk[lane * kSelWaves + wave] = mine;
    __syncthreads();
    if (wave == 0) {                                         // exclusive prefix over the chunks
        constexpr int PER = (KPT * kSelWaves + 63) / 64;
        uint32_t v[PER], sum = 0;
#pragma unroll
        for (int t = 0; t < PER; ++t) { v[t] = lane * PER + t < KPT * kSelWaves ? sh.chunk[lane * PER + t] : 0u; sum += v[t]; }
        uint32_t run = wave_scan(sum) - sum;
#pragma unroll
        for (int t = 0; t < PER; ++t) {
            if (lane * PER + t < KPT * kSelWaves) sh.chunk[lane * PER + t] = run;
            run += v[t];
        }
    }
    __syncthreads();
    if (lane < KPT) mine = sh.chunk[lane * kSelWaves + wave];
    each_key(kr, [&](int q) {
        const uint32_t before = from_lane(mine, q), eq_before = before >> 16;
        unsigned long long keep = gt[q];
        if (eq[q]) keep |= __ballot(kr[q] == vstar && eq_before + lanes_before(eq[q]) < need_eq);
        if (__builtin_amdgcn_inverse_ballot_w64(keep))
            idx[(before & 0xFFFFu) + min(eq_before, need_eq) + lanes_before(keep)] = tid + q * kSelThreads;
    });
}

template <int KPT>
static void launch_select_reg(const float* mass, const float* rank, int units, int n, double tau, int32_t* idx, int32_t* k,
                              int32_t* status, hipStream_t st) {
    hipLaunchKernelGGL((select_reg_kernel<KPT>), dim3(units), dim3(kSelThreads), 0, st, mass, rank, n, tau, idx, k, status);
}

// ---------------------------------------------------------------- two kernels: parallel first digit, then one workgroup per unit
// First-digit histograms of a slice of positions, built in LDS and added to the unit's tables.
__global__ __launch_bounds__(256) void select_hist_kernel(
    const float* __restrict__ mass_all, const float* __restrict__ rank_all, int n, int slice,
    unsigned long long* __restrict__ hm_all, uint32_t* __restrict__ hr_all)
{
    __shared__ unsigned long long lm[kSelBins];
    __shared__ uint32_t lr[kSelBins];
    const int u = blockIdx.y, tid = threadIdx.x;
    const int j0 = blockIdx.x * slice, j1 = min(n, j0 + slice);
    if (j0 >= j1) return;
    for (int b = tid; b < kSelBins; b += 256) { lm[b] = 0ull; lr[b] = 0u; }
    __syncthreads();
    const float* mass = mass_all + (int64_t)u * n;
    const float* rank = rank_all ? rank_all + (int64_t)u * n : nullptr;
    for (int j = j0 + tid; j < j1; j += 256) {
        const uint32_t key = orderable(mass[j]);
        atomicAdd(&lm[key >> kSelBinShift], (1ull << kSumBits) + fixed40_of_key(key));
        if (rank) atomicAdd(&lr[orderable(rank[j]) >> kSelBinShift], 1u);
    }
    __syncthreads();
    flush_tables<256>(lm, lr, hm_all + (int64_t)u * kSelBins, rank ? hr_all + (int64_t)u * kSelBins : nullptr);
}

// The rest of the selection of one unit; leaves the unit's tables zero for the next call.
__global__ __launch_bounds__(kSelThreads) void select_tail_kernel(
    const float* __restrict__ mass_all, const float* __restrict__ rank_all, int n, double tau,
    unsigned long long* __restrict__ hm_all, uint32_t* __restrict__ hr_all,
    int32_t* __restrict__ idx_all, int32_t* __restrict__ k_out, int key_cap, int32_t* __restrict__ status)
{
    __shared__ TailShared sh;
    extern __shared__ uint32_t lds_keys[];
    const int u = blockIdx.x;
    const float* mass = mass_all + (int64_t)u * n;
    if (status) {
        const uint32_t f = input_flags<kSelThreads>(mass, rank_all ? rank_all + (int64_t)u * n : mass, n, &sh.base_sum, &sh.sel_cnt);
        if (threadIdx.x == 0) status[u] = (int32_t)f;
        __syncthreads();
    }
    unsigned long long* hm = hm_all + (int64_t)u * kSelBins;
    uint32_t* hr = hr_all + (int64_t)u * kSelBins;
    select_tail<kSelThreads>(mass, rank_all ? rank_all + (int64_t)u * n : mass, n, tau, hm, rank_all ? hr : nullptr,
                                    idx_all + (int64_t)u * n, k_out + u, lds_keys, key_cap, sh);
    __syncthreads();
    for (int b = threadIdx.x; b < kSelBins; b += kSelThreads) { hm[b] = 0ull; hr[b] = 0u; }
}

size_t select_workspace_bytes(int units) {
    return (size_t)units * kSelBins * (sizeof(unsigned long long) + sizeof(uint32_t));
}

int launch_select(const float* mass, const float* rank, int units, int n, double tau,
                  int32_t* idx, int32_t* k, int32_t* status, void* ws, size_t ws_bytes, hipStream_t st)
{
    static std::atomic<bool> attr_done{false};
    if (!attr_done) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&select_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kSelMaxLdsKeys * (int)sizeof(uint32_t)) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(&select_tail_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kSelMaxLdsKeys * (int)sizeof(uint32_t)) != hipSuccess)
            return set_error(ZIPVL_EHIP, "select: cannot reserve LDS for the keys");
        attr_done = true;
    }
    if (n <= kRegKeys * kSelThreads) {
        KernelTimer tm(ZIPVL_K_SELECT, st);
        const int kpt = (n + kSelThreads - 1) / kSelThreads;
#define ZIPVL_SEL(KPT) launch_select_reg<KPT>(mass, rank, units, n, tau, idx, k, status, st)
        if (kpt <= 1) ZIPVL_SEL(1);
        else if (kpt <= 2) ZIPVL_SEL(2);
        else if (kpt <= 3) ZIPVL_SEL(3);
        else if (kpt <= 4) ZIPVL_SEL(4);
        else if (kpt <= 6) ZIPVL_SEL(6);
        else if (kpt <= 8) ZIPVL_SEL(8);
        else if (kpt <= 12) ZIPVL_SEL(12);
        else if (kpt <= 16) ZIPVL_SEL(16);
        else if (kpt <= 20) ZIPVL_SEL(20);
        else if (kpt <= 24) ZIPVL_SEL(24);
        else if (kpt <= 28) ZIPVL_SEL(28);
        else ZIPVL_SEL(32);
#undef ZIPVL_SEL
        return check_launch("select");
    }
    if (ws && ws_bytes >= select_workspace_bytes(units) && tau < 1.0) {
        // two kernels: the first digit of both descents from every CU, then one workgroup per unit
        unsigned long long* hm = (unsigned long long*)ws;
        uint32_t* hr = (uint32_t*)(hm + (size_t)units * kSelBins);
        const int slices = std::max(1, std::min((n + 255) / 256, (512 + units - 1) / units));
        const int slice = ((n + slices - 1) / slices + 63) / 64 * 64;
        {
            KernelTimer tm(ZIPVL_K_SELECT_HIST, st);
            hipLaunchKernelGGL(select_hist_kernel, dim3((n + slice - 1) / slice, units), dim3(256), 0, st, mass, rank, n, slice, hm, hr);
        }
        int rc = check_launch("select_hist");
        if (rc) return rc;
        const int key_cap = kSelMaxLdsKeys;
        KernelTimer tm(ZIPVL_K_SELECT, st);
        hipLaunchKernelGGL(select_tail_kernel, dim3(units), dim3(kSelThreads), (size_t)key_cap * sizeof(uint32_t), st,
                           mass, rank, n, tau, hm, hr, idx, k, key_cap, status);
        return check_launch("select_tail");
    }
    const size_t dyn = (size_t)kSelMaxLdsKeys * sizeof(uint32_t);          // stages the blocks of the emission
    KernelTimer tm(ZIPVL_K_SELECT, st);
    hipLaunchKernelGGL(select_kernel, dim3(units), dim3(kSelThreads), dyn, st, mass, rank, n, tau, idx, k, status);
    return check_launch("select");
}

// ---------------------------------------------------------------- shared selection
// One important set per batch element: the per-unit scores are averaged over the Hkv units, units
// added in ascending order in fp32 and the sum multiplied by fp32(1/Hkv), so that the result is a
// fixed function of the inputs (the selection that follows is decided by these bits).
__global__ __launch_bounds__(256) void share_scores_kernel(
    const float* __restrict__ mass, const float* __restrict__ rank, int Hkv, int n, float inv,
    float* __restrict__ mass_b, float* __restrict__ rank_b)
{
    const int b = blockIdx.y;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const float* mp = mass + (int64_t)b * Hkv * n + j;
    float a = mp[0];
    for (int g = 1; g < Hkv; ++g) a += mp[(int64_t)g * n];
    mass_b[(int64_t)b * n + j] = a * inv;
    if (rank) {
        const float* rp = rank + (int64_t)b * Hkv * n + j;
        float r = rp[0];
        for (int g = 1; g < Hkv; ++g) r += rp[(int64_t)g * n];
        rank_b[(int64_t)b * n + j] = r * inv;
    }
}

int launch_share_scores(const float* mass, const float* rank, int B, int Hkv, int n,
                        float* mass_b, float* rank_b, hipStream_t st)
{
    KernelTimer tm(ZIPVL_K_SHARE_SCORES, st);
    hipLaunchKernelGGL(share_scores_kernel, dim3((n + 255) / 256, B), dim3(256), 0, st,
        mass, rank, Hkv, n, (float)(1.0 / Hkv), mass_b, rank_b);
    return check_launch("share_scores");
}

}  // namespace zipvl
