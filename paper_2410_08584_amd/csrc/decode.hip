// Decode-phase attention against the (evicted) KV cache (Eq. (5); Algorithm 2).
// Memory-bound: one query per head, every cached row read exactly once, all
// query heads of a KV group served from the same read.
// Split-KV: a unit's device-resident length is cut into equal splits, as many as fill
// the chip when all units are alike (from the units, on the host) and more where the
// unit is long (from its length; SplitRule), so that short and full caches as well as
// batches of unequal lengths keep the workgroups busy.
// Groups of two and more heads run on the matrix cores, 16 cached rows per wave
// step (attend_split); a single head runs on the vector units over rows as stored,
// where 16 lanes cover one cached row (16 bytes each at d = 128 bf16), reduce the dot
// product with shuffles and keep an online-softmax state per row group (attend_rows),
// and in integer matrix products over codes (decode_q1_partial_kernel).  Waves and
// finally splits are merged with the usual (max, sum, weighted output) rule.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "launch.h"
#include "rowops.h"

namespace zipvl {

constexpr int kDecMaxSplit = 64;

template <typename T> __device__ __forceinline__ T to_out(float x);
template <> __device__ __forceinline__ float to_out<float>(float x) { return x; }
template <> __device__ __forceinline__ __bf16 to_out<__bf16>(float x) { return (__bf16)x; }

// One cached row against a query: kf / vf are this lane's EPL elements of the row.
template <int EPL>
__device__ __forceinline__ void attend_row(bool valid, const float (&kf)[EPL], const float (&vf)[EPL],
                                           const float (&qv)[EPL], float& m, float& l, float (&o)[EPL]) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) s += qv[e] * kf[e];
    s += __shfl_xor(s, 1); s += __shfl_xor(s, 2); s += __shfl_xor(s, 4); s += __shfl_xor(s, 8);
    if (valid) {
        const float m_new = fmaxf(m, s);
        const float a = fast_exp2(m - m_new), p = fast_exp2(s - m_new);
        l = l * a + p;
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[e] = o[e] * a + p * vf[e];
        m = m_new;
    }
}

// The partial states (o[D], m, l; log2 domain) of a launch: the outputs of all (unit, head, split) first, each D floats
// on a 16-byte boundary, then their (m, l) pairs.
struct PartialOut {
    float* o; float* ml; int nsplit;                         // rows of one unit: head * nsplit + split
    __device__ __forceinline__ PartialOut(float* part, int D, int u, int G, int nsplit_, int units) : nsplit(nsplit_) {
        o = part + (int64_t)u * G * nsplit * D;
        ml = part + (int64_t)units * G * nsplit * D + (int64_t)u * G * nsplit * 2;
    }
};

// A 16-byte load past the caches that are not coherent between XCDs (the states were written through by other
// workgroups of the same launch).
__device__ __forceinline__ floatx4 load16_coherent(const float* base, int byte_offset) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0x7FFFFFFF, 0x00020000);
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rs, byte_offset, 0, 16));   // sc1: device scope
}

// The waves' states in red[wave][head][o[D], m, l] -> the workgroup's partial state.
// COHERENT: the partial state is read by another workgroup of the same launch (possibly on another XCD,
// whose L2 is not coherent with this one's): written through with device-scope stores.
template <int D, int GT, int WAVES, bool COHERENT = false>
__device__ __forceinline__ void combine_waves(float (&red)[WAVES][GT][D + 2], int heads, const PartialOut& po, int gbase, int split) {
    auto put = [](float* p, float v) {
        if constexpr (COHERENT) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else *p = v;
    };
    for (int wi = threadIdx.x; wi < heads * D; wi += 64 * WAVES) {
        const int t = wi / D, dd = wi - t * D;
        float M = -INFINITY;
#pragma unroll
        for (int ww = 0; ww < WAVES; ++ww) M = fmaxf(M, red[ww][t][D]);
        float acc = 0.f, lsum = 0.f;
        if (M > -INFINITY) {
#pragma unroll
            for (int ww = 0; ww < WAVES; ++ww) {
                const float a = fast_exp2(red[ww][t][D] - M);
                acc += red[ww][t][dd] * a;
                lsum += red[ww][t][D + 1] * a;
            }
        }
        const int64_t row = (int64_t)(gbase + t) * po.nsplit + split;
        put(po.o + row * D + dd, acc);
        if (dd == 0) { put(po.ml + 2 * row, M); put(po.ml + 2 * row + 1, lsum); }
    }
}

// The partial states of one head's splits -> its output row, by a workgroup of THREADS threads: every wave turns the splits'
// (max, sum) pairs into weights a_s / sum_s(a_s l_s), a_s = exp2(m_s - max), one split per lane; every thread has four output
// elements of every kGroups-th split on the way meanwhile, and the partial sums of an element meet in LDS, added in a fixed order.
// nsplit <= 64.  COHERENT: the states were written by other workgroups of the same launch.
template <int D, int THREADS, bool COHERENT>
struct HeadStates {
    static constexpr int kCols = D / 4, kGroups = THREADS / kCols, N = 64 / kGroups;
    float m, l;                                              // of split `lane`
    floatx4 v[N];
    // the states of splits [from, nsplit), from a multiple of kGroups
    __device__ __forceinline__ void fetch_outputs(const PartialOut& po, int head, int from, int nsplit) {
        const int tid = threadIdx.x, sg = tid / kCols, col = tid - sg * kCols;
        const int off = head * po.nsplit * (D * 4) + col * 16;                        // the unit's base is wave-uniform
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (q * kGroups >= from && q * kGroups < nsplit) {                        // uniform over the workgroup
                const int at = off + min(sg + q * kGroups, nsplit - 1) * (D * 4);
                if constexpr (COHERENT) v[q] = load16_coherent(po.o, at);
                else v[q] = *reinterpret_cast<const floatx4*>(reinterpret_cast<const char*>(po.o) + at);
            }
    }
    __device__ __forceinline__ void fetch_sums(const PartialOut& po, int head, int nsplit) {
        const int lane = threadIdx.x & 63;
        const float* p = po.ml + ((int64_t)head * po.nsplit + min(lane, nsplit - 1)) * 2;
        if constexpr (COHERENT) {
            m = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            l = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else { m = p[0]; l = p[1]; }
        if (lane >= nsplit) { m = -INFINITY; l = 0.f; }
    }
    __device__ __forceinline__ float weight() const {        // of split `lane`
        const float M = wave_max(m);
        const float a = M > -INFINITY ? fast_exp2(m - M) : 0.f;
        const float tot = wave_sum(a * l);
        return tot > 0.f ? a / tot : 0.f;
    }
    template <typename T>
    __device__ __forceinline__ void finish(int nsplit, floatx4 (&sum)[THREADS], T* __restrict__ out) const {
        const int tid = threadIdx.x, sg = tid / kCols, col = tid - sg * kCols;
        const float w = weight();
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (q * kGroups < nsplit) {
                const float ws = __shfl(w, min(sg + q * kGroups, 63));
                if (sg + q * kGroups < nsplit) acc += ws * v[q];
            }
        sum[tid] = acc;
        __syncthreads();
        if (sg == 0) {
            for (int x = 1; x < min(kGroups, nsplit); ++x) acc += sum[x * kCols + col];
            T* dst = out + col * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[e] = to_out<T>(acc[e]);
        }
    }
};

// Merge the 4 row groups of every wave, then the 4 waves, and write the workgroup's partial state (one head).
template <int D, bool COHERENT>
__device__ __forceinline__ void write_partial(float m, float l, float (&o)[D / 16], float (&red)[4][1][D + 2], const PartialOut& po, int split) {
    constexpr int EPL = D / 16;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, sub = lane & 15, rg = lane >> 4;
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
        const float m2 = __shfl_xor(m, off), l2 = __shfl_xor(l, off);
        float o2[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) o2[e] = __shfl_xor(o[e], off);
        merge_state<EPL>(m, l, o, m2, l2, o2);
    }
    if (rg == 0) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) red[w][0][sub * EPL + e] = o[e];
        if (sub == 0) { red[w][0][D] = m; red[w][0][D + 1] = l; }
    }
    __syncthreads();
    combine_waves<D, 1, 4, COHERENT>(red, 1, po, 0, split);
}

// rows [r_begin, r_end) of a segment of L rows that split `split` of nsplit handles (multiples of 64 rows: 16 per wave step)
__device__ __forceinline__ void split_range64(int L, int split, int nsplit, int& r_begin, int& r_end) {
    int per = (L + nsplit - 1) / nsplit;
    per = (per + 63) & ~63;
    r_begin = split * per;
    r_end = min(L, r_begin + per);
}

// ---------------------------------------------------------------- attention over a cache as stored
// One wave works on tiles of 16 cached rows with the matrix cores, all query heads of the group in the 16 columns:
//   S = K q^T     A = 16 cached rows, B = the queries: a bf16 row feeds v_mfma_f32_16x16x32_bf16, an fp32 row
//                 v_mfma_f32_16x16x4_f32 (products exact or fp32, sums fp32); lane (j, kk) receives the scores of
//                 head j for rows 4 kk .. 4 kk + 3.
//   O^T += V^T P  with v_mfma_f32_16x16x4_f32: step r contracts rows {4 kk + r}, so the score registers are the B
//                 operand as they are, and the A operand of output block e is element e of the lane's piece of row
//                 4 kk + r - a 16-byte load of the row, widened to fp32.  No value crosses lanes, P stays fp32.
//                 bf16 rows: v_mfma_f32_16x16x16_bf16, the weights as three bf16 planes whose sum they are exactly, so that the
//                 products and all 24 bits of the weights are kept; 384 matrix cycles a tile and not 1024, and no widening.  An
//                 infinity in V meets planes of 0: a wave whose sums are no numbers takes its tiles again in fp32 products.
//                 us a layer: 28 heads on 4, 7200 rows 12.4 -> 11.5; 8 x 28 on 4, 1750 rows 13.4 -> 12.1; 4 x 32 on 8, 900 rows
//                 10.4 -> 9.4; 8 x 32 on 8, 6000 rows 41 -> 39; 28 on 4, 33 000 rows 20.7 -> 19.4.
// The offset of the exponentials follows the running maximum of a head lazily (moves when it is exceeded by
// 2^kDecLazyLog2), so the accumulators are rescaled on few tiles.
constexpr float kDecLazyLog2 = 8.f;
// A group of one head keeps the vector units (attend_rows, 16 lanes per row): 15 of the 16 columns would be empty and
// the fp32 products of 16 rows cost 1024 matrix cycles whatever the columns hold.  One step at B = 4, 32 heads, 2050 rows:
// 33 us against 36 us on the matrix cores; B = 1, 28 heads on 4, 7200 rows: 86 us (16 lanes per row, seven heads in
// turn, 64 workgroups) against 14 us.
template <int GT> constexpr bool kDecMfma = GT > 1;
template <int GT> constexpr int kDecWaves = kDecMfma<GT> ? 8 : 4;        // waves per workgroup (8: 14.0 us, 4: 18.5 us at the shape above)
constexpr int kDecTile = 16;          // cached rows per wave step
// Tiles of a split that is called long (SplitRule).  Such a split takes about 85 us (one head, 3072 rows) and 100 us (groups,
// 6144 rows) on one workgroup; for shorter ones more workgroups mostly add launching and merging.
constexpr int kDecLongOne = 192, kDecLongGroups = 384;
// Splits of a group of heads that the step kernel merges itself.  us, one launch and two: 8 x 32 heads on 8, 4 splits 26.7, 28.0; 8 x 28
// on 4, 8 splits 13.6, 14.8; 4 x 28 on 4, 16 splits 19.3, 20.2; 28 on 4, 41 splits 14.4, 12.2; 14 on 2, 17 splits 11.6, 10.9.  With room for 32
// states in registers 14.0, 20.1 and 11.2.  bf16 at d = 64, half the bytes: 28 on 4, 17 splits 9.0, 10.5, 22 splits 9.4, 10.5 (two launches cost the
// host more than the GPU there), 47 splits 11.1, 9.7; fp32, 17 splits 11.2, 10.4.
template <typename T, int D> constexpr int kMergeSplits = D == 64 && sizeof(T) == 2 ? 24 : 16;

template <typename T, int EPL> struct alignas(sizeof(T) * EPL > 16 ? 16 : sizeof(T) * EPL) RawChunk { T v[EPL]; };

template <typename T, int D>
struct DecTile {
    static constexpr int NK = D * (int)sizeof(T) / 64;       // 16-byte pieces of a K row per lane (4 lanes cover 64 bytes)
    uintx4 k[NK];
    RawChunk<T, D / 16> v[4];
};

// a b^T of one 16-byte piece per lane: short chains, which the caller adds up pairwise.  One fp32 chain through all of
// d = 128 puts 3.5 times the rounding error into the output (1.3e-6 against 0.35e-6 relative; 28 heads on 4, 2400 rows).
__device__ __forceinline__ floatx4 mma16(const uintx4& a, const uintx4& b, __bf16) {
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), zero, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mma16(const uintx4& a, const uintx4& b, float) {
    const floatx4 fa = __builtin_bit_cast(floatx4, a), fb = __builtin_bit_cast(floatx4, b);
    floatx4 x = {0.f, 0.f, 0.f, 0.f}, y = x;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        x = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[e], fb[e], x, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[e + 2], fb[e + 2], y, 0, 0, 0);
    }
    return x + y;
}

template <typename T, int EPL>
__device__ __forceinline__ void raw_to_floats(const RawChunk<T, EPL>& r, float (&f)[EPL]) {
    RowChunk<T, EPL>::load(r.v, f);
}

// Rows [r_begin, r_end) of one unit against the query in qv.  Row r comes from the cache, except row
// `new_row` (>= 0 only in the fused step), which comes from k_new / v_new and is also written to the cache.
// The 16 row groups of the workgroup take rows r_begin + g, r_begin + g + 16, ...; the loads of a group's next
// row are in flight while the current one is consumed.
template <typename T, int D>
__device__ __forceinline__ void attend_rows(const T* Kb, const T* Vb, T* Kw, T* Vw, const T* kn, const T* vn, int new_row,
                                            int r_begin, int r_end, int group, const float (&qv)[D / 16], float& m, float& l, float (&o)[D / 16]) {
    constexpr int EPL = D / 16;
    using Raw = RawChunk<T, EPL>;
    auto fetch = [&](int r, Raw& kr, Raw& vr) {
        const int rr = r < r_end ? r : r_begin;             // clamped rows are loaded and ignored
        const bool fresh = rr == new_row;
        kr = *reinterpret_cast<const Raw*>(fresh ? kn : Kb + (int64_t)rr * D);
        vr = *reinterpret_cast<const Raw*>(fresh ? vn : Vb + (int64_t)rr * D);
    };
    if (r_begin >= r_end) return;
    Raw kc, vc;
    int r = r_begin + group;
    fetch(r, kc, vc);
    for (int base = r_begin; base < r_end; base += 16, r += 16) {   // workgroup-uniform trip count
        Raw kx = kc, vx = vc;
        if (base + 16 < r_end) fetch(r + 16, kx, vx);
        const bool valid = r < r_end;
        if (valid && r == new_row) {
            *reinterpret_cast<Raw*>(Kw + (int64_t)r * D) = kc;
            *reinterpret_cast<Raw*>(Vw + (int64_t)r * D) = vc;
        }
        float kf[EPL], vf[EPL];
        raw_to_floats<T, EPL>(kc, kf);
        raw_to_floats<T, EPL>(vc, vf);
        attend_row<EPL>(valid, kf, vf, qv, m, l, o);
        kc = kx; vc = vx;
    }
}

// Splits of a unit: `least`, which fill the chip together with the other units' when all are alike; `more` where those would
// be longer than `tiles`, and `most` where these would be (split_rule).  A unit goes by its own length: a long one among
// short ones is not left to few workgroups, and units that are all long make whole rounds of workgroups.  One conversation of
// 8192 rows among 31 of 200, 32 heads: 228 us with equal splits, 92 so; 8 KV heads of four heads: 132, 80; 32 conversations of
// 8192 rows as before (737 and 198).
// Workgroups are dealt to XCDs and CUs in turn.  Without idle ones the splits of a unit follow each other; where a short unit
// leaves some idle the units do, each row of units turned by `turn`, so that neither the busy workgroups of short units nor
// those of a long one fall on the same CUs (one conversation of 32768 rows among three of 500, 32 heads: 213 us without the
// turn, 145 with it, 16 splits either way).
// A unit of fewer than `from` tiles has `coarse` splits: finer ones would cost more than they give (finer_from).  Never where a KV head has several
// heads, and their kernels do not look at it (0.05 us of 7: 8 layers of 28 on 4, cap 1600 65.9 us with the look, 65.3 without).
struct SplitRule {
    int least, more, most, tiles, units, turn;               // turn 0: nothing is left idle
    int coarse, from;                                        // from 0: `least` splits for all
    dim3 grid() const { return turn ? dim3(units, most) : dim3(most, units); }
    __device__ __forceinline__ int split() const { return turn ? blockIdx.y : blockIdx.x; }
    __device__ __forceinline__ int unit() const { return turn ? (blockIdx.x + blockIdx.y * (unsigned)turn) % (unsigned)units : blockIdx.y; }
};
__device__ __forceinline__ int tiles_of(int L) { return (L + kDecTile - 1) / kDecTile; }
template <bool GROUPS>
__device__ __forceinline__ int tiles_per_split(int T, const SplitRule& rule) {
    const int s = !GROUPS && T < rule.from ? rule.coarse : T <= rule.least * rule.tiles ? rule.least : T <= rule.more * rule.tiles ? rule.more : rule.most;
    return max(1, (T + s - 1) / s);
}

// Rows [r_begin, r_end) of one unit against heads gbase .. gbase + GT - 1 of its group; the workgroup's state goes to
// `part`.  Kb / Vb: the unit's cache.  Row `new_row` (>= 0 only in the fused step) comes from kn / vn and is written
// to the cache.
template <typename T, int D, int GT, bool COHERENT>
__device__ __forceinline__ void attend_split(const T* q0, int heads, float c, T* Kb, T* Vb, const T* kn, const T* vn, int new_row,
                                             int r_begin, int r_end, float (&red)[kDecWaves<GT>][GT][D + 2],
                                             const PartialOut& po, int gbase, int split)
{
    constexpr int EPL = D / 16, NK = DecTile<T, D>::NK, E16 = 16 / (int)sizeof(T);
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 15, kk = lane >> 4;
    using Tile = DecTile<T, D>;
    using Raw = RawChunk<T, EPL>;
    auto fetch = [&](int t0, Tile& x) {
        const int rk = min(t0 + j, r_end - 1);               // rows past the end re-read the last one and weigh nothing
        const T* kp = (rk == new_row ? kn : Kb + (int64_t)rk * D) + kk * E16;
#pragma unroll
        for (int cc = 0; cc < NK; ++cc) x.k[cc] = load16(kp + cc * 4 * E16);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rv = min(t0 + 4 * kk + r, r_end - 1);
            x.v[r] = *reinterpret_cast<const Raw*>((rv == new_row ? vn : Vb + (int64_t)rv * D) + j * EPL);
        }
    };
    const int step = kDecWaves<GT> * kDecTile, first = r_begin + w * kDecTile;
    Tile cur;
    if (first < r_end) fetch(first, cur);
    uintx4 qf[NK];
#pragma unroll
    for (int cc = 0; cc < NK; ++cc) {
        qf[cc] = uintx4{0, 0, 0, 0};
        if (j < heads) qf[cc] = load16(q0 + (int64_t)j * D + kk * E16 + cc * 4 * E16);
    }
    float m, l;                                              // head j
    floatx4 o[EPL];                                          // o[e][r]: element EPL (4 kk + r) + e of head j
    auto pass = [&](auto planes_tag) {
    constexpr bool kPlanes = decltype(planes_tag)::value;
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[e] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int t0 = first; t0 < r_end; t0 += step) {
        Tile nxt;
        if (t0 + step < r_end) fetch(t0 + step, nxt);        // in flight while this tile is multiplied
        if (new_row >= t0 && new_row < t0 + kDecTile) {
            if (t0 + j == new_row) {
#pragma unroll
                for (int cc = 0; cc < NK; ++cc) store16(Kb + (int64_t)new_row * D + kk * E16 + cc * 4 * E16, cur.k[cc]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + 4 * kk + r == new_row) *reinterpret_cast<Raw*>(Vb + (int64_t)new_row * D + j * EPL) = cur.v[r];
        }
        floatx4 sp[NK];
#pragma unroll
        for (int cc = 0; cc < NK; ++cc) sp[cc] = mma16(cur.k[cc], qf[cc], T());
#pragma unroll
        for (int half = NK / 2; half; half >>= 1)
#pragma unroll
            for (int cc = 0; cc < half; ++cc) sp[cc] += sp[cc + half];
        floatx4 s = sp[0];
        if (t0 + kDecTile > r_end) {                         // the last tile of the split: wave-uniform
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + 4 * kk + r >= r_end) {
                    s[r] = -INFINITY;
                    cur.v[r] = Raw{};                        // zero weight times an infinite element would be NaN
                }
        }
        float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * c;
        if (__any(mx > m + kDecLazyLog2)) {
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m, mx), a = m_new > -INFINITY ? fast_exp2(m - m_new) : 1.f;
            l *= a;
#pragma unroll
            for (int e = 0; e < EPL; ++e) o[e] *= a;
            m = m_new;
        }
        const float ms = m > -INFINITY ? m : 0.f;
        float p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) { p[r] = fast_exp2(fmaf(s[r], c, -ms)); l += p[r]; }
        if constexpr (kPlanes) {
            typedef short shortx4 __attribute__((ext_vector_type(4)));
            shortx4 pp[3];                                   // p = pp[0] + pp[1] + pp[2]
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                const uintx2 h = {pack_bf16x2(p[0], p[1]), pack_bf16x2(p[2], p[3])};
                pp[x] = __builtin_bit_cast(shortx4, h);
#pragma unroll
                for (int r = 0; r < 4; ++r) p[r] -= __uint_as_float(r & 1 ? h[r >> 1] & 0xFFFF0000u : h[r >> 1] << 16);
            }
            struct Pairs { uint32_t of[EPL / 2]; } row[4];   // the rows' pieces, two elements each
#pragma unroll
            for (int r = 0; r < 4; ++r) row[r] = __builtin_bit_cast(Pairs, cur.v[r]);
#pragma unroll
            for (int x = 2; x >= 0; --x)
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    const uint32_t pick = e & 1 ? 0x07060302u : 0x05040100u;
                    const uintx2 v = {__builtin_amdgcn_perm(row[1].of[e >> 1], row[0].of[e >> 1], pick), __builtin_amdgcn_perm(row[3].of[e >> 1], row[2].of[e >> 1], pick)};
                    o[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(shortx4, v), pp[x], o[e], 0, 0, 0);
                }
        } else {
            float vf[4][EPL];
#pragma unroll
            for (int r = 0; r < 4; ++r) RowChunk<T, EPL>::load(cur.v[r].v, vf[r]);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int e = 0; e < EPL; ++e) o[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][e], p[r], o[e], 0, 0, 0);
        }
        cur = nxt;
    }
    };
    if constexpr (sizeof(T) == 2) {
        pass(std::true_type{});
        float probe = 0.f;                                   // NaN if a sum is no finite number
#pragma unroll
        for (int e = 0; e < EPL; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r) probe = fmaf(o[e][r], 0.f, probe);
        if (__any(probe != 0.f)) {                           // an infinity in V times a plane of 0
            fetch(first, cur);
            pass(std::false_type{});
        }
    } else {
        pass(std::false_type{});
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (j < heads) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < EPL; ++e) red[w][j][EPL * (4 * kk + r) + e] = o[e][r];
        if (kk == 0) { red[w][j][D] = m; red[w][j][D + 1] = l; }
    }
    __syncthreads();
    combine_waves<D, GT, kDecWaves<GT>, COHERENT>(red, heads, po, gbase, split);
}

// The same for a group of one head.
template <typename T, int D, bool COHERENT>
__device__ __forceinline__ void attend_split_one(const T* q, float c, T* Kb, T* Vb, const T* kn, const T* vn, int new_row,
                                                 int r_begin, int r_end, float (&red)[4][1][D + 2], const PartialOut& po, int split)
{
    constexpr int EPL = D / 16;
    const int tid = threadIdx.x, sub = tid & 15;
    float qv[EPL], m = -INFINITY, l = 0.f, o[EPL];
    RowChunk<T, EPL>::load(q + sub * EPL, qv);
#pragma unroll
    for (int e = 0; e < EPL; ++e) { qv[e] *= c; o[e] = 0.f; }
    Kb += sub * EPL; Vb += sub * EPL;
    if constexpr (COHERENT) { kn += sub * EPL; vn += sub * EPL; }         // the fused step: the only caller with a new row
    attend_rows<T, D>(Kb, Vb, Kb, Vb, kn, vn, new_row, r_begin, r_end, tid >> 4, qv, m, l, o);
    write_partial<D, COHERENT>(m, l, o, red, po, split);
}

template <typename T, int D, int GT, bool COHERENT>
__device__ __forceinline__ void attend_one(const T* q0, int heads, float c, T* Kb, T* Vb, const T* kn, const T* vn, int new_row,
                                           int r_begin, int r_end, float (&red)[kDecWaves<GT>][GT][D + 2],
                                           const PartialOut& po, int gbase, int split)
{
    if constexpr (kDecMfma<GT>) attend_split<T, D, GT, COHERENT>(q0, heads, c, Kb, Vb, kn, vn, new_row, r_begin, r_end, red, po, gbase, split);
    else attend_split_one<T, D, COHERENT>(q0, c, Kb, Vb, kn, vn, new_row, r_begin, r_end, red, po, split);
}

template <typename T, int D, int GT>
__global__ __launch_bounds__(64 * kDecWaves<GT>) void decode_partial_kernel(
    const T* __restrict__ q, const T* __restrict__ Kc, const T* __restrict__ Vc,
    const int32_t* __restrict__ len, int cap, int Hq, int Hkv, int gbase, float c, SplitRule rule, float* __restrict__ part)
{
    __shared__ float red[kDecWaves<GT>][GT][D + 2];
    const int G = Hq / Hkv;
    const int u = rule.unit(), split = rule.split();
    const int L = max(0, min(len[u], cap));
    const int rows = tiles_per_split<(GT > 1)>(tiles_of(L), rule) * kDecTile;
    const int r_begin = split * rows, r_end = min(L, r_begin + rows);
    if (split > 0 && r_begin >= L) return;                  // split 0 always reports (an empty state when L = 0)
    const PartialOut po(part, D, u, G, rule.most, rule.units);
    attend_one<T, D, GT, false>(q + ((int64_t)u * G + gbase) * D, min(GT, G - gbase), c, const_cast<T*>(Kc) + (int64_t)u * cap * D,
                                  const_cast<T*>(Vc) + (int64_t)u * cap * D, nullptr, nullptr, -1, r_begin, r_end, red, po, gbase, split);
}

struct Lengths { const int32_t* len[3]; int cap[3]; };     // row counts of a unit's parts (NULL: no such part), on the device

// Merges the splits of a unit that hold rows (all of them when no lengths are given), one workgroup per unit and head: a CU takes in
// 42 GB/s, and the 41 states of seven heads are 147 KB.
template <typename T, int D, int THREADS>
__global__ __launch_bounds__(THREADS) void decode_combine_kernel(const float* __restrict__ part, Lengths parts, SplitRule rule, int G, T* __restrict__ o)
{
    __shared__ floatx4 sum[THREADS];
    const int u = blockIdx.x, head = blockIdx.y;
    int nsplit = rule.most;
    if (parts.len[0]) {
        int tiles = 0;
        for (int p = 0; p < 3; ++p)
            if (parts.len[p]) tiles += tiles_of(max(0, min(parts.len[p][u], parts.cap[p])));
        const int per = tiles_per_split<false>(tiles, rule);
        nsplit = max(1, (tiles + per - 1) / per);
    }
    const PartialOut po(const_cast<float*>(part), D, u, G, rule.most, rule.units);
    HeadStates<D, THREADS, false> x;
    x.fetch_outputs(po, head, 0, nsplit);
    x.fetch_sums(po, head, nsplit);
    x.template finish<T>(nsplit, sum, o + ((int64_t)u * G + head) * D);
}

// ---------------------------------------------------------------- a decode step
// Append and attention of Algorithm 2 together.  The new row (k_new / v_new) becomes row len of the
// cache: the workgroup whose split contains that row takes it from k_new / v_new in its place in the row
// order (the arithmetic is that of the two separate calls) and stores it in the cache.
// One launch (kMerge): every workgroup of a unit - those without rows too - reads len and then arrives at a
// per-unit counter; the one that arrives last merges the unit's partial states, writes the output, advances len and
// clears the counter.  Since all workgroups have read len before the last one arrives, the update cannot be seen by
// a reader of the old value.
// Groups of heads with many splits: a second launch merges, a workgroup per unit and head, and advances len.  Every split leaves a
// state, those without rows one that says so (kNoRows), because len is about to change and cannot be read for their number.
// 28 heads on 4, 7200 rows, 41 splits: 12.3 us a layer, 14.4 with one launch (the last workgroup alone takes 4.3 us for the 147 KB of a
// unit's states); the merge shared by the last workgroups to arrive, each waiting for the counter a bounded number of times: 19.5.
constexpr float kNoRows = -1.f;                              // instead of a sum

// One wave per head, all of at most kMergeSplits states on the way at once; the sums are those of HeadStates, bit for bit.
template <typename T, int D>
__device__ __forceinline__ void merge_few_states(const PartialOut& po, int head, int nsplit, T* __restrict__ out) {
    constexpr int EPL = D / 64, kMost = kMergeSplits<T, D>;
    const int lane = threadIdx.x & 63;
    HeadStates<D, 512, true> x;
    float v[kMost][EPL];
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(po.o, 0, 0x7FFFFFFF, 0x00020000);
#pragma unroll
    for (int s = 0; s < kMost; ++s)
        if (s < nsplit) {
            const int at = (head * po.nsplit + s) * (D * 4) + lane * (EPL * 4);
            if constexpr (EPL == 2) {
                const uintx2 r = __builtin_bit_cast(uintx2, __builtin_amdgcn_raw_buffer_load_b64(rs, at, 0, 16));      // sc1, as load16_coherent
                v[s][0] = __uint_as_float(r[0]);
                v[s][EPL - 1] = __uint_as_float(r[1]);
            } else v[s][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, at, 0, 16));
        }
    x.fetch_sums(po, head, nsplit);
    const float w = x.weight();
    static_assert(kMost <= HeadStates<D, 512, true>::kGroups, "one state in each partial sum");
    float acc[EPL] = {};
#pragma unroll
    for (int s = 0; s < kMost; ++s)
        if (s < nsplit) {
            const float ws = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), s));
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
                float p = fmaf(ws, v[s][e], 0.f);
                asm volatile("" : "+v"(p));                  // rounded before it is added
                acc[e] = s == 0 ? p : acc[e] + p;
            }
        }
#pragma unroll
    for (int e = 0; e < EPL; ++e) out[lane * EPL + e] = to_out<T>(acc[e]);
}

template <typename T, int D, int GT, bool kMerge>
__global__ __launch_bounds__(64 * kDecWaves<GT>) void decode_step_kernel(
    const T* __restrict__ q, T* __restrict__ Kc, T* __restrict__ Vc, int32_t* __restrict__ len, int cap,
    const T* __restrict__ k_new, const T* __restrict__ v_new, int Hq, int Hkv, float c, SplitRule rule,
    float* __restrict__ part, unsigned* __restrict__ arrived, T* __restrict__ out)
{
    constexpr int kThreads = 64 * kDecWaves<GT>;
    __shared__ __attribute__((aligned(16))) union { float red[kDecWaves<GT>][GT][D + 2]; floatx4 sum[GT == 1 ? kThreads : 1]; } lds;
    __shared__ int is_last;
    const int G = Hq / Hkv;
    const int u = rule.unit(), split = rule.split(), tid = threadIdx.x;
    const int Lraw = len[u];
    const bool room = Lraw >= 0 && Lraw < cap;               // a full cache is left unchanged, as by the append call
    const int L0 = max(0, min(Lraw, cap));
    const int L = L0 + (room ? 1 : 0);                       // rows attended: the new one included
    const int rows = tiles_per_split<(GT > 1)>(tiles_of(L), rule) * kDecTile;
    const int r_begin = split * rows, r_end = min(L, r_begin + rows);
    const int nsplit = max(1, (L + rows - 1) / rows);
    const PartialOut po(part, D, u, G, rule.most, rule.units);

    if (split < nsplit)
        attend_one<T, D, GT, kMerge>(q + (int64_t)u * G * D, G, c, Kc + (int64_t)u * cap * D, Vc + (int64_t)u * cap * D,
                                     k_new + (int64_t)u * D, v_new + (int64_t)u * D, room ? L0 : -1, r_begin, r_end, lds.red, po, 0, split);
    else if (!kMerge && tid < G) {
        po.ml[2 * ((int64_t)tid * po.nsplit + split)] = -INFINITY;
        po.ml[2 * ((int64_t)tid * po.nsplit + split) + 1] = kNoRows;
    }
    if constexpr (kMerge) {
        // The partial state went out with device-scope (write-through) stores: once they have completed
        // (vmcnt 0) it is visible to every XCD, and only then is this workgroup counted.  A release fence
        // would do the same by writing back the whole L2, 150 us per launch here.
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) is_last = atomicAdd(&arrived[u], 1u) == rule.most - 1u;
        __syncthreads();
        if (!is_last) return;
        if (tid == 0) {
            if (room) len[u] = Lraw + 1;
            arrived[u] = 0u;                                 // ready for the next step
        }
        T* const o = out + (int64_t)u * G * D;
        if constexpr (GT == 1) {
            HeadStates<D, kThreads, true> x;
            x.fetch_outputs(po, 0, 0, nsplit);
            x.fetch_sums(po, 0, nsplit);
            x.template finish<T>(nsplit, lds.sum, o);
        } else {
            static_assert(GT <= kDecWaves<GT>, "a wave per head");
            const int head = __builtin_amdgcn_readfirstlane(tid >> 6);
            if (head < G) merge_few_states<T, D>(po, head, nsplit, o + head * D);
        }
    }
}

template <typename T, int D, int THREADS>
__global__ __launch_bounds__(THREADS) void decode_step_combine_kernel(const float* __restrict__ part, int32_t* __restrict__ len, int cap, SplitRule rule,
                                                                      int G, T* __restrict__ o)
{
    __shared__ floatx4 sum[THREADS];
    using States = HeadStates<D, THREADS, false>;
    const int u = blockIdx.x, head = blockIdx.y;
    const PartialOut po(const_cast<float*>(part), D, u, G, rule.most, rule.units);
    States x;
    const int first = (rule.least + States::kGroups - 1) / States::kGroups * States::kGroups;      // states that most likely hold rows: not waited for the sums
    x.fetch_outputs(po, head, 0, min(first, rule.most));
    x.fetch_sums(po, head, rule.most);
    const bool none = x.l == kNoRows || (int)(threadIdx.x & 63) >= rule.most;
    const int nsplit = 64 - __popcll(__ballot(none));
    if (none) x.l = 0.f;
    x.fetch_outputs(po, head, first, nsplit);
    if (head == 0 && threadIdx.x == 0) {
        const int L = len[u];
        if (L >= 0 && L < cap) len[u] = L + 1;
    }
    x.template finish<T>(nsplit, sum, o + ((int64_t)u * G + head) * D);
}

// ---------------------------------------------------------------- mixed-precision cache
struct QTensor {                 // device pointers of one mixed-precision tensor, by value in the kernel arguments
    const uint8_t* hi_codes; const uint32_t* hi_params;
    const uint8_t* lo_codes; const uint32_t* lo_params;
};

// the NB-byte code string of one lane -> EPL = NB * 8 / BITS floats (codes as numbers), element e at bits [e*BITS, ..)
template <int BITS, int NW>
__device__ __forceinline__ void codes_to_floats(const uint32_t (&w)[NW], float (&f)[NW * 32 / BITS]) {
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        if constexpr (BITS == 4) {
            const uint32_t ev = w[i] & 0x0F0F0F0Fu, od = (w[i] >> 4) & 0x0F0F0F0Fu;   // codes 0,2,4,6 / 1,3,5,7 as bytes
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                f[8 * i + 2 * b] = (float)((ev >> (8 * b)) & 0xFFu);
                f[8 * i + 2 * b + 1] = (float)((od >> (8 * b)) & 0xFFu);
            }
        } else {
#pragma unroll
            for (int sft = 0; sft < 4; ++sft) {
                const uint32_t t = (w[i] >> (2 * sft)) & 0x03030303u;                  // codes sft, sft+4, sft+8, sft+12 as bytes
#pragma unroll
                for (int b = 0; b < 4; ++b) f[16 * i + 4 * b + sft] = (float)((t >> (8 * b)) & 0xFFu);
            }
        }
    }
}

template <int NW> __device__ __forceinline__ void load_words(const uint8_t* p, uint32_t (&w)[NW]);
template <> __device__ __forceinline__ void load_words<4>(const uint8_t* p, uint32_t (&w)[4]) {
    const uintx4 v = load16(p); w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
}
template <> __device__ __forceinline__ void load_words<2>(const uint8_t* p, uint32_t (&w)[2]) {
    const uintx2 v = *reinterpret_cast<const uintx2*>(p); w[0] = v[0]; w[1] = v[1];
}
template <> __device__ __forceinline__ void load_words<1>(const uint8_t* p, uint32_t (&w)[1]) {
    w[0] = *reinterpret_cast<const uint32_t*>(p);
}

__device__ __forceinline__ void unpack_params(uint32_t v, float& scale, float& zero) {   // fp16 scale (low half), fp16 zero (high half)
    scale = (float)__builtin_bit_cast(_Float16, (uint16_t)(v & 0xFFFFu));
    zero = (float)__builtin_bit_cast(_Float16, (uint16_t)(v >> 16));
}

// Eq. (5) over [4-bit rows of T | 2-bit rows of the other tokens | rows appended during decoding], for groups of several
// heads: the tiles of attend_split.  V rows are dequantised to fp32 (zero + scale * code) in registers.  K rows are for fp32
// queries; bf16 queries meet the doubled codes about their middle, 2 code - 15 or 2 code - 3, in exact bf16 products:
//   q . (zero + scale * code) = (zero + scale * mid) * sum(q) + scale / 2 * (q . (2 code - 2 mid))
// (either term is of the size of the scores then; with plain codes they cancel: 2.4e-6 of the output, fp32 queries, against
// 0.36e-6 dequantised).
// Lane (j, kk) reads a quarter kk of the codes of K row j in one piece (the queries are held in that order) and, of the V
// rows 4 kk + r, the codes of elements EPL j ... EPL j + EPL - 1.  The tiles of the three parts form one list, dealt to
// splits and waves in turn.  One step of 28 heads on 4, 18432 rows: 36 us a layer (append and merge
// included), 66 with the heads in turn on the vector units.
template <typename T, int D, int GT>
__global__ __launch_bounds__(64 * kDecWaves<GT>) void decode_q_partial_kernel(
    const T* __restrict__ q, QTensor Kq, QTensor Vq, const int32_t* __restrict__ len_hi, const int32_t* __restrict__ len_lo,
    int cap_hi, int cap_lo, const T* __restrict__ Kt, const T* __restrict__ Vt, const int32_t* __restrict__ len_t, int cap_t,
    int Hq, int Hkv, int gbase, float c, float* __restrict__ part, SplitRule rule)
{
    constexpr bool kExact = sizeof(T) == 2;                              // codes meet the queries in bf16
    constexpr int EPL = D / 16, QE = D / 4, E16 = 16 / (int)sizeof(T), NK = QE / E16, NP = kExact ? 4 : 1, NW4 = QE / 8, NW2 = QE / 16;
    __shared__ float red[kDecWaves<GT>][GT][D + 2];
    const int G = Hq / Hkv, heads = min(GT, G - gbase);
    const int u = rule.unit(), split = rule.split();
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, j = lane & 15, kk = lane >> 4;
    const int L4 = max(0, min(len_hi[u], cap_hi)), L2 = max(0, min(len_lo[u], cap_lo)), Lt = Kt ? max(0, min(len_t[u], cap_t)) : 0;
    const int T4 = tiles_of(L4), T2 = tiles_of(L2), Tt = tiles_of(Lt);
    const int per = tiles_per_split<true>(T4 + T2 + Tt, rule);
    if (rule.turn && split > 0 && split * per >= T4 + T2 + Tt) return;   // equal splits all report, and are all merged
    const int t_end = min(T4 + T2 + Tt, (split + 1) * per), t_codes = min(t_end, T4 + T2);

    struct Codes { uint32_t k[NW4], kp[NP], v[4], vp[4]; };
    auto fetch = [&](int t, Codes& x) {
        const bool hi = t < T4;                                          // wave-uniform
        const int t0 = (hi ? t : t - T4) * kDecTile, last = (hi ? L4 : L2) - 1;
        const int64_t base = (int64_t)u * (hi ? cap_hi : cap_lo);
        const uint32_t* kpar = hi ? Kq.hi_params : Kq.lo_params;
        const uint32_t* vpar = hi ? Vq.hi_params : Vq.lo_params;
        const int64_t rk = base + min(t0 + j, last);                     // rows past the end re-read the last one and weigh nothing
        if (hi) {
            load_words<NW4>(Kq.hi_codes + rk * (D / 2) + kk * (QE / 2), x.k);
        } else {
            uint32_t lo[NW2];
            load_words<NW2>(Kq.lo_codes + rk * (D / 4) + kk * (QE / 4), lo);
#pragma unroll
            for (int i = 0; i < NW4; ++i) x.k[i] = i < NW2 ? lo[i % NW2] : 0u;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t row = base + min(t0 + 4 * kk + r, last);
            if (hi) x.v[r] = reinterpret_cast<const typename CodeWord<EPL, 4>::type*>(Vq.hi_codes + row * (D / 2))[j];
            else x.v[r] = reinterpret_cast<const typename CodeWord<EPL, 2>::type*>(Vq.lo_codes + row * (D / 4))[j];
            x.vp[r] = vpar[row];
            if (kExact) x.kp[r % NP] = kpar[row];
        }
        if (!kExact) x.kp[0] = kpar[rk];
    };
    int t = split * per + w;
    Codes cur;
    if (t < t_codes) fetch(t, cur);

    uintx4 qf[NK];                                                       // elements QE kk ... of head j
    float qsum = 0.f;
#pragma unroll
    for (int cc = 0; cc < NK; ++cc) {
        qf[cc] = uintx4{0, 0, 0, 0};
        if (j < heads) {
            const T* qp = q + ((int64_t)u * G + gbase + j) * D + kk * QE + cc * E16;
            float f[E16];
            qf[cc] = load16(qp);
            RowChunk<T, E16>::load(qp, f);
#pragma unroll
            for (int e = 0; e < E16; ++e) qsum += f[e];
        }
    }
    qsum += __shfl_xor(qsum, 16);
    qsum += __shfl_xor(qsum, 32);
    auto products = [&](const uintx4 (&kf)[NK]) {
        floatx4 sp[NK];
#pragma unroll
        for (int cc = 0; cc < NK; ++cc) sp[cc] = mma16(kf[cc], qf[cc], T());
#pragma unroll
        for (int half = NK / 2; half; half >>= 1)
#pragma unroll
            for (int cc = 0; cc < half; ++cc) sp[cc] += sp[cc + half];
        return sp[0];
    };
    float m = -INFINITY, l = 0.f;                                        // head j
    floatx4 o[EPL];                                                      // o[e][r]: element EPL (4 kk + r) + e of head j
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[e] = floatx4{0.f, 0.f, 0.f, 0.f};
    // one tile of which the first `left` rows exist; s: its scores before the softmax scale
    auto attend = [&](floatx4 s, float (&vf)[4][EPL], int left) {
        if (left < kDecTile) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * kk + r >= left) {
                    s[r] = -INFINITY;
#pragma unroll
                    for (int e = 0; e < EPL; ++e) vf[r][e] = 0.f;        // zero weight times an infinite element would be NaN
                }
        }
        const float mx1 = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * c;
        if (__any(mx1 > m + kDecLazyLog2)) {
            float mx = fmaxf(mx1, __shfl_xor(mx1, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m, mx), a = m_new > -INFINITY ? fast_exp2(m - m_new) : 1.f;
            l *= a;
#pragma unroll
            for (int e = 0; e < EPL; ++e) o[e] *= a;
            m = m_new;
        }
        const float ms = m > -INFINITY ? m : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float p = fast_exp2(fmaf(s[r], c, -ms));
            l += p;
#pragma unroll
            for (int e = 0; e < EPL; ++e) o[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][e], p, o[e], 0, 0, 0);
        }
    };
    for (; t < t_codes; t += kDecWaves<GT>) {
        Codes nxt;
        if (t + kDecWaves<GT> < t_codes) fetch(t + kDecWaves<GT>, nxt);  // in flight while this tile is multiplied
        const bool hi = t < T4;
        float kv[QE], vf[4][EPL], scale, zero;
        if (hi) {
            codes_to_floats<4, NW4>(cur.k, kv);
        } else {
            uint32_t lo[NW2];
#pragma unroll
            for (int i = 0; i < NW2; ++i) lo[i] = cur.k[i];
            codes_to_floats<2, NW2>(lo, kv);
        }
        const float two_mid = hi ? 15.f : 3.f;
        if (!kExact) unpack_params(cur.kp[0], scale, zero);
        uintx4 kf[NK];
#pragma unroll
        for (int cc = 0; cc < NK; ++cc) {
            RawChunk<T, E16> raw;
#pragma unroll
            for (int e = 0; e < E16; ++e) raw.v[e] = to_out<T>(kExact ? fmaf(2.f, kv[cc * E16 + e], -two_mid) : fmaf(scale, kv[cc * E16 + e], zero));
            kf[cc] = __builtin_bit_cast(uintx4, raw);
        }
        floatx4 s = products(kf);
        if (kExact) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                unpack_params(cur.kp[r % NP], scale, zero);
                s[r] = fmaf(0.5f * scale, s[r], fmaf(0.5f * scale, two_mid, zero) * qsum);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            unpack_params(cur.vp[r], scale, zero);
#pragma unroll
            for (int e = 0; e < EPL; ++e) vf[r][e] = fmaf(scale, (float)(hi ? (cur.v[r] >> (4 * e)) & 15u : (cur.v[r] >> (2 * e)) & 3u), zero);
        }
        attend(s, vf, hi ? L4 - t * kDecTile : L2 - (t - T4) * kDecTile);
        cur = nxt;
    }
    for (; t < t_end; t += kDecWaves<GT>) {                              // rows appended during decoding, as stored
        const int t0 = (t - T4 - T2) * kDecTile;
        const T* kp = Kt + ((int64_t)u * cap_t + min(t0 + j, Lt - 1)) * D + kk * QE;
        uintx4 kf[NK];
#pragma unroll
        for (int cc = 0; cc < NK; ++cc) kf[cc] = load16(kp + cc * E16);
        float vf[4][EPL];
#pragma unroll
        for (int r = 0; r < 4; ++r) RowChunk<T, EPL>::load(Vt + ((int64_t)u * cap_t + min(t0 + 4 * kk + r, Lt - 1)) * D + j * EPL, vf[r]);
        attend(products(kf), vf, Lt - t0);
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (j < heads) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < EPL; ++e) red[w][j][EPL * (4 * kk + r) + e] = o[e][r];
        if (kk == 0) { red[w][j][D] = m; red[w][j][D + 1] = l; }
    }
    __syncthreads();
    combine_waves<D, GT, kDecWaves<GT>>(red, heads, PartialOut(part, D, u, G, rule.most, rule.units), gbase, split);
}

// ---- the same, for one head per group: integer matrix products on the codes.
// A group of one head leaves 15 of 16 columns of a floating-point tile empty, and the vector units need 1.6 instructions per
// element and side.  The codes are small integers, so both products run on v_mfma_i32_16x16x64_i8, the other operand cut
// into four signed bytes of a 30-bit fixed-point number (the columns that one head leaves empty): every product and sum is
// exact, the only rounding is that of a query element to 2^-29 of the largest and of a weight to 2^-27 of the largest that the
// wave has met under the present exponent offset.
// Scores and outputs are sums of two terms that may cancel,
//   q . (zero + scale * code) = zero * sum(q) + scale * (q . code),
//   sum_j p_j (zero_j + scale_j * code_j) = sum_j p_j zero_j + sum_j w_j code_j,   w_j = p_j scale_j in fixed point,
// whichever number of a row's codes is taken for the middle one: at the lowest code where a row has an outlier, in the middle of
// the codes where it has none.  So they meet in double precision: the first is summed in it (one row per lane, 64 rows a step),
// the second is exact, and what the fixed point leaves of p_j scale_j is weighed with the code that stands for the value 0,
// which leaves the output with a slightly other weight of the whole row.  fp32, added about the middle: scores up to 1e-3 off
// beside an outlier of 1000 in rows of K (now by their own rounding), single channels up to 1.1e-5 beside one in V (now 1e-7);
// from the lowest code: 1e-3 beside an outlier of -1000 in K, 1.8e-6 of ordinary outputs (0.3e-6).
// A wave takes 64 rows at a time:
//   scores   A = the bytes of q (row m of the tile: byte m % 4), B = 16 cached rows, lane (n, kk) unpacking a quarter kk of the
//            codes of row n (1.5 instructions per 4 codes): the lane's accumulators are the four bytes' sums of row n, and
//            lane L keeps those of row L.
//   weights  one row per lane: exponential, p * scale rounded to fixed point, its bytes to LDS.
//   output   A = the bytes of the 64 weights, B = codes of 16 channels x 64 rows, from the row-major codes in LDS through the
//            transposing 4-bit read (2-bit codes: two channels a nibble).
// The exponent offset is the wave's and moves lazily; it and the fixed-point scale of the weights are fixed until a row
// outgrows them, and then the integer sums go over to fp32.  A new offset takes a new scale: rows of V a thousand times larger
// than the others, which then turn out to weigh nothing, would leave the others 10 bits less (with 1e4 and 1e-3, 3 % off).
// Four layers of 128 units x 8192 rows: 116 us a step, 23 us a layer in this kernel (151 and 33 on the vector units).
// Error of the output against float64, fp32 queries, n = 300 to 30000: 2.0e-7 in the mean (2.3e-6 on the vector units).
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx2 __attribute__((ext_vector_type(2)));

// |x| < 2^30 as four signed bytes of weight 256^i, byte i in bits 8 i ...
__device__ __forceinline__ uint32_t signed_bytes(int x) { return ((uint32_t)x + 0x00808080u) ^ 0x00808080u; }
// and back, from sums over each byte (of one row's channels: below 2^18, two of them fit an integer)
__device__ __forceinline__ double from_bytes(const intx4& s) {
    return fma(fma(fma((double)s[3], 256.0, (double)s[2]), 256.0, (double)s[1]), 256.0, (double)s[0]);
}
__device__ __forceinline__ double from_row_bytes(const intx4& s) {
    return fma((double)(s[3] * 256 + s[2]), 65536.0, (double)(s[1] * 256 + s[0]));
}
// exponent e of a power of two with |x| * 2^e in [2^(bits - 1), 2^bits); 0 for x = 0
__device__ __forceinline__ int fixed_exponent(float x, int bits) {
    return x > 0.f ? max(-100, min(100, bits - (int)((__float_as_uint(x) >> 23) & 255u) + 126)) : 0;
}
__device__ __forceinline__ float power_of_two(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }

constexpr float kNoScale = 0x1p100f;      // fixed-point scale until a weight is met: the largest that fixed_exponent gives

// Rows of BITS-bit codes as a wave of decode_q1_partial_kernel takes them.
template <int D, int BITS> struct CodeRows {
    static constexpr int RB = D * BITS / 8;                  // bytes of a row
    static constexpr int CPR = RB / 16;                      // 16-byte chunks of a row = V loads per lane for 64 rows
    static constexpr int NW = RB / 16;                       // dwords of a quarter of a row
    static constexpr int ND = D / 16;                        // dwords of one code per byte that they unpack to
    // chunk swizzle of the rows in LDS: 16 rows read at one 8-byte piece fall on different banks, or on the two halves of one chunk
    __device__ static __forceinline__ int swizzle(int row) { return CPR == 4 ? (row >> 2) & 3 : CPR == 2 ? (row >> 3) & 1 : 0; }
    // one code per byte; the same order of channels as query_operand
    __device__ static __forceinline__ void unpack(const uint32_t (&w)[NW], uint32_t (&b)[ND]) {
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int s = 0; s < 8 / BITS; ++s) b[s * NW + i] = (w[i] >> (BITS * s)) & (BITS == 4 ? 0x0F0F0F0Fu : 0x03030303u);
    }
    // d: the bytes of this lane's quarter of the channels in their own order
    __device__ static __forceinline__ void query_operand(const uint32_t (&d)[ND], uint32_t (&a)[ND]) {
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int s = 0; s < 8 / BITS; ++s) {
                if constexpr (BITS == 4) {
                    a[s * NW + i] = __builtin_amdgcn_perm(d[2 * i + 1], d[2 * i], 0x06040200u + 0x01010101u * s);
                } else {
                    const uint32_t sel = (uint32_t)s | (uint32_t)(4 + s) << 8;
                    const uint32_t lo = __builtin_amdgcn_perm(d[4 * i + 1], d[4 * i], sel), hi = __builtin_amdgcn_perm(d[4 * i + 3], d[4 * i + 2], sel);
                    a[s * NW + i] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                }
            }
    }
};

template <typename T, int D>
__global__ __launch_bounds__(256, D == 128 ? 3 : 4) void decode_q1_partial_kernel(
    const T* __restrict__ q, QTensor Kq, QTensor Vq, const int32_t* __restrict__ len_hi, const int32_t* __restrict__ len_lo,
    int cap_hi, int cap_lo, const T* __restrict__ Kt, const T* __restrict__ Vt, const int32_t* __restrict__ len_t, int cap_t,
    float c, float* __restrict__ part, SplitRule rule)
{
    constexpr int NG = D / 16, ND = D / 16, NM = D / 64;     // output blocks of 16 channels; dwords and products of an operand
    __shared__ __attribute__((aligned(16))) uint8_t vrows[4][64 * D / 2];    // per wave: V codes of its 64 rows
    __shared__ __attribute__((aligned(16))) uint8_t wbytes[4][4 * 64];       // per wave: byte i of the 64 weights at 64 i
    __shared__ __attribute__((aligned(16))) uint8_t qbytes[4][4 * D];        // per wave: byte i of the query at D i
    __shared__ float red[12][1][D + 2];                      // per wave: states of the 4-bit, the 2-bit and the appended rows
    const int u = blockIdx.y, split = blockIdx.x, nsplit = rule.most;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15, kk = lane >> 4;
    const int L4 = max(0, min(len_hi[u], cap_hi)), L2 = max(0, min(len_lo[u], cap_lo));
    // Blocks of 64 rows, the 4-bit ones first, dealt to the splits in shares of as many bytes and to their waves in turn.  In shares of as
    // many blocks the first split, all of it 4-bit rows, reads 1.6 times the mean: us, so -> now: 4 layers of 128 units x 8192, a quarter at
    // 4 bits 111 -> 108; of 40 x 20 000, 30 % 94.6 -> 89.6; 55 % of 128 x 8192 127 -> 126.
    constexpr int kBytes4 = D / 2 + 4, kBytes2 = D / 4 + 4;  // of a row of K or V
    const int B4 = (L4 + 63) >> 6, B2 = (L2 + 63) >> 6;
    auto edge = [&](int sp) {                                // the block nearest to the sp-th share's end
        const int64_t at = ((int64_t)kBytes4 * B4 + (int64_t)kBytes2 * B2) * sp / nsplit, over = at - (int64_t)kBytes4 * B4;
        return (int)(over <= 0 ? (at + kBytes4 / 2) / kBytes4 : B4 + (over + kBytes2 / 2) / kBytes2);
    };
    const int b0 = edge(split), b1 = edge(split + 1);

    double qsum = 0.0;                                       // sum of the scaled query
    float q_inv = 1.f;                                       // 1 / its fixed-point scale
    auto prepare_query = [&]() {
        float f[D / 64], mx = 0.f;
#pragma unroll
        for (int e = 0; e < D / 64; ++e) {
            f[e] = (float)q[(int64_t)u * D + 64 * e + lane] * c;
            qsum += (double)f[e];
            mx = fmaxf(mx, fabsf(f[e]));
        }
        qsum = wave_sum(qsum);
        const int ex = fixed_exponent(wave_max(mx), 29);
        q_inv = power_of_two(-ex);
#pragma unroll
        for (int e = 0; e < D / 64; ++e) {
            const uint32_t z = signed_bytes(__float2int_rn(f[e] * power_of_two(ex)));
#pragma unroll
            for (int i = 0; i < 4; ++i) qbytes[w][i * D + 64 * e + lane] = (uint8_t)(z >> (8 * i));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };

    // One part of the cache: blocks first, first + 4, ... below last (of 64 rows) of L rows -> the state red[out].
    bool have_query = false;
    auto attend_codes = [&](auto bits, const uint8_t* kc, const uint32_t* kp, const uint8_t* vc, const uint32_t* vp, int64_t base,
                            int L, int first, int last, float* out) {
        constexpr int BITS = decltype(bits)::value, kTop = (1 << BITS) - 1;
        using R = CodeRows<D, BITS>;
        struct Block { uint32_t k[4][R::NW]; uintx4 v[R::CPR]; uint32_t kp, vp; };
        auto fetch = [&](int blk, Block& x) {
            const int r0 = blk * 64;                         // rows past the end re-read the last one and weigh nothing
#pragma unroll
            for (int t = 0; t < 4; ++t) load_words<R::NW>(kc + (base + min(r0 + 16 * t + n, L - 1)) * R::RB + kk * (R::RB / 4), x.k[t]);
#pragma unroll
            for (int p = 0; p < R::CPR; ++p) {
                const int piece = p * 64 + lane;
                x.v[p] = load16(vc + (base + min(r0 + piece / R::CPR, L - 1)) * R::RB + (piece % R::CPR) * 16);
            }
            const int64_t row = base + min(r0 + lane, L - 1);
            x.kp = kp[row];
            x.vp = vp[row];
        };
        // of the wave: m, ws, w_inv (the scale of the weights and its reciprocal), any (integer sums other than 0)
        float m = -INFINITY, l = 0.f, ws = kNoScale, w_inv = 1.f / kNoScale, of[NG];
        double zacc = 0.0;                                    // this lane's rows: what their weight has besides the integer sums
        bool any = false;
        intx4 o[NG];                                          // sums of weight bytes times codes
#pragma unroll
        for (int g = 0; g < NG; ++g) { of[g] = 0.f; o[g] = intx4{0, 0, 0, 0}; }
        auto flush = [&](float a) {                           // all sums -> fp32, which are then scaled by a
            const double z = any ? wave_sum(zacc) : 0.0;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (any) of[g] = (float)fma(from_bytes(o[g]), (double)w_inv, z + (double)of[g]);
                of[g] *= a;
                o[g] = intx4{0, 0, 0, 0};
            }
            zacc = 0.0;
            any = false;
        };
        if (first < last) {
            Block cur;
            fetch(first, cur);
            if (!have_query) prepare_query();
            have_query = true;
            uint32_t qa[ND];
            {
                uint32_t d[ND];
#pragma unroll
                for (int i = 0; i < ND; ++i) d[i] = *reinterpret_cast<const uint32_t*>(&qbytes[w][(n & 3) * D + kk * (D / 4) + 4 * i]);
                R::query_operand(d, qa);
            }
            auto query = [&](int h) { return intx4{(int)qa[4 * h], (int)qa[4 * h + 1], (int)qa[4 * h + 2], (int)qa[4 * h + 3]}; };
            uint8_t* vb = vrows[w];
            for (int blk = first; blk < last; blk += 4) {
#pragma unroll
                for (int p = 0; p < R::CPR; ++p) {
                    const int piece = p * 64 + lane, r = piece / R::CPR;
                    store16(vb + r * R::RB + ((piece % R::CPR) ^ R::swizzle(r)) * 16, cur.v[p]);
                }
                intx4 mine;                                  // lane L: of row L
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    uint32_t b[ND];
                    R::unpack(cur.k[t], b);
                    intx4 s = {0, 0, 0, 0};
#pragma unroll
                    for (int h = 0; h < NM; ++h)
                        s = __builtin_amdgcn_mfma_i32_16x16x64_i8(query(h), intx4{(int)b[4 * h], (int)b[4 * h + 1], (int)b[4 * h + 2], (int)b[4 * h + 3]}, s, 0, 0, 0);
                    if (t == 0 || kk == t) mine = s;
                }
                float ks, kz, vs, vz;
                unpack_params(cur.kp, ks, kz);
                unpack_params(cur.vp, vs, vz);
                if (blk + 4 < last) fetch(blk + 4, cur);     // in flight while this block is worked on
                const bool valid = blk * 64 + lane < L;
                const float sc = valid ? (float)fma((double)(ks * q_inv), from_row_bytes(mine), (double)kz * qsum) : -INFINITY;
                if (__any(sc > m + kDecLazyLog2)) {
                    const float top = wave_max(sc), a = m > -INFINITY ? fast_exp2(m - top) : 0.f;
                    flush(a);
                    l *= a;
                    m = top;
                    ws = kNoScale;                           // weights under the new offset: the rows that set the scale may not count any more
                }
                const float p = valid ? fast_exp2(sc - (m > -INFINITY ? m : 0.f)) : 0.f, wt = p * vs;
                l += p;
                if (__any(fabsf(wt) * ws >= 0x1p30f)) {
                    flush(1.f);
                    const int ex = fixed_exponent(wave_max(fabsf(wt)), 28);
                    ws = power_of_two(ex);
                    w_inv = power_of_two(-ex);
                }
                const float wf = rintf(wt * ws);
                // the rest of p * scale, exact, times the code of the value 0 (NaN where a weight is no number)
                const float rest = fmaf(-wf, w_inv, wt) + fmaf(p, vs, -wt);
                const float code0 = fminf(fmaxf(-vz * __builtin_amdgcn_rcpf(vs), 0.f), (float)kTop);
                zacc = fma((double)p, (double)vz, zacc) + (double)(rest * code0);
                any = true;
                const uint32_t z = signed_bytes(__float2int_rn(wf));
                // byte i of row `lane`, where the unpacked nibbles of a transposed read have that row
                const int pos = 16 * kk + 8 * (n >> 3) + 4 * (n & 1) + ((n & 7) >> 1);
#pragma unroll
                for (int i = 0; i < 4; ++i) wbytes[w][64 * i + pos] = (uint8_t)(z >> (8 * i));
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const uintx4 wa = load16(&wbytes[w][64 * (n & 3) + 16 * kk]);
                const intx4 a4 = __builtin_bit_cast(intx4, wa);
                const int vrow = 16 * kk + n;
#pragma unroll
                for (int g = 0; g < R::RB / 8; ++g) {        // an 8-byte piece of 64 rows
                    using lds_ptr = __attribute__((address_space(3))) intx2*;
                    const uint8_t* at = vb + vrow * R::RB + ((g >> 1) ^ R::swizzle(vrow)) * 16 + (g & 1) * 8;
                    const intx2 t2 = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_ptr)at);
                    const uint32_t x0 = (uint32_t)t2[0], x1 = (uint32_t)t2[1];
                    constexpr uint32_t M = BITS == 4 ? 0x0F0F0F0Fu : 0x03030303u;
                    if constexpr (BITS == 4) {
                        o[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a4, intx4{(int)(x0 & M), (int)(x0 >> 4 & M), (int)(x1 & M), (int)(x1 >> 4 & M)}, o[g], 0, 0, 0);
                    } else {
                        o[2 * g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a4, intx4{(int)(x0 & M), (int)(x0 >> 4 & M), (int)(x1 & M), (int)(x1 >> 4 & M)}, o[2 * g], 0, 0, 0);
                        o[2 * g + 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a4, intx4{(int)(x0 >> 2 & M), (int)(x0 >> 6 & M), (int)(x1 >> 2 & M), (int)(x1 >> 6 & M)}, o[2 * g + 1], 0, 0, 0);
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
            flush(1.f);
            l = wave_sum(l);
        }
        // all four quarters of the wave hold the same sums: each writes a quarter of the blocks
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (g % 4 == kk) out[BITS == 4 ? 16 * g + n : 32 * (g >> 1) + 2 * n + (g & 1)] = of[g];
        if (lane == 0) { out[D] = m; out[D + 1] = l; }
    };
    // this wave's first block at or after `from`
    auto next_block = [&](int from) { const int behind = from - (b0 + w); return b0 + w + (behind > 0 ? (behind + 3) / 4 * 4 : 0); };
    attend_codes(std::integral_constant<int, 4>(), Kq.hi_codes, Kq.hi_params, Vq.hi_codes, Vq.hi_params, (int64_t)u * cap_hi,
                 L4, b0 + w, min(b1, B4), red[3 * w][0]);
    attend_codes(std::integral_constant<int, 2>(), Kq.lo_codes, Kq.lo_params, Vq.lo_codes, Vq.lo_params, (int64_t)u * cap_lo,
                 L2, next_block(B4) - B4, b1 - B4, red[3 * w + 1][0]);

    // rows appended during decoding, as stored: 16 lanes per row, as in a cache without codes
    float* out = red[3 * w + 2][0];
    int r_begin = 0, r_end = 0;
    if (Kt) split_range64(max(0, min(len_t[u], cap_t)), split, nsplit, r_begin, r_end);
    if (r_begin < r_end) {
        constexpr int EPL = D / 16;
        float qv[EPL], m = -INFINITY, l = 0.f, o[EPL];
        RowChunk<T, EPL>::load(q + (int64_t)u * D + n * EPL, qv);
#pragma unroll
        for (int e = 0; e < EPL; ++e) { qv[e] *= c; o[e] = 0.f; }
        const int64_t base = (int64_t)u * cap_t * D + n * EPL;
        attend_rows<T, D>(Kt + base, Vt + base, nullptr, nullptr, nullptr, nullptr, -1, r_begin, r_end, tid >> 4, qv, m, l, o);
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            const float m2 = __shfl_xor(m, off), l2 = __shfl_xor(l, off);
            float o2[EPL];
#pragma unroll
            for (int e = 0; e < EPL; ++e) o2[e] = __shfl_xor(o[e], off);
            merge_state<EPL>(m, l, o, m2, l2, o2);
        }
        if (kk == 0) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) out[n * EPL + e] = o[e];
            if (n == 0) { out[D] = m; out[D + 1] = l; }
        }
    } else {
        for (int e = lane; e < D + 2; e += 64) out[e] = e == D ? -INFINITY : 0.f;
    }
    __syncthreads();
    combine_waves<D, 1, 12>(red, 1, PartialOut(part, D, u, 1, nsplit, rule.units), 0, split);
}

static int decode_splits(const zipvl_dims& d, int cap, int rows = 256) {       // at least `rows` rows per split
    const int units = d.B * d.Hkv;
    int s = (1024 + units - 1) / units;
    const int by_len = (cap + rows - 1) / rows;
    s = s < by_len ? s : by_len;
    return s < 1 ? 1 : (s > kDecMaxSplit ? kDecMaxSplit : s);
}

// Partial states that the smallest workspace of a cache of `cap` rows holds per head.
static int least_splits(const zipvl_dims& d, int cap) {
    const int per = std::max(256, ((cap + 15) / 16 + 15) / 16 * 16);
    return std::max(decode_splits(d, cap), (cap + per - 1) / per);
}

// Finer splits, of 128 rows (fp32 of few heads 64), where splits of 256 leave the chip idle.
//
// One head: a tile less in a split saves 0.37 us, a workgroup more costs some 10 ns, idle ones too, for those whose units share a line of
// arrival counters, kLineUnits of them.  So a line has at most kMostMore more, a unit takes the finer splits from the tiles on where that pays
// (finer_from), and they are launched at all where caches from seven tenths of the capacity on take them (from 85 % where they put two workgroups on
// every CU: full caches, seven tenths -> so, 32 heads, cap 3461 137.8 -> 132.1, 2 x 32, cap 1700 134.3 -> 127.2, and as before at 25 and 60 %); up to kFewMore more cost nothing
// from some 30 rows on.  us a step of 8 layers, splits of 256 rows -> so, cache full, at 60 %, at 12 %: 8 heads, d = 128, cap 2700 98 -> 85, 81 -> 75, 57 -> 57; 32 heads,
// cap 1300 92 -> 88, 78 -> 77, 56 -> 57; 32 heads, cap 2700 140 -> 130, 92 -> 92, 68 -> 69; 4 heads, cap 5500 98 -> 87, 82 -> 78; fp32, d = 64, 8 heads, cap 1300
// 85 -> 71, 67 -> 60.  Finer splits at every length, without the line, and the idle workgroups dispatched before busy ones: 8 heads, cap 5500, full, 25 %, 12 %
// 106 -> 103, 73 -> 85, 65 -> 79; fp32, 64 rows, 8 heads, cap 2700, 25 % 58 -> 77.  Past the lines: 16 heads, cap 5500, fp32 183 -> 187;
// near them 16 heads, d = 64, cap 2700, full, 60 %, 4 % 101 -> 98, 84 -> 87, 54 -> 58.
// Limits of a launch whatever its units, of a line, finer at every length, us: 4 x 40 heads, cap 482, 32 % full 75.5, 68.3, 68.3; 4 layers of 4 x 14, fp32, cap 1015, 53 % 51.2, 46.5, 45.5;
// 4 x 32, fp32, d = 64, cap 561, 38 % 73.6, 68.3, 68.1; 4 x 8, cap 1562, 59 % 84.8, 85.6, 80.7.  Twice kMostMore makes steps 5 to 8 % slower a quarter full (8 heads, cap 5500 64.6 -> 69.2).
//
// Groups: bf16 at d = 128 above kFineGroups splits, where all forms of the step merge them in a launch of their own, up to a workgroup a CU.  us, 16 layers,
// full, 25 % full: 28 on 4, cap 7000 176 -> 171; 14 on 2, cap 7000 175 -> 156; 8 of them over quantised caches, 28 on 4, cap 7000 95 -> 79, 67 -> 70,
// cap 10 500 99 -> 91, 68 -> 70, 14 on 2, cap 7000 93 -> 77, 66 -> 68, cap 13 000 and more alike.  At kFineGroups, steps of 28 on 4: cap 6100 175 -> 166, 6200 175 -> 168.
// It is not the line where the gain ends (8 on 2, cap 700 139 -> 117; 28 on 4, cap 4110 176 -> 155; fp32, cap 2300 240 -> 173, but 32 on 8, cap 6200
// 306 -> 311; d = 64, 32 on 8, cap 2300 138 -> 140): below it the tests of the merge count the states that a step leaves by splits of 256 rows.
constexpr int kFewMore = 32, kMostMore = 96;                 // workgroups of kLineUnits units
constexpr int kLineUnits = 32;
constexpr int kFineGroups = 24;                              // splits of 256 rows

// Tiles of a unit from which it has `fine` splits and not `coarse` ones.
static int finer_from(const zipvl_dims& d, int coarse, int fine) {
    const int line = std::min(d.B * d.Hkv, kLineUnits);
    return d.Hq > d.Hkv || line * (fine - coarse) <= kFewMore ? 0 : ((line + 4) * coarse * fine + 47) / 48;
}

// Partial states that a call makes use of.
static int useful_splits(const zipvl_dims& d, int cap) {
    const bool groups = d.Hq > d.Hkv, bf16 = d.dtype == ZIPVL_BF16;
    const int units = d.B * d.Hkv, line = std::min(units, kLineUnits), coarse = least_splits(d, cap);
    if (groups) {
        if (!bf16 || d.d == 64 || decode_splits(d, cap) <= kFineGroups) return coarse;
        return std::max(coarse, std::min(decode_splits(d, cap, 128), 256 / units));
    }
    if (!bf16) {
        const int fine = std::min(decode_splits(d, cap, 64), 512 / units);
        if (line * (fine - coarse) <= kFewMore) return std::max(coarse, fine);
    }
    const int fine = std::min({decode_splits(d, cap, 128), 512 / units, coarse + kMostMore / line});
    const bool even = fine == 512 / units && units * fine > 480;                // two workgroups on every CU
    return fine > coarse && 20 * (int64_t)finer_from(d, coarse, fine) <= (even ? 17 : 14) * (((int64_t)cap + kDecTile - 1) / kDecTile) ? fine : coarse;
}
static size_t state_bytes(const zipvl_dims& d) { return (size_t)d.B * d.Hq * (d.d + 2) * sizeof(float); }       // of a split of every unit

// One head: 1024 workgroups of 4 waves (512: 151 us for four layers of 128 units, 1024: 131, 2048: 142), then 1792: seven per CU
// are resident together, and a few more would run alone at the end (four conversations of 32768 rows, 32 heads: 1024 387 us,
// 1792 382, 2048 424).  Groups: 256 of 8 waves (one per CU: 512 is 3-10 % slower from 32 units on, and as fast below), then twice.
static SplitRule split_rule(const zipvl_dims& d, int cap, size_t ws_bytes) {
    const int units = d.B * d.Hkv, room = (int)std::min<size_t>(useful_splits(d, cap), ws_bytes / state_bytes(d));
    const bool groups = d.Hq / d.Hkv > 1;
    const int tiles = groups ? kDecLongGroups : kDecLongOne, fill = ((groups ? 256 : 1024) + units - 1) / units;
    const int least = std::max(1, std::min(room, fill)), coarse = std::max(1, std::min(least_splits(d, cap), fill));
    const int most = std::min(room, 4 * least), more = std::min(most, groups ? 2 * least : std::max(least, 1792 / units));
    const int64_t longest = (int64_t)tiles * kDecTile;       // what no unit reaches is not launched
    const int launched = cap <= least * longest ? least : cap <= more * longest ? more : most;
    const int from = least > coarse ? finer_from(d, coarse, least) : 0;
    const int turn = launched > least || from ? std::max(1, (int)(units * 0.618)) : 0;     // rows of any number of units start all over the chip
    return {least, std::min(more, launched), launched, tiles, units, turn, coarse, from};
}

size_t decode_workspace_bytes(const zipvl_dims& d, int cap) { return useful_splits(d, cap) * state_bytes(d); }
size_t decode_workspace_least(const zipvl_dims& d, int cap) { return least_splits(d, cap) * state_bytes(d); }

template <typename T, int D>
static int launch_decode_t(const void* q, const void* Kc, const void* Vc, const int32_t* len, int32_t cap,
                           const zipvl_dims& d, float scale, void* o, void* ws, size_t ws_bytes, hipStream_t st)
{
    const int G = d.Hq / d.Hkv, units = d.B * d.Hkv;
    const SplitRule rule = split_rule(d, cap, ws_bytes);
    const Lengths lengths{{len, nullptr, nullptr}, {cap, 0, 0}};
    const float c = scale * kLog2e;
#define ZIPVL_DEC(GT)                                                                                \
    hipLaunchKernelGGL((decode_partial_kernel<T, D, GT>), rule.grid(), dim3(64 * kDecWaves<GT>), 0, st, \
        (const T*)q, (const T*)Kc, (const T*)Vc, len, cap, d.Hq, d.Hkv, gb, c, rule, (float*)ws)
    for (int gb = 0; gb < G; gb += 8) {
        KernelTimer tm(ZIPVL_K_DECODE_PARTIAL, st);
        if (G > 1) ZIPVL_DEC(8);
        else ZIPVL_DEC(1);
        int rc = check_launch("decode_partial");
        if (rc) return rc;
    }
#undef ZIPVL_DEC
    KernelTimer tm(ZIPVL_K_DECODE_COMBINE, st);
    // as many threads as in the fused step, which makes the two paths add the splits in the same order
    if (G > 1)
        hipLaunchKernelGGL((decode_combine_kernel<T, D, 64 * kDecWaves<8>>), dim3(units, G), dim3(64 * kDecWaves<8>), 0, st,
            (const float*)ws, lengths, rule, G, (T*)o);
    else
        hipLaunchKernelGGL((decode_combine_kernel<T, D, 64 * kDecWaves<1>>), dim3(units), dim3(64 * kDecWaves<1>), 0, st,
            (const float*)ws, lengths, rule, G, (T*)o);
    return check_launch("decode_combine");
}

template <typename T, int D>
static int launch_decode_q_t(const void* q, const zipvl_qtensor& Kq, const zipvl_qtensor& Vq, const int32_t* len_hi,
                             const int32_t* len_lo, int32_t cap_hi, int32_t cap_lo, const void* Kt, const void* Vt,
                             const int32_t* len_t, int32_t cap_t, const zipvl_dims& d, float scale, void* o, void* ws, size_t ws_bytes, hipStream_t st)
{
    const int G = d.Hq / d.Hkv, units = d.B * d.Hkv, cap = cap_hi + cap_lo + cap_t;
    // one head: as many splits as are resident together (three workgroups of four waves per CU), whatever the lengths are; each
    // takes its share of the cache (four layers of 128 units x 8192 rows: 1024 workgroups 153 us, 768 123, 512 137, 384 134)
    const SplitRule rule = G > 1 ? split_rule(d, cap, ws_bytes) : SplitRule{1, 1, std::min(decode_splits(d, cap), std::max(1, 768 / units)), 0, units, 0, 1, 0};
    Lengths lengths{{nullptr, nullptr, nullptr}, {0, 0, 0}};
    if (rule.turn) lengths = {{len_hi, len_lo, Kt ? len_t : nullptr}, {cap_hi, cap_lo, cap_t}};      // else every split reports: 0.5 us less
    const float c = scale * kLog2e;
    const QTensor kq{(const uint8_t*)Kq.hi_codes, (const uint32_t*)Kq.hi_params, (const uint8_t*)Kq.lo_codes, (const uint32_t*)Kq.lo_params};
    const QTensor vq{(const uint8_t*)Vq.hi_codes, (const uint32_t*)Vq.hi_params, (const uint8_t*)Vq.lo_codes, (const uint32_t*)Vq.lo_params};
#define ZIPVL_DECQ_ARGS (const T*)q, kq, vq, len_hi, len_lo, cap_hi, cap_lo, (const T*)Kt, (const T*)Vt, len_t, cap_t
    for (int gb = 0; gb < G; gb += 8) {
        KernelTimer tm(ZIPVL_K_DECODE_Q_PARTIAL, st);
        // one head: integer products on the codes (four layers of 128 units x 8192 rows 116 us; 152 on the vector units, 440 in
        // floating-point tiles of which one column in 16 is used); two and more: floating-point tiles (two heads, 32 units x 4000:
        // 122 us on the vector units, 100)
        if (G > 1)
            hipLaunchKernelGGL((decode_q_partial_kernel<T, D, 8>), rule.grid(), dim3(64 * kDecWaves<8>), 0, st, ZIPVL_DECQ_ARGS,
                d.Hq, d.Hkv, gb, c, (float*)ws, rule);
        else
            hipLaunchKernelGGL((decode_q1_partial_kernel<T, D>), rule.grid(), dim3(256), 0, st, ZIPVL_DECQ_ARGS, c, (float*)ws, rule);
        int rc = check_launch("decode_q_partial");
        if (rc) return rc;
    }
#undef ZIPVL_DECQ_ARGS
    KernelTimer tm(ZIPVL_K_DECODE_COMBINE, st);
    hipLaunchKernelGGL((decode_combine_kernel<T, D, 256>), dim3(units, G), dim3(256), 0, st,
        (const float*)ws, lengths, rule, G, (T*)o);
    return check_launch("decode_combine");
}

static size_t step_counter_bytes(const zipvl_dims& d) { return ((size_t)d.B * d.Hkv * sizeof(unsigned) + 255) / 256 * 256; }

size_t decode_step_workspace_bytes(const zipvl_dims& d, int cap) {
    return step_counter_bytes(d) + decode_workspace_bytes(d, cap);
}
size_t decode_step_workspace_least(const zipvl_dims& d, int cap) { return step_counter_bytes(d) + decode_workspace_least(d, cap); }

template <typename T, int D>
static int launch_decode_step_t(const void* q, void* Kc, void* Vc, int32_t* len, int32_t cap, const void* k_new,
                                const void* v_new, const zipvl_dims& d, float scale, void* o, void* ws, size_t ws_bytes, hipStream_t st)
{
    const int G = d.Hq / d.Hkv;
    unsigned* arrived = (unsigned*)ws;
    float* part = (float*)((char*)ws + step_counter_bytes(d));
    if (G > 8) {                                            // several passes over the cache per step: not fused
        int rc = launch_kv_append(Kc, Vc, len, cap, k_new, v_new, d, st);
        if (rc) return rc;
        return launch_decode_attn(q, Kc, Vc, len, cap, d, scale, o, part, ws_bytes - step_counter_bytes(d), st);
    }
    const float c = scale * kLog2e;
    const SplitRule rule = split_rule(d, cap, ws_bytes - step_counter_bytes(d));
    const bool one_launch = G == 1 || rule.most <= kMergeSplits<T, D>;
    {
        KernelTimer tm(ZIPVL_K_DECODE_STEP, st);
#define ZIPVL_STEP(GT, MERGE)                                                                        \
    hipLaunchKernelGGL((decode_step_kernel<T, D, GT, MERGE>), rule.grid(), dim3(64 * kDecWaves<GT>), 0, st, (const T*)q, (T*)Kc, (T*)Vc, len, cap, \
        (const T*)k_new, (const T*)v_new, d.Hq, d.Hkv, c, rule, part, arrived, (T*)o)
        if (G == 1) ZIPVL_STEP(1, true);
        else if (one_launch) ZIPVL_STEP(8, true);
        else ZIPVL_STEP(8, false);
#undef ZIPVL_STEP
    }
    int rc = check_launch("decode_step");
    if (rc || one_launch) return rc;
    KernelTimer tm(ZIPVL_K_DECODE_COMBINE, st);
    constexpr int kThreads = 64 * kDecWaves<8>;
    hipLaunchKernelGGL((decode_step_combine_kernel<T, D, kThreads>), dim3(d.B * d.Hkv, G), dim3(kThreads), 0, st, (const float*)part, len, cap, rule, G, (T*)o);
    return check_launch("decode_combine");
}

int launch_decode_step(const void* q, void* Kc, void* Vc, int32_t* len, int32_t cap, const void* k_new,
                       const void* v_new, const zipvl_dims& d, float scale, void* o, void* ws, size_t ws_bytes, hipStream_t st)
{
    if (d.dtype == ZIPVL_BF16) {
        if (d.d == 128) return launch_decode_step_t<__bf16, 128>(q, Kc, Vc, len, cap, k_new, v_new, d, scale, o, ws, ws_bytes, st);
        return launch_decode_step_t<__bf16, 64>(q, Kc, Vc, len, cap, k_new, v_new, d, scale, o, ws, ws_bytes, st);
    }
    if (d.d == 128) return launch_decode_step_t<float, 128>(q, Kc, Vc, len, cap, k_new, v_new, d, scale, o, ws, ws_bytes, st);
    return launch_decode_step_t<float, 64>(q, Kc, Vc, len, cap, k_new, v_new, d, scale, o, ws, ws_bytes, st);
}

int launch_decode_attn_q(const void* q, const zipvl_qtensor& Kq, const zipvl_qtensor& Vq, const int32_t* len_hi,
                         const int32_t* len_lo, int32_t cap_hi, int32_t cap_lo, const void* Kt, const void* Vt,
                         const int32_t* len_t, int32_t cap_t, const zipvl_dims& d, float scale, void* o, void* ws, size_t ws_bytes, hipStream_t st)
{
#define ZIPVL_ARGS q, Kq, Vq, len_hi, len_lo, cap_hi, cap_lo, Kt, Vt, len_t, cap_t, d, scale, o, ws, ws_bytes, st
    if (d.dtype == ZIPVL_BF16) {
        if (d.d == 128) return launch_decode_q_t<__bf16, 128>(ZIPVL_ARGS);
        return launch_decode_q_t<__bf16, 64>(ZIPVL_ARGS);
    }
    if (d.d == 128) return launch_decode_q_t<float, 128>(ZIPVL_ARGS);
    return launch_decode_q_t<float, 64>(ZIPVL_ARGS);
#undef ZIPVL_ARGS
}

// ---------------------------------------------------------------- decode attention without a caller workspace
// The partial states of the split-KV kernels live in a fixed device array of this library instead of a
// workspace argument, for callers that cannot allocate.  Every GPU holds its own copy of the array at its
// own address: the address is looked up once per device (with that device current) and only that pointer
// is ever handed to kernels.  Nothing in the array has to start at zero: every (unit, head, split) slot is
// written by the partial kernel before the combine kernel of the same call reads it.
constexpr size_t kStaticScratchBytes = ZIPVL_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

static int static_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return set_error(ZIPVL_EHIP, "decode_attn_static: hipGetDevice failed: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return set_error(ZIPVL_EUNSUPPORTED, "decode_attn_static: device ordinal %d is beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return set_error(ZIPVL_EHIP, "decode_attn_static: no device address for the scratch array: %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return ZIPVL_OK;
}

int launch_decode_attn_static(const void* q, const void* Kc, const void* Vc, const int32_t* len, int32_t cap,
                              const zipvl_dims& d, float scale, void* o, hipStream_t st)
{
    const size_t need = decode_workspace_least(d, cap);
    if (need > kStaticScratchBytes)
        return set_error(ZIPVL_ESHAPE, "decode_attn_static: these dims need %zu bytes of partial states, the built-in scratch holds %zu "
                                       "(use zipvl_decode_attn with a workspace)", need, kStaticScratchBytes);
    void* ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc) return rc;
    return launch_decode_attn(q, Kc, Vc, len, cap, d, scale, o, ws, kStaticScratchBytes, st);
}

int launch_decode_attn(const void* q, const void* Kc, const void* Vc, const int32_t* len, int32_t cap,
                       const zipvl_dims& d, float scale, void* o, void* ws, size_t ws_bytes, hipStream_t st)
{
    if (d.dtype == ZIPVL_BF16) {
        if (d.d == 128) return launch_decode_t<__bf16, 128>(q, Kc, Vc, len, cap, d, scale, o, ws, ws_bytes, st);
        return launch_decode_t<__bf16, 64>(q, Kc, Vc, len, cap, d, scale, o, ws, ws_bytes, st);
    }
    if (d.d == 128) return launch_decode_t<float, 128>(q, Kc, Vc, len, cap, d, scale, o, ws, ws_bytes, st);
    return launch_decode_t<float, 64>(q, Kc, Vc, len, cap, d, scale, o, ws, ws_bytes, st);
}

}  // namespace zipvl
