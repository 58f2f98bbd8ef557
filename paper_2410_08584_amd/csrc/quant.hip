// Mixed-precision KV cache keyed by the important set (Section 5.3.1: important
// tokens at 4 bits, the others at 2 bits).  The quantiser the paper leaves open
// is taken as uniform asymmetric per row (one token of one KV head) with an
// fp16 (scale, zero) pair:
//   zero = fp16(min), scale = fp16((max - min) * fp32(1 / (2^bits - 1))),
//   code = clamp(rint((x - zero) / scale), 0, 2^bits - 1)   (0 when scale = 0), all in fp32.
// Two kernels.  `kept_masks` turns T (in any order) into a bit per token and, for every 64 tokens, the number of kept ones before them: a token's
// row in the 4-bit group (rank among the kept tokens) or in the 2-bit group (rank among the others, Eq. (10)).  `quantize_rows`: a
// workgroup takes 64 tokens, 8 lanes per row, each with 8 (d = 64) or 2 x 8 (d = 128) of its elements.
#include <type_traits>

#include "launch.h"

namespace zipvl {

constexpr int kQuantMaxTokens = 262144;      // the bits of a set fit 32 KB of LDS
constexpr int kSetThreads = 1024;
constexpr int kQuantRows = 64;               // rows per workgroup: a bit each of a 64-bit mask
constexpr int kLanes = 8, kPass = 256 / kLanes, kPasses = kQuantRows / kPass;      // lanes per row, rows per pass

// Of one set, in its n words of the workspace: a bit per token (words 0 ... W - 1, W = ceil(n / 32)), then the number of kept tokens before
// token 64 x for x = 1, 2, ...  Positions outside [0, n) are passed over, a position that comes twice counts once.
// Latency: the count, the positions, the bits in LDS, their sums; 1.5 to 5 us of a call (4 sets of 60 000 positions 22).  A bisection of T by every wave
// of quantize_rows takes no launch, and gives two tokens one row wherever T does not ascend.
__global__ __launch_bounds__(kSetThreads) void kept_masks_kernel(const int32_t* __restrict__ idx, const int32_t* __restrict__ kcnt, int n,
                                                                 uint32_t* __restrict__ masks)
{
    extern __shared__ uint32_t words[];
    __shared__ int wave_total[kSetThreads / 64];
    const int set = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int blocks = (n + 63) >> 6, W = (n + 31) >> 5;
    const int32_t* T = idx + (int64_t)set * n;
    uint32_t* out = masks + (int64_t)set * n;
    const int kk = max(0, min(kcnt[set], n));
    for (int i = tid; i < 2 * blocks; i += kSetThreads) words[i] = 0;
    __syncthreads();
    constexpr int kAhead = 4;                                // positions of a thread on the way at once
    for (int i0 = tid; i0 < kk; i0 += kAhead * kSetThreads) {
        int t[kAhead];
#pragma unroll
        for (int a = 0; a < kAhead; ++a) t[a] = T[min(i0 + a * kSetThreads, kk - 1)];
#pragma unroll
        for (int a = 0; a < kAhead; ++a)
            if (i0 + a * kSetThreads < kk && (unsigned)t[a] < (unsigned)n) atomicOr(&words[t[a] >> 5], 1u << (t[a] & 31));
    }
    __syncthreads();
    for (int i = tid; i < W; i += kSetThreads) out[i] = words[i];
    // every thread has a run of blocks: their sum, the sums before it in the wave, the waves before
    const int per = (blocks + kSetThreads - 1) / kSetThreads, x0 = min(tid * per, blocks), x1 = min(x0 + per, blocks);
    auto count = [&](int x) { return __popc(words[2 * x]) + __popc(words[2 * x + 1]); };
    int mine = 0;
    for (int x = x0; x < x1; ++x) mine += count(x);
    int upto = mine;
    upto += lane_moved<0x111, 0xF>(upto, 0);
    upto += lane_moved<0x112, 0xF>(upto, 0);
    upto += lane_moved<0x114, 0xF>(upto, 0);
    upto += lane_moved<0x118, 0xF>(upto, 0);
    upto += lane_moved<0x142, 0xA>(upto, 0);
    upto += lane_moved<0x143, 0xC>(upto, 0);
    if (lane == 63) wave_total[w] = upto;
    __syncthreads();
    if (x0 == x1) return;
    int before = upto - mine;
    for (int x = 0; x < w; ++x) before += wave_total[x];
    for (int x = x0; x < x1; ++x) {
        if (x) out[W + x - 1] = before;
        before += count(x);
    }
}

// Minimum and maximum over the 8 lanes of a row, of a row of K and one of V at a time, result in all of them.  One instruction a step
// and value, where the compiler takes three (a lane permute, a quieting, the minimum); a lane permute may not read what the two
// instructions before it wrote, and here three others always lie between.
__device__ __forceinline__ void row8_extremes(float& klo, float& khi, float& vlo, float& vhi) {
#define ZIPVL_STEP(CTRL)                                                            \
    "v_min_f32_dpp %0, %0, %0 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
    "v_max_f32_dpp %1, %1, %1 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
    "v_min_f32_dpp %2, %2, %2 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
    "v_max_f32_dpp %3, %3, %3 " CTRL " row_mask:0xf bank_mask:0xf\n\t"
    asm("s_nop 1\n\t" ZIPVL_STEP("quad_perm:[1,0,3,2]") ZIPVL_STEP("quad_perm:[2,3,0,1]") ZIPVL_STEP("row_half_mirror")
        : "+v"(klo), "+v"(khi), "+v"(vlo), "+v"(vhi));
#undef ZIPVL_STEP
}

// 8 elements of a row as loaded
template <typename T> struct RawPiece;
template <> struct RawPiece<__bf16> {
    uintx4 v;
    __device__ __forceinline__ void load(const __bf16* p) { v = load16(p); }
    __device__ __forceinline__ float operator[](int e) const { return __uint_as_float(e & 1 ? v[e >> 1] & 0xFFFF0000u : v[e >> 1] << 16); }
};
template <> struct RawPiece<float> {
    floatx4 v[2];
    __device__ __forceinline__ void load(const float* p) { v[0] = *reinterpret_cast<const floatx4*>(p); v[1] = *reinterpret_cast<const floatx4*>(p + 4); }
    __device__ __forceinline__ float operator[](int e) const { return v[e >> 2][e & 3]; }
};

// Codes (8 to a word) and parameters of one row, P pieces of 8 elements in each of its lanes, lo and hi its extremes, at 4 or 2
// bits, chosen per row: one instruction stream serves the rows of both widths that share a wave.
// The code is rint of the correctly rounded (x - zero) / scale, clamped.  One correction of the product with a reciprocal gives that
// quotient: the remainder it takes is exact, and as scale has 11 bits no quotient lies closer than 2^-12 of its last place to the
// middle of two floats, where what is left of the error (2^-22 of a last place) could turn the rounding.  bf16 rows meet exact halves in every fifth
// wave step, so that a division only near them, as it was, took a fifth of the instructions.  The products of the row's extremes
// say whether a code needs the clamp; only then, or where an element is not a number, divisions and clamps are taken.
// Four codes are put together by fused multiply-adds (below 2^16: exact).
template <typename T, int P>
__device__ __forceinline__ void quantize_chunk(const RawPiece<T> (&x)[P], float lo, float hi, bool wide, uint32_t (&word)[P], uint32_t& params) {
    const float qmax = wide ? 15.f : 3.f, base = wide ? 16.f : 4.f;
    const int bits = wide ? 4 : 2;
    const _Float16 zero_h = (_Float16)lo;
    float step = (hi - lo) * (wide ? (float)(1.0 / 15.0) : (float)(1.0 / 3.0));
    asm volatile("" : "+v"(step));            // the product is rounded to fp32 first: no fused multiply-convert
    const _Float16 scale_h = (_Float16)step;
    const float zero = (float)zero_h, scale = (float)scale_h;
    const float inv = scale > 0.f ? __builtin_amdgcn_rcpf(scale) : 0.f;
    float sum = 0.f;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        float four[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
#pragma unroll
            for (int e = 3; e >= 0; --e) {
                const float d = x[p][4 * f + e] - zero, t = d * inv, q = __builtin_rintf(fmaf(fmaf(-t, scale, d), inv, t));
                four[f] = e == 3 ? q : fmaf(four[f], base, q);
            }
            sum += four[f];
        }
        word[p] = ((uint32_t)four[1] << (4 * bits)) | (uint32_t)four[0];
    }
    const bool plain = ((lo - zero) * inv >= -0.499f) & ((hi - zero) * inv <= qmax + 0.499f) & (sum >= 0.f);
    if (__any(!plain)) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            word[p] = 0;
#pragma unroll
            for (int e = 7; e >= 0; --e) {
                float t = scale > 0.f ? (x[p][e] - zero) / scale : 0.f;
                t = fminf(fmaxf(__builtin_rintf(t), 0.f), qmax);
                word[p] = (word[p] << bits) | (uint32_t)t;
            }
        }
    }
    params = (uint32_t)__builtin_bit_cast(uint16_t, scale_h) | ((uint32_t)__builtin_bit_cast(uint16_t, zero_h) << 16);
}

template <typename T, int P>
__device__ __forceinline__ void chunk_extremes(const RawPiece<T> (&x)[P], float& lo, float& hi) {
    lo = hi = x[0][0];
#pragma unroll
    for (int e = 1; e < 8 * P; ++e) { lo = fminf(lo, x[e >> 3][e & 7]); hi = fmaxf(hi, x[e >> 3][e & 7]); }
}

struct QTensorOut {
    uint8_t* hi_codes; uint32_t* hi_params;
    uint8_t* lo_codes; uint32_t* lo_params;
};

// Bound by memory and vector instructions alike: 630 MB at 128 units x 8192 rows of 256 bytes.  us a call (with kept_masks), 16 lanes a row, a
// division near every half and a launch before that wrote every token's row -> now: that shape 154 -> 131, 4 x 18432 23.4 -> 16.5,
// 32 x 2933 24.2 -> 15.9; d = 64, 64 x 9000 53.7 -> 37.4; fp32, 40 x 4097 34.7 -> 31.8.
template <typename T, int D>
__global__ __launch_bounds__(256) void quantize_rows_kernel(
    const T* __restrict__ K, const T* __restrict__ V,
    int64_t ks0, int64_t ks1, int64_t ks2, int64_t vs0, int64_t vs1, int64_t vs2,
    const uint32_t* __restrict__ masks, const int32_t* __restrict__ kcnt,
    QTensorOut Kq, QTensorOut Vq, int cap_hi, int cap_lo, int32_t* __restrict__ len_hi, int32_t* __restrict__ len_lo,
    int n, int Hkv, int t_per_batch)
{
    constexpr int P = D / 64;
    const int u = blockIdx.y, b = u / Hkv, g = u - b * Hkv;
    const int ut = t_per_batch ? b : u;
    const int tid = threadIdx.x, sub = tid % kLanes, rl = tid / kLanes;
    int kk = kcnt ? kcnt[ut] : n;
    kk = max(0, min(kk, n));
    if (blockIdx.x == 0 && tid == 0) {
        len_hi[u] = min(kk, cap_hi);
        len_lo[u] = min(n - kk, cap_lo);
    }
    const int j0 = blockIdx.x * kQuantRows, left = n - 1 - j0;
    // All rows of the workgroup are requested at once.  Rows past the end are loaded from the last one and dropped.
    const T* Kb = K + b * ks0 + g * ks1 + (int64_t)j0 * ks2;
    const T* Vb = V + b * vs0 + g * vs1 + (int64_t)j0 * vs2;
    const T* kl = Kb + rl * ks2;
    const T* vl = Vb + rl * vs2;
    RawPiece<T> kr[kPasses][P], vr[kPasses][P];
    auto request = [&](auto whole) {
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const int r = min(rl + kPass * p, left);
            const T* kp = whole ? kl + kPass * p * ks2 : Kb + r * ks2;
            const T* vp = whole ? vl + kPass * p * vs2 : Vb + r * vs2;
#pragma unroll
            for (int c = 0; c < P; ++c) {
                kr[p][c].load(kp + 64 * c + 8 * sub);
                vr[p][c].load(vp + 64 * c + 8 * sub);
            }
        }
    };
    if (left >= kQuantRows - 1) request(std::true_type{});
    else request(std::false_type{});
    // which of the workgroup's tokens are kept, and how many before them (without T all are)
    uint64_t mask = ~0ull;
    int before = j0;
    if (masks) {
        const uint32_t* of_set = masks + (int64_t)ut * n;
        const int x = blockIdx.x, W = (n + 31) >> 5;
        mask = of_set[2 * x];
        if (2 * x + 1 < W) mask |= (uint64_t)of_set[2 * x + 1] << 32;
        before = x ? of_set[W + x - 1] : 0;
    }
    // of this unit: a row's offset in bytes fits 32 bits
    const int64_t hi0 = (int64_t)u * cap_hi, lo0 = (int64_t)u * cap_lo;
    auto put = [](auto* first, unsigned bytes, auto v) {
        *reinterpret_cast<decltype(v)*>(reinterpret_cast<char*>(first) + bytes) = v;
    };
    const uint64_t mine = mask >> rl;                                   // bit kPass p: this lane's row of pass p
    int kept_before = before + __popcll(mask & ((1ull << rl) - 1));
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
        const int r = rl + kPass * p;
        const bool wide = (uint32_t)(mine >> (kPass * p)) & 1u;
        const unsigned i = wide ? kept_before : j0 + r - kept_before;
        kept_before += __popc((uint32_t)(mine >> (kPass * p)));
        float klo, khi, vlo, vhi;
        chunk_extremes(kr[p], klo, khi);
        chunk_extremes(vr[p], vlo, vhi);
        row8_extremes(klo, khi, vlo, vhi);
        uint32_t kp, vp, kw[P], vw[P];
        quantize_chunk(kr[p], klo, khi, wide, kw, kp);
        quantize_chunk(vr[p], vlo, vhi, wide, vw, vp);
        if (r <= left) {
            if (wide) {
                if (i < (unsigned)cap_hi) {
                    const unsigned at = i * (D / 2) + sub * 4;
#pragma unroll
                    for (int c = 0; c < P; ++c) {
                        put(Kq.hi_codes + hi0 * (D / 2), at + 32 * c, kw[c]);
                        put(Vq.hi_codes + hi0 * (D / 2), at + 32 * c, vw[c]);
                    }
                    if (sub == 0) { put(Kq.hi_params + hi0, i * 4, kp); put(Vq.hi_params + hi0, i * 4, vp); }
                }
            } else if (i < (unsigned)cap_lo) {
                const unsigned at = i * (D / 4) + sub * 2;
#pragma unroll
                for (int c = 0; c < P; ++c) {
                    put(Kq.lo_codes + lo0 * (D / 4), at + 16 * c, (uint16_t)kw[c]);
                    put(Vq.lo_codes + lo0 * (D / 4), at + 16 * c, (uint16_t)vw[c]);
                }
                if (sub == 0) { put(Kq.lo_params + lo0, i * 4, kp); put(Vq.lo_params + lo0, i * 4, vp); }
            }
        }
    }
}
static_assert(kPass == 32, "a pass takes one half of the mask");

size_t quantize_workspace_bytes(const zipvl_dims& d) { return (size_t)d.B * d.Hkv * d.n * sizeof(int32_t); }

template <typename T, int D>
static int launch_quantize_t(const void* K, const void* V, const zipvl_dims& d, const int32_t* idx, const int32_t* k,
                             const zipvl_qtensor& Kq, const zipvl_qtensor& Vq, int32_t cap_hi, int32_t cap_lo,
                             int32_t* len_hi, int32_t* len_lo, int flags, void* ws, hipStream_t st)
{
    const int units = d.B * d.Hkv;
    const int t_per_batch = (flags & ZIPVL_T_PER_BATCH) ? 1 : 0;
    const QTensorOut kq{(uint8_t*)Kq.hi_codes, (uint32_t*)Kq.hi_params, (uint8_t*)Kq.lo_codes, (uint32_t*)Kq.lo_params};
    const QTensorOut vq{(uint8_t*)Vq.hi_codes, (uint32_t*)Vq.hi_params, (uint8_t*)Vq.lo_codes, (uint32_t*)Vq.lo_params};
    uint32_t* masks = idx ? (uint32_t*)ws : nullptr;
    if (masks) {
        {
            KernelTimer tm(ZIPVL_K_TOKEN_SLOTS, st);
            hipLaunchKernelGGL(kept_masks_kernel, dim3(t_per_batch ? d.B : units), dim3(kSetThreads), (d.n + 63) / 64 * 8, st, idx, k, d.n, masks);
        }
        const int rc = check_launch("kept_masks");
        if (rc) return rc;
    }
    KernelTimer tm(ZIPVL_K_QUANTIZE_ROWS, st);
    hipLaunchKernelGGL((quantize_rows_kernel<T, D>), dim3((d.n + kQuantRows - 1) / kQuantRows, units), dim3(256), 0, st,
        (const T*)K, (const T*)V, d.k_strides[0], d.k_strides[1], d.k_strides[2],
        d.v_strides[0], d.v_strides[1], d.v_strides[2], masks, k, kq, vq, cap_hi, cap_lo, len_hi, len_lo,
        d.n, d.Hkv, t_per_batch);
    return check_launch("quantize_rows");
}

int launch_quantize_kv(const void* K, const void* V, const zipvl_dims& d, const int32_t* idx, const int32_t* k,
                       const zipvl_qtensor& Kq, const zipvl_qtensor& Vq, int32_t cap_hi, int32_t cap_lo,
                       int32_t* len_hi, int32_t* len_lo, int flags, void* ws, hipStream_t st)
{
    if (d.n > kQuantMaxTokens) return set_error(ZIPVL_ESHAPE, "quantize_kv: n = %d exceeds %d", d.n, kQuantMaxTokens);
#define ZIPVL_ARGS K, V, d, idx, k, Kq, Vq, cap_hi, cap_lo, len_hi, len_lo, flags, ws, st
    if (d.dtype == ZIPVL_BF16) {
        if (d.d == 128) return launch_quantize_t<__bf16, 128>(ZIPVL_ARGS);
        return launch_quantize_t<__bf16, 64>(ZIPVL_ARGS);
    }
    if (d.d == 128) return launch_quantize_t<float, 128>(ZIPVL_ARGS);
    return launch_quantize_t<float, 64>(ZIPVL_ARGS);
#undef ZIPVL_ARGS
}

}  // namespace zipvl
