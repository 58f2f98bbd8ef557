// KV-cache eviction (Section 4.2; Algorithm 1, cache step) and the cache append
// of the decode phase (Eq. (4); Algorithm 2).  Pure data movement: every row
// is d*e contiguous bytes and moves as 16-byte vectors, 16 (or 8/32) lanes per
// row, so both the gathered reads and the packed writes are full-line accesses.
#include "launch.h"

namespace zipvl {

constexpr int kCompactRows = 64;   // kept rows handled by one workgroup

// CPR = 16-byte chunks per row.  A workgroup's life is a chain of two round trips to memory, positions -> rows: all of its
// positions, then all of its rows are requested at once.  With one pass of 256 threads after the other, the same call again
// and again, 32 units x 970 of 2933 rows of 256 bytes took 6.9 us (6.1 so), 128 x 2048 of 8192 49.7 (46.2: 5.8 TB/s), 4 x 69 of 576 3.5
// (2.7); inside a layer, where the rows come from memory, 9.7 (10.2; shortest 8.4 and 7.8), 54.1 (53.9) and 3.8 (3.2).
template <int CPR>
__global__ __launch_bounds__(256) void compact_kv_kernel(
    const char* __restrict__ K, const char* __restrict__ V,
    int64_t kb_stride, int64_t kh_stride, int64_t kt_stride,     // bytes
    int64_t vb_stride, int64_t vh_stride, int64_t vt_stride,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ kcnt,
    char* __restrict__ Kc, char* __restrict__ Vc, int32_t* __restrict__ len,
    int n, int Hkv, int cap, int t_per_batch)
{
    constexpr int row_bytes = CPR * 16, kPass = 256 / CPR, kPasses = kCompactRows / kPass;
    const int u = blockIdx.y;
    const int b = u / Hkv, g = u - b * Hkv;
    const int ut = t_per_batch ? b : u;                   // row of idx / k that holds this unit's T
    int kk = kcnt ? kcnt[ut] : n;
    kk = max(0, min(min(kk, n), cap));
    if (blockIdx.x == 0 && threadIdx.x == 0) len[u] = kk;
    const int r0 = blockIdx.x * kCompactRows;
    if (r0 >= kk) return;
    const int c = (threadIdx.x % CPR) * 16, r1 = r0 + threadIdx.x / CPR;
    const char* Kb = K + b * kb_stride + g * kh_stride + c;
    const char* Vb = V + b * vb_stride + g * vh_stride + c;
    int src[kPasses];                                     // rows past the last are read from it and not stored
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
        const int r = min(r1 + p * kPass, kk - 1);
        src[p] = idx ? idx[(int64_t)ut * n + r] : r;
    }
    uintx4 kr[kPasses], vr[kPasses];
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
        kr[p] = load16(Kb + (int64_t)src[p] * kt_stride);
        vr[p] = load16(Vb + (int64_t)src[p] * vt_stride);
    }
    const int64_t out = ((int64_t)u * cap + r1) * row_bytes + c;
#pragma unroll
    for (int p = 0; p < kPasses; ++p)
        if (r1 + p * kPass < kk) {
            store16(Kc + out + p * kPass * row_bytes, kr[p]);
            store16(Vc + out + p * kPass * row_bytes, vr[p]);
        }
}

__global__ __launch_bounds__(64) void kv_append_kernel(
    char* __restrict__ Kc, char* __restrict__ Vc, int32_t* __restrict__ len, int cap,
    const char* __restrict__ k_new, const char* __restrict__ v_new, int row_bytes)
{
    const int u = blockIdx.x;
    const int L = len[u];
    if (L < 0 || L >= cap) return;
    const int cpr = row_bytes >> 4;
    const int64_t o = ((int64_t)u * cap + L) * row_bytes;
    for (int c = threadIdx.x; c < cpr; c += 64) {
        store16(Kc + o + c * 16, load16(k_new + (int64_t)u * row_bytes + c * 16));
        store16(Vc + o + c * 16, load16(v_new + (int64_t)u * row_bytes + c * 16));
    }
    __syncthreads();                 // every lane has read len[u] before it changes
    if (threadIdx.x == 0) len[u] = L + 1;
}

int launch_compact_kv(const void* K, const void* V, const zipvl_dims& d, const int32_t* idx,
                      const int32_t* k, void* Kc, void* Vc, int32_t cap, int32_t* len, int flags, hipStream_t st)
{
    const int e = d.dtype == ZIPVL_BF16 ? 2 : 4;
    const int units = d.B * d.Hkv;
    dim3 grid((min(d.n, cap) + kCompactRows - 1) / kCompactRows, units);
    KernelTimer tm(ZIPVL_K_COMPACT_KV, st);
#define ZIPVL_COMPACT(CPR)                                                                          \
    hipLaunchKernelGGL((compact_kv_kernel<CPR>), grid, dim3(256), 0, st, (const char*)K, (const char*)V, \
        d.k_strides[0] * e, d.k_strides[1] * e, d.k_strides[2] * e,                                 \
        d.v_strides[0] * e, d.v_strides[1] * e, d.v_strides[2] * e,                                 \
        idx, k, (char*)Kc, (char*)Vc, len, d.n, d.Hkv, cap, (flags & ZIPVL_T_PER_BATCH) ? 1 : 0)
    if (d.d * e == 128) ZIPVL_COMPACT(8);
    else if (d.d * e == 256) ZIPVL_COMPACT(16);
    else ZIPVL_COMPACT(32);                               // d is 64 or 128
#undef ZIPVL_COMPACT
    return check_launch("compact_kv");
}

int launch_kv_append(void* Kc, void* Vc, int32_t* len, int32_t cap, const void* k_new,
                     const void* v_new, const zipvl_dims& d, hipStream_t st)
{
    const int e = d.dtype == ZIPVL_BF16 ? 2 : 4;
    KernelTimer tm(ZIPVL_K_KV_APPEND, st);
    hipLaunchKernelGGL(kv_append_kernel, dim3(d.B * d.Hkv), dim3(64), 0, st,
        (char*)Kc, (char*)Vc, len, cap, (const char*)k_new, (const char*)v_new, d.d * e);
    return check_launch("kv_append");
}

}  // namespace zipvl
