// Shared device-side helpers for the gfx950 kernels (64-wide wavefronts, MFMA).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "zipvl.h"
#include "zipvl_bench.h"

namespace zipvl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;

int set_error(int code, const char* fmt, ...);
int check_launch(const char* what);

// One 16-byte operand fragment per lane.  A 32x32 MFMA tile is fed by 64 lanes:
// lane = (row or column index i = lane % 32, half h = lane / 32).
//   bf16: the fragment holds 8 consecutive elements  [16*c + 8*h, +8)  of row i
//         and feeds one v_mfma_f32_32x32x16_bf16.
//   fp32: the fragment holds 4 consecutive elements  [8*c + 4*h, +4)   of row i
//         and feeds four v_mfma_f32_32x32x2_f32 (element t in step t).  The
//         contraction order is permuted the same way for both operands, which
//         leaves the sum unchanged.
template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int kBytes = 4;
    static constexpr int kPerFrag = 4;     // elements per 16-byte fragment
    static constexpr int kPerChunk = 8;    // contraction elements covered by the two halves
};
template <> struct Elem<__bf16> {
    static constexpr int kBytes = 2;
    static constexpr int kPerFrag = 8;
    static constexpr int kPerChunk = 16;
};

template <typename T>
__device__ __forceinline__ floatx16 mma_frag(const uintx4& a, const uintx4& b, floatx16 acc);

template <>
__device__ __forceinline__ floatx16 mma_frag<__bf16>(const uintx4& a, const uintx4& b, floatx16 acc) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ floatx16 mma_frag<float>(const uintx4& a, const uintx4& b, floatx16 acc) {
    floatx4 fa = __builtin_bit_cast(floatx4, a);
    floatx4 fb = __builtin_bit_cast(floatx4, b);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[0], fb[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[1], fb[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[2], fb[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[3], fb[3], acc, 0, 0, 0);
    return acc;
}

// Row of the 32x32 accumulator held in register r of a lane with half h.
__device__ __forceinline__ int acc_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ uintx4 load16(const void* p) { return *reinterpret_cast<const uintx4*>(p); }
__device__ __forceinline__ void store16(void* p, const uintx4& v) { *reinterpret_cast<uintx4*>(p) = v; }

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    floatx2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// acc + lo + hi of a packed bf16 pair (the values as rounded to bf16, accumulated in fp32)
__device__ __forceinline__ float add_bf16x2(uint32_t packed, float acc) {
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, packed), ones, acc, false);
}

// Over the wave by lane permutes in registers (a shuffle through LDS takes some 100 clocks a step): shifts inside rows of 16
// lanes, then across the rows; the last lane has it all.
template <int CTRL, int ROWS>
__device__ __forceinline__ float lane_moved(float v, float none) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(none), __float_as_int(v), CTRL, ROWS, 0xF, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int lane_moved(int v, int none) { return __builtin_amdgcn_update_dpp(none, v, CTRL, ROWS, 0xF, false); }
template <int CTRL, int ROWS>
__device__ __forceinline__ double lane_moved(double v, double none) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(__double2hiint(none), __double2hiint(v), CTRL, ROWS, 0xF, false),
                            __builtin_amdgcn_update_dpp(__double2loint(none), __double2loint(v), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ int last_lane(int v) { return __builtin_amdgcn_readlane(v, 63); }
__device__ __forceinline__ float last_lane(float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63)); }
__device__ __forceinline__ double last_lane(double v) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63), __builtin_amdgcn_readlane(__double2loint(v), 63));
}
template <typename N, typename F>
__device__ __forceinline__ N wave_reduce(N v, N none, F&& f) {
    v = f(v, lane_moved<0x111, 0xF>(v, none));
    v = f(v, lane_moved<0x112, 0xF>(v, none));
    v = f(v, lane_moved<0x114, 0xF>(v, none));
    v = f(v, lane_moved<0x118, 0xF>(v, none));
    v = f(v, lane_moved<0x142, 0xA>(v, none));
    v = f(v, lane_moved<0x143, 0xC>(v, none));
    return last_lane(v);
}
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, -INFINITY, [](float a, float b) { return fmaxf(a, b); }); }
template <typename N>
__device__ __forceinline__ N wave_sum(N v) { return wave_reduce(v, N(0), [](N a, N b) { return a + b; }); }

// n / d of whole numbers below 2^31, inv = inverse(d) from the host: the high half of the product is the quotient or one less.  The compiler's own division by
// a number it does not know is some 20 dependent vector instructions, and a workgroup needs five of them to know its place: 0.8 us, 0.3 so.  Attention with
// its set and cache, us: d = 64, 3 x 40 heads, n = 8000, a fifth kept 107.0 -> 104.1, 4 x 32, n = 4000, a third 115.2 -> 113.5, long tiles as before.
static uint32_t inverse(int d) { return d == 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (uint32_t)d); }
__device__ __forceinline__ int divided(int n, int d, uint32_t inv) {
    const uint32_t q = (uint32_t)((uint64_t)(uint32_t)n * inv >> 32);
    return (int)(q + ((uint32_t)n - q * d >= (uint32_t)d));
}

}  // namespace zipvl
