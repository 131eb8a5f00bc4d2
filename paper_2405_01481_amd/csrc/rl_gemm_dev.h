// Device helpers shared by the GEMM kernels (rl_gemm.hip, rl_gemm_stream.hip).
#pragma once
#include "rl_common.h"

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __fp16 fp16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ half8 bf16x8_to_half8(u32x4_t w) {
    fp16x2 p0 = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u));
    fp16x2 p1 = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w[1] << 16), __uint_as_float(w[1] & 0xffff0000u));
    fp16x2 p2 = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w[2] << 16), __uint_as_float(w[2] & 0xffff0000u));
    fp16x2 p3 = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w[3] << 16), __uint_as_float(w[3] & 0xffff0000u));
    return half8{(f16_t)p0[0], (f16_t)p0[1], (f16_t)p1[0], (f16_t)p1[1], (f16_t)p2[0], (f16_t)p2[1], (f16_t)p3[0], (f16_t)p3[1]};
}

// k index into W for k index `k` of an A operand carried as fp16 pairs ([hi | lo] along K, K = 2 Kw): both
// halves multiply the same W columns.  For a plain operand Kw = K and nothing wraps.
__device__ __forceinline__ int wrap_k(int k, int Kw) { return k >= Kw ? k - Kw : k; }

// fp16 pair of a float: hi = fp16(v), lo = fp16(v - hi); hi + lo carries about 22 significant bits.
__device__ __forceinline__ void split_f16(float v, f16_t& hi, f16_t& lo) {
    hi = (f16_t)v;
    lo = (f16_t)(v - (float)hi);
}

// s_waitcnt operand: at most vm vector loads and lgkm LDS operations outstanding.
constexpr int dma_waitcnt(int vm, int lgkm) { return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | (lgkm << 8); }

// Value of the lane that a data-parallel-primitive control selects within a row of 16 lanes.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// The value as rounded to fp32, whatever is done with it next: a conversion to fp16 behind it may otherwise be fused with
// the operation that produced it in one kernel and not in another.
__device__ __forceinline__ float as_fp32(float v) {
    asm("" : "+v"(v));
    return v;
}

// SiLU(g) * u.  The quotient is g times a reciprocal (1 ulp) instead of a division (ten instructions): the result is
// rounded to fp16 right after.  Very negative g: exp overflows to +inf, its reciprocal is 0, the product -0.
__device__ __forceinline__ float swiglu_act(float g, float u) {
    return as_fp32(g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u);
}

// Rotation of a (j, j + hd/2) pair by (cos, sin), the fused operations written out: every tile kernel rounds alike.
__device__ __forceinline__ float rope_lo(float x0, float x1, float c, float s) { return as_fp32(fmaf(x0, c, -(x1 * s))); }
__device__ __forceinline__ float rope_hi(float x0, float x1, float c, float s) { return as_fp32(fmaf(x1, c, x0 * s)); }
