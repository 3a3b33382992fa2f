// Device helpers shared by the HIP kernels of libwfq.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.h"

namespace wfq {

// Round a double to bfloat16 (nearest, ties to even) from its bits, so no intermediate float
// rounding can alter the result. Finite values in the normal range (or zero) only.
__device__ inline uint16_t bf16_rne(double v) {
    uint64_t b = (uint64_t)__double_as_longlong(v);
    uint64_t sign = b >> 63;
    int e = (int)((b >> 52) & 0x7ff);
    if (e == 0) return (uint16_t)(sign << 15);
    uint64_t mant = b & 0xfffffffffffffull;
    uint64_t keep = mant >> 45;
    uint64_t rest = mant & ((1ull << 45) - 1);
    const uint64_t half = 1ull << 44;
    uint32_t out = (uint32_t)(((uint64_t)(e - 1023 + 127) << 7) | keep);
    if (rest > half || (rest == half && (keep & 1))) out += 1;
    return (uint16_t)((sign << 15) | out);
}

__device__ inline float bf16_to_float(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

template <typename E>
__device__ inline E cast_from_double(double v);
template <>
__device__ inline double cast_from_double<double>(double v) { return v; }
template <>
__device__ inline float cast_from_double<float>(double v) { return (float)v; }  // round to nearest even
template <>
__device__ inline uint16_t cast_from_double<uint16_t>(double v) { return bf16_rne(v); }

__device__ inline double widen(double v) { return v; }
__device__ inline double widen(float v) { return (double)v; }

// v plus the value `n` lanes further round its row of 16
template <int n>
__device__ inline double row_rotate_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + n, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + n, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}

// Sum over the 64 lanes of a wave; every lane receives the total. Fixed order, so the result does not depend
// on scheduling: the butterfly over the lane distances 32, 16, 8, 4, 2, 1. The first two steps swap half waves and
// rows of 16 between two copies of v; after the step of distance d the values repeat every d lanes, so that
// the next, within a row, is a rotation. All of it stays in the vector ALU: about a quarter of the latency of
// the same butterfly through LDS permutes, which the small reductions of a Krylov step wait for.
__device__ inline double half_swap(double v) {   // the value 32 lanes on
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    const bool low = (threadIdx.x & 32) == 0;
    return __hiloint2double(low ? hi[1] : hi[0], low ? lo[1] : lo[0]);
}
__device__ inline double half_wave_sum(double v) {   // the sum over each half, in all of its lanes
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    v = row_rotate_add<8>(v);
    v = row_rotate_add<4>(v);
    v = row_rotate_add<2>(v);
    return row_rotate_add<1>(v);
}
__device__ inline double wave_sum(double v) {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return half_wave_sum(__hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]));
}
// sum of x^2, the first addition fused with the lane's own square; valid in lanes 0 .. 31 (the two halves may
// differ in the last bit)
__device__ inline double wave_sum_sq(double x) { return half_wave_sum(fma(x, x, half_swap(x * x))); }

// ---- FP32 operands of the FP16 matrix cores: x = h + l + e, h the FP16 rounding of x, l that of x - h
__device__ inline halfx8 split_hi(const float (&x)[8]) {
    halfx8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (_Float16)x[e];
    return h;
}
__device__ inline halfx8 split_lo(const float (&x)[8], const halfx8& h) {
    halfx8 l;
#pragma unroll
    for (int e = 0; e < 8; ++e) l[e] = (_Float16)(x[e] - (float)h[e]);
    return l;
}

// The same with fewer vector instructions, for kernels that these bound (a kernel bound by its matrix
// products was slower with it: the asm pins the order): h is made in pairs, one conversion for two values,
// and x - h is one mixed-precision fused multiply-add. The empty asm keeps the compiler from
// converting every value a second time for it, and one (1.0f) has to come from a register it knows nothing of.
__device__ inline void split_f16(const float (&x)[8], float one, halfx8& h, halfx8& l) {
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        unsigned bits = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{x[e], x[e + 1]}, halfx2));
        asm("" : "+v"(bits));
        const halfx2 p = __builtin_bit_cast(halfx2, bits);
        h[e] = p.x;
        h[e + 1] = p.y;
        l[e] = (_Float16)fmaf(x[e], one, -(float)p.x);
        l[e + 1] = (_Float16)fmaf(x[e + 1], one, -(float)p.y);
    }
}

}  // namespace wfq
