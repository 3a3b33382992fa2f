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

// v plus the value that a DPP move brings from another lane (0 where the move has no source lane)
template <int kCtrl, int kRowMask>
__device__ inline double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, kRowMask, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, kRowMask, 0xf, true);
    return v + __hiloint2double(hi, lo);
}

// Sum over the 64 lanes of a wave; every lane receives the total. Fixed order, so the result does not depend
// on scheduling. Lanes are added within their row of 16 (shifts by 1, 2, 4, 8), row 0 into 1 and 2 into 3, then
// the lower half into the upper; lane 63 holds the total. DPP moves stay in the vector ALU: about a quarter of the
// latency of the same sum through LDS permutes, which the small reductions of a Krylov step wait for.
__device__ inline double wave_sum(double v) {
    v = dpp_add<0x111, 0xf>(v);   // row_shr:1
    v = dpp_add<0x112, 0xf>(v);   // row_shr:2
    v = dpp_add<0x114, 0xf>(v);   // row_shr:4
    v = dpp_add<0x118, 0xf>(v);   // row_shr:8
    v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63), hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}

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
