// fp32 numbers as sums of three bf16 numbers, for the direct kernels that multiply them on the bf16 matrix cores.
//
// 2^16 x = x0 + x1 + x2 with 8 significant bits each holds the 24 bits of x, or all that a subnormal x has: bf16 reaches down to 2^-133,
// so without the factor operands below 2^-110 would lose bits (all but eight at 2^-126).  A product is taken as x0 y0 + (x0 y1 + x1 y0) +
// (x0 y2 + x1 y1 + x2 y0): what is left out is below 2^-24 of it, every partial product is exact, and sums are kept in fp32, 2^32
// too large until they are done.  Sums from 2^96 on may so be infinite, as parts of operands from 2^112 on are: results that are not
// finite are taken again by the kernels, in fp32 from memory.
// Six v_mfma_f32_16x16x32_bf16 (16 clocks each) do the work of eight v_mfma_f32_16x16x4_f32 (32 clocks each).
//
// How far such sums are from 64 bits (2-norm, dot products of 5000 / 40 000 terms; fp32 instruction: 1.2e-6 / 3.6e-6): added
// into one running sum 1.1e-6 / 3.5e-6 -- and 1.16 times the fp32 error where half of one operand is zero --, each step of six
// summed from zero and then added 2.3e-7 / 6.3e-7.  The kernels do the latter.
//
// The instruction rounds its sums downwards (fp32 MFMAs round to nearest): results were low by 2e-8 to 1.3e-7 of their root mean
// square, all by the same, and the gradients of a net of six layers, which add that up, 2e-6 off where rounding to nearest leaves
// 3e-7.  So one operand changes its sign from step to step, and every second step is subtracted: what rounds down in one
// rounds up in the next.
#pragma once

#include "znn_internal.h"

namespace znn {
namespace split {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const char* lds_bytes;
typedef __attribute__((address_space(3))) const uintx4* lds_quads;
typedef __attribute__((address_space(3))) const int* lds_ints;
typedef __attribute__((address_space(1))) const float* global_floats;

constexpr int kPartBytes = 16;      // one part of eight numbers
constexpr int kVectorBytes = 48;    // three parts of eight numbers
constexpr float kLargest = 3.4028234e38f;
constexpr float kScale = 65536.f;                       // of an operand
constexpr float kUnscale = 1.f / (kScale * kScale);     // of a sum

// The leading bf16 part of x and y, packed; x and y keep the rest, which is exact.
__device__ __forceinline__ unsigned take_part(float& x, float& y)
{
    const unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2){x, y}, bf16x2));
    x -= __builtin_bit_cast(float, u << 16);
    y -= __builtin_bit_cast(float, u & 0xffff0000u);
    return u;
}

__device__ __forceinline__ uintx4 take_part8(float (&x)[8])
{
    uintx4 u;
    u[0] = take_part(x[0], x[1]);
    u[1] = take_part(x[2], x[3]);
    u[2] = take_part(x[4], x[5]);
    u[3] = take_part(x[6], x[7]);
    return u;
}

__device__ __forceinline__ floatx4 mfma(const bf16x8& a, const bf16x8& b, const floatx4& c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// acc += sign t; SIGN: 1 or -1, or 0 where only `sign` (uniform) says it
template <int SIGN>
__device__ __forceinline__ void add_signed(floatx4& acc, const floatx4& t, float sign)
{
    if (SIGN > 0) acc += t;
    else if (SIGN < 0) acc -= t;
    else {
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = fmaf(t[r], sign, acc[r]);
    }
}

// Six products of a step, from zero, smallest first, for NJ row tiles and one column tile.  acc += sign before (add_signed) is the
// column tile before, whose products are done by now: between the instructions of this one they cost nothing.
template <int NJ, int SIGN>
__device__ __forceinline__ void products(floatx4 (&t)[NJ], const bf16x8 (&a)[NJ][3], const uintx4 (&b)[3], const floatx4 (&before)[NJ],
                                         float sign, floatx4* const (&acc)[NJ])
{
    const bf16x8 c0 = __builtin_bit_cast(bf16x8, b[0]), c1 = __builtin_bit_cast(bf16x8, b[1]), c2 = __builtin_bit_cast(bf16x8, b[2]);
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NJ; ++j) t[j] = mfma(a[j][0], c2, zero);
#pragma unroll
    for (int j = 0; j < NJ; ++j) t[j] = mfma(a[j][2], c0, t[j]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) add_signed<SIGN>(*acc[j], before[j], sign);
#pragma unroll
    for (int j = 0; j < NJ; ++j) t[j] = mfma(a[j][1], c1, t[j]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) t[j] = mfma(a[j][0], c1, t[j]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) t[j] = mfma(a[j][1], c0, t[j]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) t[j] = mfma(a[j][0], c0, t[j]);
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace split
}  // namespace znn
