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
typedef __attribute__((address_space(1))) const char* global_bytes;
typedef __attribute__((address_space(1))) const void* global_ptr;
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef __attribute__((address_space(1))) const uintx4* global_quads;

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
__device__ __forceinline__ float add_signed(float acc, float t, float sign)
{
    return SIGN > 0 ? acc + t : SIGN < 0 ? acc - t : fmaf(t, sign, acc);
}

template <int SIGN>
__device__ __forceinline__ void add_signed(floatx4& acc, const floatx4& t, float sign)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = add_signed<SIGN>(acc[r], t[r], sign);
}

// Six products of a step, from zero, smallest first, for NJ row tiles and one column tile.  acc += sign before (add_signed) is the
// column tile before, whose products are done by now.  An MFMA keeps the matrix core for 16 clocks, of which its wave needs four to issue it: one
// addition and one request for an operand (request(slot), slot = 0 .. 6 NJ - 1) in between cost nothing, many in a row, or an addition of what
// the last MFMA has not finished, do.  PACED: in that order, which takes a few registers more (40 -> 40 maps, 64^3, 5^3, 469 -> 461 us forward and 523 -> 511 the gradient);
// products of a single row tile wait for each other anyway.
template <int NJ, int SIGN, bool PACED, class Request>
__device__ __forceinline__ void products(floatx4 (&t)[NJ], const bf16x8 (&a)[NJ][3], const uintx4 (&b)[3], const floatx4 (&before)[NJ],
                                         float sign, floatx4* const (&acc)[NJ], Request request)
{
    constexpr int ofA[6] = {0, 2, 1, 0, 1, 0}, ofB[6] = {2, 0, 1, 1, 0, 0};
    if (!PACED)
#pragma unroll
        for (int slot = 0; slot < 6 * NJ; ++slot) request(slot);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < 6; ++g)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            t[j] = mfma(a[j][ofA[g]], __builtin_bit_cast(bf16x8, b[ofB[g]]), g ? t[j] : floatx4{0.f, 0.f, 0.f, 0.f});
            if (PACED) request(g * NJ + j);
            if (g >= 1 && g <= 4) (*acc[j])[g - 1] = add_signed<SIGN>((*acc[j])[g - 1], before[j][g - 1], sign);
            if (PACED || (g == 5 && j == NJ - 1)) __builtin_amdgcn_sched_barrier(0);
        }
}

}  // namespace split
}  // namespace znn
