// fp32 operands on the bf16 matrix units, without losing fp32's precision.
//
// An fp32 value x, times 2^24, is the exact sum of three bf16 values,
//   h = bf16(x'),  m = bf16(x' - h),  l = x' - h - m,   x' = 2^24 x
// (round to nearest: |m| <= 2^-8 |x'|, |l| <= 2^-17 |x'|; l fits in eight bits,
// so nothing is lost).  The factor keeps every part that is not zero a normal
// bf16 number: x may be any fp32 value, subnormal or not, while without it
// the parts of values below 2^-110 fell under bf16's smallest subnormal (2e-6
// off at 2^-118, 2.5e-4 at 2^-125).  A product x' * y' is then six bf16 products,
//   hh + (hm + mh) + (hl + mm + lh),
// each exact in fp32; the three left out (ml, lm, ll) are below 2^-24 |x' y'|,
// under half a unit in the last place of the fp32 product.  On gfx950 a bf16
// MFMA does 16 times the multiply-adds of an fp32 one per cycle, so six of
// them still take 2.7 times less time than the fp32 MFMA.
//
// Sums of them times kUnscale are the sums of x * y.
//
// Values whose h overflows (infinities, NaN, and magnitudes from about 2^104 on) make
// every product they enter non-finite (h * h' is infinite or NaN), as do sums
// from 2^80 on, so a kernel finds them by looking at its own results and
// computes those again in plain fp32 arithmetic.
#pragma once

#include "common.hpp"

namespace dpg {
namespace split {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

constexpr float kScale = 16777216.0f;                   // 2^24
constexpr float kUnscale = 1.0f / (kScale * kScale);

// two floats rounded to bf16, the first in the low half
__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

__device__ __forceinline__ float low_f32(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float high_f32(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

// the three parts of two values (times kScale), packed pairwise
__device__ __forceinline__ void split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    a *= kScale;
    b *= kScale;
    h = pack2(a, b);
    const float ra = a - low_f32(h), rb = b - high_f32(h);
    m = pack2(ra, rb);
    l = pack2(ra - low_f32(m), rb - high_f32(m));
}

__device__ __forceinline__ bool finite_f32(float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; }

}  // namespace split
}  // namespace dpg
