// fp32 products on the bf16 matrix cores: every operand is cut into three bf16 parts, x = h + m + l, and the product
// of two operands is taken as the six products of parts that reach fp32 precision (h h, h m, m h, m m, h l, l h; the
// three left out are below 2^-24 of the product).  A v_mfma_f32_16x16x32_bf16 does 16 times the multiply-adds of an fp32
// matrix instruction in the same time, so six of them still leave a factor of 16 / 6; sums stay in fp32.  Measured on
// register operands: 1937 TFLOP/s of bf16 products = 323 TFLOP/s of fp32 products, against 155 of the fp32 instructions
// (32x32x16_bf16: 1430 - 1690).  Error of a sum of n such products against 64 bits (relative, 2-norm; x uniform on
// [0, 1], w normal), fp32 instructions / this: n = 144 2.2e-7 / 1.9e-7, 576 4.2e-7 / 3.5e-7, 4608 1.23e-6 / 0.99e-6,
// 12800 1.9e-6 / 1.7e-6.  Three products (two parts) would give 4e-6 at every n: not used.
#ifndef IOLB_SPLIT_MFMA_H
#define IOLB_SPLIT_MFMA_H

#include <hip/hip_runtime.h>

namespace iolb {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// x = h + m + l with h, m, l bf16 (8 significant bits each, rounded to nearest, so that the two differences are
// exact): two operands at a time, one packed conversion per part.
__device__ __forceinline__ void split_pair(float a, float b, unsigned& h, unsigned& m, unsigned& l)
{
    const bf16x2 hv = {(__bf16)a, (__bf16)b};
    h = __builtin_bit_cast(unsigned, hv);
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
    const bf16x2 mv = {(__bf16)ra, (__bf16)rb};
    m = __builtin_bit_cast(unsigned, mv);
    const float sa = ra - __uint_as_float(m << 16), sb = rb - __uint_as_float(m & 0xffff0000u);
    const bf16x2 lv = {(__bf16)sa, (__bf16)sb};
    l = __builtin_bit_cast(unsigned, lv);
}

// The same for eight values: the three 16-byte operands of a lane.
__device__ __forceinline__ void split_eight(const float (&v)[8], u32x4& h, u32x4& m, u32x4& l)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        unsigned hj, mj, lj;
        split_pair(v[2 * j], v[2 * j + 1], hj, mj, lj);
        h[j] = hj; m[j] = mj; l[j] = lj;
    }
}

// For values that are kept (weights): parts whose sum is the value for infinities, NaN and the largest finite
// values too (h truncated where rounding would overflow, no differences of infinities).
__device__ __forceinline__ void split_kept(float a, unsigned short& h, unsigned short& m, unsigned short& l)
{
    const unsigned u = __float_as_uint(a);
    unsigned hu = (unsigned)__builtin_bit_cast(unsigned short, (__bf16)a) << 16;
    if ((hu & 0x7f800000u) == 0x7f800000u && (u & 0x7f800000u) != 0x7f800000u) hu = u & 0xffff0000u;
    h = (unsigned short)(hu >> 16);
    m = l = 0;
    if ((hu & 0x7f800000u) != 0x7f800000u) {
        const float r = a - __uint_as_float(hu);
        const unsigned mu = (unsigned)__builtin_bit_cast(unsigned short, (__bf16)r) << 16;
        m = (unsigned short)(mu >> 16);
        l = __builtin_bit_cast(unsigned short, (__bf16)(r - __uint_as_float(mu)));
    }
}

__device__ __forceinline__ float bf16_bits_to_float(unsigned short b) { return __uint_as_float((unsigned)b << 16); }

}  // namespace iolb

#endif
