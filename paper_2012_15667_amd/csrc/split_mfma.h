// fp32 products on the bf16 matrix cores: every operand is cut into three bf16 parts, x = h + m + l, and the product
// of two operands is taken as the six products of parts that reach fp32 precision (h h, h m, m h, m m, h l, l h; the
// three left out are each below 2^-24 of the product).  A v_mfma_f32_16x16x32_bf16 does 16 times the multiply-adds of an fp32
// matrix instruction in the same time, so six of them still leave a factor of 16 / 6; sums stay in fp32.  Measured on
// register operands: 1937 TFLOP/s of bf16 products = 323 TFLOP/s of fp32 products, against 155 of the fp32 instructions
// (32x32x16_bf16: 1430 - 1690).  Error of a sum of n such products against 64 bits (relative, 2-norm; x uniform on
// [0, 1], w normal), fp32 instructions / this: n = 144 2.2e-7 / 1.9e-7, 576 4.2e-7 / 3.5e-7, 4608 1.23e-6 / 0.99e-6,
// 12800 1.9e-6 / 1.7e-6.  Three products (two parts) would give 4e-6 at every n: not used.
#ifndef IOLB_SPLIT_MFMA_H
#define IOLB_SPLIT_MFMA_H

#include <hip/hip_runtime.h>

#include <type_traits>

namespace iolb {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// The same value, of which the compiler does not know that: what is derived from it is computed where it is used and
// not kept in registers from an equal expression before (here: through the matrix loop).
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Calls f with the integral constants FROM ... TO - 1.
template <int FROM, int TO, class F>
__device__ __forceinline__ void static_range(F f)
{
    if constexpr (FROM < TO) {
        f(std::integral_constant<int, FROM>{});
        static_range<FROM + 1, TO>(f);
    }
}

// voffset of an element that does not exist: beyond every buffer's range, so that the load returns zero
constexpr unsigned OUTSIDE = 0x80000000u;

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Both operands are scaled by 2^23 before they are cut: every bit of an fp32 value, down to 2^-149, is then at least the
// smallest normal bf16, so that the three parts hold any value exactly and no instruction sees a denormal operand.  Sums
// are scaled back by 2^-46 when they are written.  At the other end operands from 2^105 and sums from 2^82 on overflow,
// which the sum shows: it is infinite or NaN, as with operands that are not finite, and the output is computed again in
// plain fp32.
constexpr float SPLIT_SCALE = 8388608.f;                     // 2^23
constexpr float SPLIT_UNSCALE = 1.f / SPLIT_SCALE / SPLIT_SCALE;

// The two as one register, which the compiler takes apart with a shift and a mask; it would convert the first one a
// second time otherwise.
__device__ __forceinline__ unsigned packed(bf16x2 v)
{
    unsigned u = __builtin_bit_cast(unsigned, v);
    asm("" : "+v"(u));
    return u;
}

// 2^23 x = h + m + l with h, m, l bf16 (8 significant bits each, rounded to nearest, so that the two differences are
// exact): two operands at a time, one packed conversion per part.
__device__ __forceinline__ void split_pair(float a, float b, unsigned& h, unsigned& m, unsigned& l)
{
    a *= SPLIT_SCALE;
    b *= SPLIT_SCALE;
    const bf16x2 hv = {(__bf16)a, (__bf16)b};
    h = packed(hv);
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
    const bf16x2 mv = {(__bf16)ra, (__bf16)rb};
    m = packed(mv);
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

// For values that are kept (weights): a value beyond the parts' range is kept whole, its two halves in place of m and l,
// under a NaN that makes every sum it enters NaN.
__device__ __forceinline__ void split_kept(float a, unsigned short& h, unsigned short& m, unsigned short& l)
{
    const float v = a * SPLIT_SCALE;
    const unsigned u = __float_as_uint(a);
    h = __builtin_bit_cast(unsigned short, (__bf16)v);
    const float r = v - __uint_as_float((unsigned)h << 16);
    m = __builtin_bit_cast(unsigned short, (__bf16)r);
    l = __builtin_bit_cast(unsigned short, (__bf16)(r - __uint_as_float((unsigned)m << 16)));
    const bool beyond = (h & 0x7f80) == 0x7f80;
    h = beyond ? (unsigned short)0x7fc0 : h;
    m = beyond ? (unsigned short)(u >> 16) : m;
    l = beyond ? (unsigned short)u : l;
}

// The value that split_kept was given.
__device__ __forceinline__ float kept_value(unsigned h, unsigned m, unsigned l)
{
    const float parts = __uint_as_float(h << 16) + (__uint_as_float(m << 16) + __uint_as_float(l << 16));
    return h == 0x7fc0 ? __uint_as_float(m << 16 | l) : parts * (1.f / SPLIT_SCALE);
}

// Eight of them from the three pieces of a lane.
__device__ __forceinline__ void kept_eight(const u32x4& h, const u32x4& m, const u32x4& l, float (&v)[8])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[2 * j] = kept_value(h[j] & 0xffffu, m[j] & 0xffffu, l[j] & 0xffffu);
        v[2 * j + 1] = kept_value(h[j] >> 16, m[j] >> 16, l[j] >> 16);
    }
}

}  // namespace iolb

#endif
