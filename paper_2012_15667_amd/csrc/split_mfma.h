// fp32 products on the 16-bit matrix cores, in three bf16 parts or, from some sixty channels on, in two fp16 parts (further down).
// Three bf16 parts: every operand is cut into x = h + m + l, and the product
// of two operands is taken as the six products of parts that reach fp32 precision (h h, h m, m h, m m, h l, l h; the
// three left out are each below 2^-24 of the product).  A v_mfma_f32_16x16x32_bf16 does 16 times the multiply-adds of an fp32
// matrix instruction in the same time, so six of them still leave a factor of 16 / 6; sums stay in fp32.  Measured on
// register operands: 1937 TFLOP/s of bf16 products = 323 TFLOP/s of fp32 products, against 155 of the fp32 instructions
// (32x32x16_bf16: 1430 - 1690).  Error of a sum of n such products against 64 bits (relative, 2-norm; x uniform on
// [0, 1], w normal), fp32 instructions / this: n = 144 2.2e-7 / 1.9e-7, 576 4.2e-7 / 3.5e-7, 4608 1.23e-6 / 0.99e-6,
// 12800 1.9e-6 / 1.7e-6.  Two bf16 parts would give 4e-6 at every n: not used.
#ifndef IOLB_SPLIT_MFMA_H
#define IOLB_SPLIT_MFMA_H

#include <hip/hip_runtime.h>

#include <type_traits>

#include "wino_transform.h"

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

// ---- two fp16 parts -----------------------------------------------------------------------------
// An operand in two fp16 parts, 2^e v = h + l (11 significant bits each, rounded to nearest: what is left is at most one unit of
// the 24th bit), its products as three: l h, h l, h h; l l, at most 2^-22 of the product, is left out.  Half the matrix work of
// three bf16 parts at a smaller error, since a running sum is rounded half as often (against 64 bits, as above, three bf16 / two fp16
// parts: n = 576 3.6e-7 / 2.7e-7, 1152 5.0e-7 / 3.7e-7, 2304 7.2e-7 / 5.2e-7); single products 0.8 * 2^-24 in the mean.  The instruction
// takes denormal fp16 operands as they are and rounds each sum once, to nearest even (measured bit by bit).
//   fp16 has 5 bits of exponent, so e follows the data: a sample's largest value goes to [2^8, 2^9).  Seven bits are left above it;
// a value beyond them gives infinite or NaN parts, sums that show it, and the output is computed again in plain fp32.  Below 2^-2 parts
// lose bits to the smallest denormal, 2^-24: an operand is off by up to 2^-25 then, which is nothing beside a larger operand of
// the same sum, if that one's partner is not far smaller than its own.  So a group of operands that enter the same sums together (an
// output's window, a kernel's taps and channels) has to hold at least one of 2^-2, or only zeros, and a kernel's sums have to
// reach a line (below) that tells whether what counts in them was cut; where they do not, outputs are computed again, too.  That is slow where it
// happens: 64 -> 64 at 56 x 56, batch 32, with one value of each image 1e5 times the others 35 -> 184 us, with a quarter of each image
// 1e-5 of the rest 182, nine in ten values zero 36 (in three bf16 parts, whatever the finite values, 51).
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
constexpr int HALF_TOP = 9;                                  // sample below 2^9
constexpr float HALF_LEAST = 0.25f;                          // least largest value of a group
// (operands are scaled down by at most 2^23, so that none that is not denormal vanishes; up by what a float holds)
constexpr int HALF_DOWN = -23, HALF_UP = 126;

// Bits of |v|; those of what is not finite come after all others.
__device__ __forceinline__ unsigned magnitude(float v) { return __float_as_uint(v) & 0x7fffffffu; }
// The same, 0 in place of what is not finite.
__device__ __forceinline__ unsigned finite_bits(float v)
{
    const unsigned u = magnitude(v);
    return u < 0x7f800000u ? u : 0u;
}
// 2^e for a sample whose largest value has these bits, as that of a float and as it is; a sample of zeros counts as one up to 1.
// (TOP: the sample's largest value goes below 2^TOP)
template <int TOP = HALF_TOP>
__device__ __forceinline__ unsigned half_scale_bits(unsigned largest)
{
    const int e = TOP + 126 - (int)(largest >> 23);
    const int kept = e < HALF_DOWN ? HALF_DOWN : e > HALF_UP ? HALF_UP : e;
    return (unsigned)(127 + (largest == 0 ? TOP - 1 : kept)) << 23;
}
__device__ __forceinline__ float half_unscale(unsigned scale_bits) { return __uint_as_float((254u << 23) - scale_bits); }
// The largest magnitude of eight values, 0 where one of them is not finite.
__device__ __forceinline__ unsigned largest_of(const float (&v)[8])
{
    unsigned m = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) m = magnitude(v[j]) > m ? magnitude(v[j]) : m;
    return m < 0x7f800000u ? m : 0u;
}
// The largest of a wave's values; every lane takes part.
__device__ __forceinline__ unsigned wave_max(unsigned v)
{
    auto take = [&](unsigned o) { v = o > v ? o : v; };
    take(__builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));             // row_shr:1, 2, 4, 8: a row's last lane has the row's
    take(__builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));             // row_bcast:15, 31
    take(__builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}
// The sum over a wave, in a fixed order; every lane takes part.
__device__ __forceinline__ float wave_sum(float v)
{
    auto take = [&](int o) { v += __int_as_float(o); };
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x112, 0xf, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x114, 0xf, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x118, 0xf, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x142, 0xa, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x143, 0xc, 0xf, false));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// v of the lane whose number differs in bit 0 or 1.
template <int BIT>
__device__ __forceinline__ unsigned quad_other(unsigned v)
{
    return __builtin_amdgcn_update_dpp(0, v, BIT == 0 ? 0xB1 : 0x4E, 0xf, 0xf, false);      // quad_perm 1 0 3 2, 2 3 0 1
}

// What parts of two lose of operands that a larger one of the same sum does not make good: where that one meets a small or a zero partner,
// the lost ones may be all of the sum.  So sums are judged when they are there, per kernel.  Scaled, an operand below HALF_LEAST is off by up to
// 2^-25: those of the inputs by the kernel's elements, those of the kernel (`small` of them) by up to the largest input add an error of
// 2^-25 (|kernel| + sqrt(small) inputs), |.| the 2-norm, in the root mean square and sqrt(n) times that at worst.  Sums of a kernel of which
// none is 2^20 times that (a few pixels' of one image: one sum alone may be small by chance) are computed again: unmarked errors
// of this kind are 2^-21 of the largest of those sums in the root mean square, and no more than sqrt(n) 2^-20, which is less than the n 2^-24 of n
// sums in fp32 from 256 products on.  Sums of uniform, normal, sparse and lognormal inputs by normal, Laplace, sparse and lognormal kernels
// are 2^5 to 2^13 above the line, whatever n.
struct KernelFacts { float squares; float small; };          // sum of the scaled elements' squares; how many are small and not zero
struct KernelLine { float norm, root; };                     // what the line of a kernel follows from
constexpr float HALF_LINE = 0.03125f;
__device__ __forceinline__ KernelLine kernel_line(const KernelFacts& f, float line = HALF_LINE)
{
    return {line * __builtin_amdgcn_sqrtf(f.squares), line * __builtin_amdgcn_sqrtf(f.small)};
}
// (inputs: the largest)
__device__ __forceinline__ float line_of(const KernelLine& k, float inputs) { return k.norm + (k.root > 0.f ? k.root * inputs : 0.f); }
// A piece of a kernel has at most these squares per element that it has room for (where it has more, elements far above the sample, its parts
// are NaN): so there is a line for all kernels that asks for nothing that is not known, which sums are compared with first.
constexpr float HALF_SQUARES = 0x1p26f;
constexpr float HALF_PIECE = 128 * HALF_SQUARES;             // direct and 1 x 1 layers
constexpr float HALF_PIECE_PLANE = 32 * HALF_SQUARES;        // 32 channels of a transformed kernel's plane
// The facts of a wave's 16 MB kernels, which come in pieces `pitch` kernels apart, and their lines to LDS; every lane takes part.
template <int MB>
__device__ __forceinline__ void wave_lines(const KernelFacts* from, int pieces, size_t pitch, int lane, KernelLine* lines)
{
    KernelFacts sum[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) sum[mb] = {0.f, 0.f};
#pragma unroll 4
    for (int p = lane >> 4; p < pieces; p += 4)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const KernelFacts f = from[p * pitch + mb * 16 + (lane & 15)];
            sum[mb].squares += f.squares;
            sum[mb].small += f.small;
        }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
        for (int d = 16; d < 64; d *= 2) {
            sum[mb].squares += __shfl_xor(sum[mb].squares, d);
            sum[mb].small += __shfl_xor(sum[mb].small, d);
        }
        if (lane < 16) lines[mb * 16 + lane] = kernel_line(sum[mb]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}
// The facts of kernel thread % Z, which come in pieces `pitch` kernels apart, are added up by GROUPS = T / Z threads, a share each: the
// first EARLY of its pieces are loaded early.
template <int EARLY>
struct FactsShare {
    const KernelFacts* from;
    int piece, pieces, by;
    size_t pitch;
    KernelFacts early[EARLY];
    __device__ __forceinline__ void load(const KernelFacts* at, int first, int groups, int count, size_t step)
    {
        from = at; piece = first; by = groups; pieces = count; pitch = step;
#pragma unroll
        for (int j = 0; j < EARLY; ++j) early[j] = from[(piece + j * by < pieces ? piece + j * by : 0) * pitch];
    }
    __device__ __forceinline__ KernelFacts sum() const
    {
        KernelFacts all = {0.f, 0.f};
#pragma unroll
        for (int j = 0; j < EARLY; ++j) {
            all.squares += piece + j * by < pieces ? early[j].squares : 0.f;
            all.small += piece + j * by < pieces ? early[j].small : 0.f;
        }
#pragma unroll 4
        for (int p = piece + EARLY * by; p < pieces; p += by) {
            const KernelFacts f = from[p * pitch];
            all.squares += f.squares;
            all.small += f.small;
        }
        return all;
    }
};
// ... and the shares of all of them, in order.
template <int Z, int GROUPS>
__device__ __forceinline__ KernelFacts all_shares(const KernelFacts* shares, int kernel)
{
    KernelFacts all = shares[kernel];
#pragma unroll
    for (int j = 1; j < GROUPS; ++j) {
        all.squares += shares[j * Z + kernel].squares;
        all.small += shares[j * Z + kernel].small;
    }
    return all;
}
// v and what the lane 16 or 32 further holds, both in either lane: their sum or maximum is that of the two.
struct LanePair { float a, b; };
template <int APART>
__device__ __forceinline__ LanePair lanes_apart(float v)
{
    static_assert(APART == 16 || APART == 32);
    const unsigned u = __float_as_uint(v);
    if constexpr (APART == 16) {
        const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        return {__uint_as_float(p[0]), __uint_as_float(p[1])};
    } else {
        const auto p = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return {__uint_as_float(p[0]), __uint_as_float(p[1])};
    }
}
// The largest of four neighbouring lanes' values, where their images agree (NaN where one of them is).
__device__ __forceinline__ float quad_largest(float v, int image)
{
    auto take = [&](auto bit_c) {
        constexpr int BIT = decltype(bit_c)::value;
        const float o = __uint_as_float(quad_other<BIT>(__float_as_uint(v)));
        v = (int)quad_other<BIT>((unsigned)image) == image ? __builtin_elementwise_maximum(v, o) : v;
    };
    take(std::integral_constant<int, 0>{});
    take(std::integral_constant<int, 1>{});
    return v;
}
// The largest of the 16 lanes of a row.
__device__ __forceinline__ float row_largest(float v)
{
    auto take = [&](int o) { v = __builtin_elementwise_maximum(v, __int_as_float(o)); };
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false));             // row_ror:1, 2, 4, 8
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));
    take(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));
    return v;
}
// What the lane before and the lane after hold (of a row of 16; 0 at its ends).
__device__ __forceinline__ float lane_before(float v) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, false)); }
__device__ __forceinline__ float lane_after(float v) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x101, 0xf, 0xf, false)); }
// Which neighbours' pixels a lane of two images takes to its first and last ones: of its image, and of one scale (`scales` at either end).
struct Joins { bool before, after; };
// The sums of a kernel that are judged together, in a wave whose lanes l16 hold NB pixels each (one alone is below its line by chance once in some
// 10^3, and looking closer costs 2 us): of one image a lane's (where NB is less than four its three neighbours' too, of several images, first < last, those of its own; where some pixels are no
// outputs, ragged, all of them); of up to MOST_IMAGES all of each; of more those of four neighbouring pixels that are of one image.  Mixed: a
// lane's pixels that are of one image, several such groups, and those of the lanes beside it that `joins` allows.
// image[nb]: -1 where there is no output.
enum { JUDGE_LANE, JUDGE_IMAGES, JUDGE_QUADS, JUDGE_MIXED };
constexpr int MOST_IMAGES = 4;
constexpr float FINITE = 3.402823466e38f;                    // beyond it a value is not finite
// begin(in): a group of this lane, in(nb) whether a pixel of its is in it; see(mb, i, largest): of kernel 4 grp + i of block mb the largest sum of
// the group.  value(mb, nb, i): a sum's magnitude.  Every lane takes part.
template <int MB, int NB, class Value, class Begin, class See>
__device__ __forceinline__ void judge_sums(int mode, bool ragged, const int (&image)[NB], int first, int last, Value value, Begin begin, See see, Joins joins = {})
{
    if (mode == JUDGE_LANE) {
        begin([&](int nb) { return image[nb] >= 0; });
        float m[MB][4];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                m[mb][i] = 0.f;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) m[mb][i] = __builtin_elementwise_maximum(m[mb][i], value(mb, nb, i));
                if constexpr (NB < 4) m[mb][i] = quad_largest(m[mb][i], first < last ? image[0] : 0);
            }
        if (ragged)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) m[mb][i] = row_largest(m[mb][i]);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) see(mb, i, m[mb][i]);
    } else if (mode == JUDGE_IMAGES) {
#pragma unroll 1
        for (int im = first; im <= last; ++im) {
            begin([&](int nb) { return image[nb] == im; });
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float m = 0.f;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) m = __builtin_elementwise_maximum(m, image[nb] == im ? value(mb, nb, i) : 0.f);
                    see(mb, i, row_largest(m));
                }
        }
    } else if (mode == JUDGE_MIXED) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float m[NB];
#pragma unroll
                for (int at = 0; at < NB; ++at) {
                    m[at] = 0.f;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) m[at] = __builtin_elementwise_maximum(m[at], image[nb] == image[at] ? value(mb, nb, i) : 0.f);
                }
                const float before = lane_before(m[NB - 1]), after = lane_after(m[0]);
                static_for<NB>([&](auto at_c) {
                    constexpr int at = decltype(at_c)::value;
                    begin([&](int nb) { return nb == at && image[nb] >= 0; });
                    float all = m[at];
                    if (joins.before & (image[at] == image[0])) all = __builtin_elementwise_maximum(all, before);
                    if (joins.after & (image[at] == image[NB - 1])) all = __builtin_elementwise_maximum(all, after);
                    see(mb, i, all);
                });
            }
    } else {
        static_for<NB>([&](auto at_c) {
            constexpr int at = decltype(at_c)::value;
            begin([&](int nb) { return nb == at && image[nb] >= 0; });
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) see(mb, i, quad_largest(value(mb, at, i), image[at]));
        });
    }
}
// Two values, scaled already.
__device__ __forceinline__ void half_pair(float a, float b, unsigned& h, unsigned& l)
{
    const f16x2 hv = {(_Float16)a, (_Float16)b};
    h = __builtin_bit_cast(unsigned, hv);
    asm("" : "+v"(h));                                       // (not converted a second time)
    const f16x2 hb = __builtin_bit_cast(f16x2, h);
    const f16x2 lv = {(_Float16)(a - (float)hb[0]), (_Float16)(b - (float)hb[1])};
    l = __builtin_bit_cast(unsigned, lv);
}
// Eight, scaled here; returns the largest of them, scaled.
__device__ __forceinline__ float half_eight(const float (&v)[8], float scale, u32x4& h, u32x4& l)
{
    float most = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float a = v[2 * j] * scale, b = v[2 * j + 1] * scale;
        unsigned hj, lj;
        half_pair(a, b, hj, lj);
        h[j] = hj; l[j] = lj;
        most = __builtin_fmaxf(__builtin_fmaxf(most, __builtin_fabsf(a)), __builtin_fabsf(b));
    }
    return most;
}

}  // namespace iolb

#endif
