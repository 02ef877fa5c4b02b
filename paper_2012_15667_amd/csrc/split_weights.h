// The kernels of a block of output channels on their way to the operands of the split matrix kernels: rows of w are read
// as they lie, a wave along each, and go through LDS; the lanes then gather their channels from there.  (Gathered from memory
// each lane reads single floats a row apart: one cache line per lane and load, and every line of w once per tap and XCD.)
#ifndef IOLB_SPLIT_WEIGHTS_H
#define IOLB_SPLIT_WEIGHTS_H

#include "kernels.h"
#include "split_mfma.h"
#include "wino_mats.h"
#include "wino_transform.h"

namespace iolb {

// Floats [0, len) of ROWS rows into lds, `pitch` (odd) floats apart, by WAVES waves.  Row r starts at w + r * stride; rows from
// `rows` on, and floats from `have` on, are zero.  COLS blocks of 64 floats are in flight at a time.
template <int ROWS, int WAVES, int COLS>
__device__ __forceinline__ void stage_kernels(const float* __restrict__ w, float* lds, int wave, int lane, long long stride, int rows, int have, int len, int pitch)
{
    constexpr int MINE = ROWS / WAVES;
    for (int o0 = lane; o0 < len + lane; o0 += 64 * COLS) {
        float v[COLS][MINE];
#pragma unroll
        for (int c = 0; c < COLS; ++c)
#pragma unroll
            for (int j = 0; j < MINE; ++j) {
                const int r = wave * MINE + j, o = o0 + 64 * c;
                const bool exists = r < rows && o < have;
                v[c][j] = w[exists ? r * stride + o : 0];
                v[c][j] = exists ? v[c][j] : 0.f;
            }
#pragma unroll
        for (int c = 0; c < COLS; ++c)
#pragma unroll
            for (int j = 0; j < MINE; ++j)
                if (o0 + 64 * c < len) lds[(wave * MINE + j) * pitch + o0 + 64 * c] = v[c][j];
    }
}

// A piece of eight values: its three bf16 parts, each to its 64 lanes.
__device__ __forceinline__ void store_parts(u32x4* to, const unsigned short (&p)[3][8])
{
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        u32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (unsigned)p[q][2 * i] | ((unsigned)p[q][2 * i + 1] << 16);
        to[q * 64] = o;
    }
}

// The piece of eight transformed kernel elements in two fp16 parts, scaled already, of kernel lane % KERNELS and the channels of lane / KERNELS; the
// lanes that share a kernel, lane % KERNELS, judge it together (of `channels` < 16 some are all small now and then: left to the sums).  NaN in
// place of a kernel too small for its scale, or with larger squares (of what is returned).  Returns what the elements of the lane, or (SHARED) of all lanes that share the kernel, tell of it.
template <int KERNELS, bool SHARED>
__device__ __forceinline__ KernelFacts store_halves(u32x4* to, const float (&u)[8], int channels, float most_squares)
{
    u32x4 h, l;
    float most = half_eight(u, 1.f, h, l);
    KernelFacts facts = {0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        facts.squares = __builtin_fmaf(u[j], u[j], facts.squares);
        facts.small += magnitude(u[j]) - 1 < __float_as_uint(HALF_LEAST) - 1 ? 1.f : 0.f;       // (zero comes last)
    }
    auto share = [&](auto apart_c) {
        constexpr int APART = decltype(apart_c)::value;
        const LanePair m = lanes_apart<APART>(most);
        most = __builtin_fmaxf(m.a, m.b);
        if constexpr (SHARED) {
            const LanePair q = lanes_apart<APART>(facts.squares), s = lanes_apart<APART>(facts.small);
            facts.squares = q.a + q.b;
            facts.small = s.a + s.b;
        }
    };
    static_assert(KERNELS == 16 || KERNELS == 32);
    if constexpr (KERNELS == 16) share(std::integral_constant<int, 16>{});
    share(std::integral_constant<int, 32>{});
    const bool fits = (channels < 16 || most == 0.f || most >= HALF_LEAST) && facts.squares <= most_squares;
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] |= fits ? 0u : 0x7e007e00u;
    to[0] = h;
    to[64] = l;
    return facts;
}
// The channel of spot 0 ... 15 at which kernels are sampled for their scale: two elements of each, g[0][0] and g[2][2], which are also
// elements of the transformed kernel, times a power of two.
__device__ __forceinline__ int sampled_channel(int spot, int C) { return (int)((long long)C * spot >> 4); }
// The sample of kernel k from w[K][C][3][3]: one value in each of lanes 0 ... 31.
__device__ __forceinline__ float sampled_value(const float* __restrict__ w, int k, int K, int C, int lane)
{
    const bool exists = lane < 32 && k < K;
    const float v = w[exists ? ((size_t)k * C + sampled_channel(lane >> 1, C)) * 9 + 8 * (lane & 1) : 0];
    return exists ? v : 0.f;
}
// The scale of kernel k from U[plane][rows][cols]; the 64 / KERNELS lanes that share it take their part of the channels each.
template <int M, int KERNELS>
__device__ __forceinline__ unsigned scale_of_given(const float* __restrict__ U, int k, int K, int C, int rows, int cols, int lane)
{
    constexpr int n = M + 2, SPOTS = 16 * KERNELS / 64;
    // L begins and ends with a row of one element, a power of two
    static_assert(Mats<M>::L[n - 1][2] == 1.f && Mats<M>::L[0][1] == 0.f && Mats<M>::L[0][2] == 0.f && Mats<M>::L[n - 1][0] == 0.f && Mats<M>::L[n - 1][1] == 0.f);
    constexpr float first = 1.f / (Mats<M>::L[0][0] * Mats<M>::L[0][0]);
    float s0[SPOTS], s1[SPOTS];
    const int kc = k < K ? k : 0;
#pragma unroll
    for (int j = 0; j < SPOTS; ++j) {
        const size_t c = sampled_channel(lane / KERNELS * SPOTS + j, C);
        s0[j] = U[c * cols + kc];
        s1[j] = U[((size_t)(n * n - 1) * rows + c) * cols + kc];
    }
    unsigned some = 0;
#pragma unroll
    for (int j = 0; j < SPOTS; ++j) {
        const unsigned a = finite_bits(s0[j] * first), b = finite_bits(s1[j]);
        some = a > some ? a : some;
        some = b > some ? b : some;
    }
    some = k < K ? some : 0u;
#pragma unroll
    for (int d = KERNELS; d < 64; d *= 2) {
        const unsigned o = __shfl_xor(some, d);
        some = o > some ? o : some;
    }
    return half_scale_bits(some);
}
// What brings row `row` of a transformed kernel to the size of the kernel.
template <int M>
__device__ __forceinline__ float row_up(int row)
{
    float up = 1.f;
    static_for<M + 2>([&](auto r) { if (row == decltype(r)::value) up = power_of_two(kernel_up<M>(decltype(r)::value)); });
    return up;
}
// The weight of its sums in an output.
template <int M>
__device__ __forceinline__ float row_weight(int row)
{
    float weight = 0.f;
    static_for<M + 2>([&](auto r) {
        constexpr float of_row = plane_weight<M>(decltype(r)::value);
        if (row == decltype(r)::value) weight = of_row;
    });
    return weight;
}
// What brings it back.
template <int M>
__device__ __forceinline__ float row_down(int row)
{
    float down = 1.f;
    static_for<M + 2>([&](auto r) { if (row == decltype(r)::value) down = power_of_two(-kernel_up<M>(decltype(r)::value)); });
    return down;
}

// A transformed kernel element as the caller's kernels give it, for blocks that are taken again (their two parts are not always all of it):
// from w[K][C] (no transform), U[plane][C rounded up to 16][K rounded up to 32] or w[K][C][3][3].
struct RawKernels {
    const float* w;
    int raw, plane, C, K;
    float li[3], lj[3];
    __device__ __forceinline__ RawKernels(const float* from, int kind, int m, int which, int channels, int kernels) : w(from), raw(kind), plane(which), C(channels), K(kernels)
    {
        const int n = m + 2, row = kind == SPLIT_RAW_TAPS ? plane / n : 0, col = kind == SPLIT_RAW_TAPS ? plane % n : 0;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            li[j] = kind == SPLIT_RAW_TAPS ? coefficient(m, row, j) : 0.f;
            lj[j] = kind == SPLIT_RAW_TAPS ? coefficient(m, col, j) : 0.f;
        }
    }
    static __device__ __forceinline__ float coefficient(int m, int row, int j)
    {
        return m == 2 ? Mats<2>::L[row][j] : m == 3 ? Mats<3>::L[row][j] : m == 4 ? Mats<4>::L[row][j] : Mats<6>::L[row][j];
    }
    // (as `accumulate` adds: to the bits of a transformed kernel in memory)
    static __device__ __forceinline__ float add(float coef, float v, float to) { return coef == 0.f ? to : __builtin_fmaf(coef, v, to); }
    __device__ __forceinline__ float at(int k, int c) const
    {
        if (k >= K || c >= C) return 0.f;
        if (raw == SPLIT_RAW_ROWS) return w[(size_t)k * C + c];
        if (raw == SPLIT_RAW_PLANES) return w[((size_t)plane * ((C + 15) / 16 * 16) + c) * ((K + 31) / 32 * 32) + k];
        return of(w + ((size_t)k * C + c) * 9);
    }
    // (of nine taps)
    __device__ __forceinline__ float of(const float* t) const
    {
        float u = 0.f;
#pragma unroll
        for (int j = 0; j < 3; ++j) u = add(lj[j], add(li[2], t[6 + j], add(li[1], t[3 + j], add(li[0], t[j], 0.f))), u);
        return u;
    }
};

// Row `row` (the same in every lane of a wave) of L g for eight channels, g[3][3] one after the other from `from` on.  A branch per
// row: with every row computed and one selected, the launch that the input transform shares took 254 registers in F(3 x 3), 210 in
// F(4 x 4) (now 66 and 61 - 112, as without), which left two waves per SIMD (382 -> 132 at 121 x 121, batch 9, F(3 x 3): 633 us,
// now 579).
template <int M>
__device__ __forceinline__ void kernel_row(int row, const float* from, float (&lg)[8][3])
{
    static_for<M + 2>([&](auto r) {
        if (row != decltype(r)::value) return;
        static_for<8>([&](auto c) {
            static_for<3>([&](auto j) {
                float u = 0.f;
                bool first = true;
                static_for<3>([&](auto i) { accumulate<M, UseL, decltype(r)::value, decltype(i)::value>(u, first, from[c * 9 + i * 3 + j]); });
                lg[c][j] = u;
            });
        });
    });
}
// Element J of that row of L g L^T.
template <int M, int J>
__device__ __forceinline__ float kernel_element(const float (&lg)[3])
{
    float u = 0.f;
    bool first = true;
    static_for<3>([&](auto b) { accumulate<M, UseL, J, decltype(b)::value>(u, first, lg[b]); });
    return u;
}

}  // namespace iolb

#endif
