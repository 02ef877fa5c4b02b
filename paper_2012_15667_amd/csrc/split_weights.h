// The kernels of a block of output channels on their way to the operands of the split matrix kernels: rows of w are read
// as they lie, a wave along each, and go through LDS; the lanes then gather their channels from there.  (Gathered from memory
// each lane reads single floats a row apart: one cache line per lane and load, and every line of w once per tap and XCD.)
#ifndef IOLB_SPLIT_WEIGHTS_H
#define IOLB_SPLIT_WEIGHTS_H

#include "split_mfma.h"
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

// A piece of eight values: its three parts, each to its 64 lanes.
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

// The piece of eight transformed kernel elements in two fp16 parts, scaled already, of kernel lane & 15 and the channels of lane >> 4; the
// four lanes that share a kernel judge it together (of `channels` < 16 some are all small now and then: not judged).  NaN in place
// of a kernel too small for its scale.
__device__ __forceinline__ void store_halves(u32x4* to, const float (&u)[8], int channels)
{
    u32x4 h, l;
    float most = half_eight(u, 1.f, h, l);
    most = __builtin_fmaxf(most, __shfl_xor(most, 16));
    most = __builtin_fmaxf(most, __shfl_xor(most, 32));
    const unsigned poison = channels >= 16 && most != 0.f && most < HALF_LEAST ? 0x7e007e00u : 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] |= poison;
    to[0] = h;
    to[64] = l;
}
// The channel of spot 0 ... 15 at which kernels are sampled for their scale: two elements of each, g[0][0] and g[2][2], which are also
// elements of the transformed kernel, times a power of two.
__device__ __forceinline__ int sampled_channel(int spot, int C) { return (int)((long long)C * spot >> 4); }

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
