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

// Row `row` of L g for eight channels, g[3][3] one after the other from `from` on.
template <int M>
__device__ __forceinline__ void kernel_row(int row, const float* from, float (&lg)[8][3])
{
    constexpr int n = M + 2;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float g[3][3], t[n][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) g[i][j] = from[c * 9 + i * 3 + j];
        left_mul<M, UseL, n, 3, 3>(g, t);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            lg[c][j] = t[0][j];
#pragma unroll
            for (int i = 1; i < n; ++i)
                if (row == i) lg[c][j] = t[i][j];
        }
    }
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
