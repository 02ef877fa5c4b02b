// 1 x 1 convolution (no padding), and the product step of unfused Winograd, on the bf16 matrix cores at fp32 precision
// (operands in three parts, split_mfma.h): per group of images that share kernels y[K][HW] = w[K][C] x[C][HW], a
// transformed plane of Winograd being such a group of its own.
//
// A step is 32 channels.  The inputs of chunk t + 1 are split and written to one LDS buffer while chunk t is multiplied
// from the other; their loads are issued three chunks ahead and kept in registers, two neighbouring pixels per load where
// the layout has them.  The split's arithmetic is placed between the matrix instructions, three vector
// instructions after each, where it costs little (a bf16 matrix instruction leaves the vector pipeline free; measured:
// eight vector instructions per 32-cycle matrix instruction 1433 against 1631 TFLOP/s).  wt is not declared restrict on
// purpose: loads of memory known not to change were moved down past the barrier to their use, which undid the prefetch.
//
// What bounds it: of large products nothing found yet. Matrix cores are busy 0.57 of the cycles; a compute unit takes in 20 bytes
// of operands per clock (6.05 GB through the L2s in 1.15 M clocks on the product below; a block of z channels by npix pixels
// needs 192 z + 128 npix bytes per 32 channels), while other kernels take 24 to 36 through the same L2s; the vector work of the split
// costs clock. 16 planes of 512 x 12544 x 512 (F(2x2)) 545 us = 193 TFLOP/s with 256 x 64 blocks (fp32 instructions: 840 us; with
// single stores 580), larger blocks were slower.  Small ones the latency of their steps.  1 x 1, 768 -> 192 at 17 x 17, batch 64,
// whole call: 66 us on the fp32 instructions, 46.4 with single stores, 43.5.
// Measured and taken back: the weights of chunk t + 2 loaded before the inputs of chunk t + 3, so that these have two steps
// to arrive (the same product 545 -> 573 us).
//
// A column of a wave's 16 x 16 blocks is 16 pixels; block nb of the wave takes every NB-th pixel from nb on (VPX), so that a
// lane holds NB neighbours of each output channel and stores them at once.
#include "kernels.h"
#include "split_mfma.h"

#include <type_traits>

namespace iolb {

namespace {

template <int MB, int NB, int WM, int WN, int IN, bool VPX>
__global__ void __launch_bounds__(64 * WM * WN, 2)
split_point_kernel(const float* __restrict__ x, const u32x4* wt, float* y, SplitPointGeom g)
{
    constexpr int T = 64 * WM * WN, NPIX = 16 * NB * WN, BUF = 4 * NPIX * 48;
    // an input item: CH channels of PX neighbouring pixels
    constexpr int PX = split_point_pixels(IN), CH = IN == SPLIT_IN_PIXELS ? 4 : 8;
    constexpr int ITEMS = 32 / CH * NPIX / PX, IB = (ITEMS + T - 1) / T;
    extern __shared__ u32x4 lds16[];
    char* const lds = reinterpret_cast<char*>(lds16);       // two buffers, then 48 bytes that nobody reads
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm_i = wave % WM, wn_i = wave / WM;

    int bid;
    {
        const int nblk = gridDim.x, q = nblk >> 3, r = nblk & 7, xcd = blockIdx.x & 7;
        bid = xcd * q + (xcd < r ? xcd : r) + ((int)blockIdx.x >> 3);
    }
    const int kb = __builtin_amdgcn_readfirstlane(bid % g.nbk); bid /= g.nbk;
    const int group = __builtin_amdgcn_readfirstlane(bid / g.nbp);        // images that share kernels
    const int pix0 = __builtin_amdgcn_readfirstlane(bid % g.nbp) * NPIX;  // first pixel, in the group's images one after the other
    const int n0 = group * g.images + __builtin_amdgcn_readfirstlane(pix0 / g.HW);
    const int p0 = __builtin_amdgcn_readfirstlane(pix0 % g.HW);           // ... in image n0
    const long long left_px = (long long)g.images * g.HW - pix0;          // pixels of the group from there on

    const size_t image = (size_t)g.C * g.HWin;
    const int span = __builtin_amdgcn_readfirstlane((p0 + NPIX - 1) / g.HW + 1);              // images the block touches
    const int have = (group + 1) * g.images - n0;
    const unsigned long long xbase = reinterpret_cast<unsigned long long>(x + (size_t)n0 * image);
    // (the builtin returns a signed int: the halves have to be unsigned before they are put together)
    const unsigned xlo = __builtin_amdgcn_readfirstlane((unsigned)xbase), xhi = __builtin_amdgcn_readfirstlane((unsigned)(xbase >> 32));
    const unsigned range = __builtin_amdgcn_readfirstlane((unsigned)(4 * image * (span < have ? span : have)));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>((unsigned long long)xhi << 32 | xlo), 0, (int)range, 0x00020000);

    // the input items of this thread
    // Column l16 of a wave's block nb is pixel 16 nb + l16, or NB l16 + nb (VPX): pixels are kept in LDS in the order in which
    // the blocks read them.  Pairs of pixels are then written with half the bank conflicts (48 bytes from lane to lane, not 96).
    auto slot_of = [&](int px) { return VPX ? px / (16 * NB) * (16 * NB) + px % NB * 16 + px % (16 * NB) / NB : px; };
    auto pixel_of = [&](int nb, int l) { return wn_i * NB * 16 + (VPX ? NB * l + nb : 16 * nb + l); };
    unsigned src[IB], dst[IB];
    int c_in[IB];
#pragma unroll
    for (int i = 0; i < IB; ++i) {
        const int it = i * T + tid, px = it % (NPIX / PX) * PX;
        c_in[i] = it / (NPIX / PX) * CH;
        src[i] = OUTSIDE;
        dst[i] = 2 * BUF;
        if (it < ITEMS) {
            dst[i] = (unsigned)(48 * (c_in[i] / 8 * NPIX + slot_of(px)) + (c_in[i] & 4) * 2);
            if (px < left_px) {
                const int q = p0 + px, im = q / g.HW, r = q % g.HW;
                const int in = g.stride == 1 ? r : r / g.Q * g.stride * g.Win + r % g.Q * g.stride;
                src[i] = g.hwc ? 4u * (unsigned)((im * g.HWin + in) * g.C + c_in[i]) : 4u * (unsigned)((im * g.C + c_in[i]) * g.HWin + in);
            }
        }
    }
    const int cstep = g.hwc ? 4 : 4 * g.HWin;
    constexpr int NEXT_PX = VPX ? 48 * 16 : 48;             // LDS bytes from a pixel to the next of its item

    f32x4 acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nchunks = (g.C + 31) >> 5;
    const int kb16 = kb * (MB * WM) + wm_i * MB;
    const size_t wstep = (size_t)g.Kb16 * 192;
    const u32x4* wp = wt + (size_t)group * g.w_image + (size_t)kb16 * 192 + lane;

    float xv[2][IB][CH * PX];
    auto load_x = [&](float (&v)[IB][CH * PX], int ch) {
        const int c0 = ch < nchunks ? 32 * ch : 0, cl = ch < nchunks ? g.C - c0 : 0;
#pragma unroll
        for (int i = 0; i < IB; ++i) {
            const int some = cl - c_in[i];                  // channels of this item that exist
            if constexpr (IN == SPLIT_IN_CHANNELS) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rs, some > 4 * h ? (int)src[i] + 16 * h : (int)OUTSIDE, c0 * 4, 0);
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[i][4 * h + j] = __uint_as_float(q[j]);
                }
            } else {
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const int cj = c0 + j < g.C ? c0 + j : g.C - 1, at = some > j ? (int)src[i] : (int)OUTSIDE;
                    if constexpr (PX == 2) {
                        const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(rs, at, cj * cstep, 0);
                        v[i][j] = __uint_as_float(q[0]);
                        v[i][CH + j] = __uint_as_float(q[1]);
                    } else {
                        v[i][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, at, cj * cstep, 0));
                    }
                }
            }
        }
    };
    auto write_x = [&](const float (&v)[IB][CH * PX], char* buf) {
#pragma unroll
        for (int i = 0; i < IB; ++i) {
            char* d = (dst[i] == 2 * BUF ? lds : buf) + dst[i];
            if constexpr (CH == 8) {
                u32x4 h, m, l;
                split_eight(v[i], h, m, l);
                u32x4* d4 = reinterpret_cast<u32x4*>(d);
                d4[0] = h; d4[1] = m; d4[2] = l;
            } else {
#pragma unroll
                for (int p = 0; p < PX; ++p) {
                    u32x2 h, m, l;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        unsigned hj, mj, lj;
                        split_pair(v[i][p * 4 + 2 * j], v[i][p * 4 + 2 * j + 1], hj, mj, lj);
                        h[j] = hj; m[j] = mj; l[j] = lj;
                    }
                    // (an item that does not exist writes all its pixels to the same spare place)
                    char* dp = d + (dst[i] == 2 * BUF ? 0 : NEXT_PX * p);
                    *reinterpret_cast<u32x2*>(dp) = h;
                    *reinterpret_cast<u32x2*>(dp + 16) = m;
                    *reinterpret_cast<u32x2*>(dp + 32) = l;
                }
            }
        }
    };
    auto load_a = [&](u32x4 (&a)[MB * 3]) {
#pragma unroll
        for (int j = 0; j < MB * 3; ++j) a[j] = wp[j * 64];
    };
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    const char* const mine = lds + 48 * (grp * NPIX + wn_i * NB * 16 + l16);
    u32x4 bf[2][3];
    auto fetch = [&](u32x4 (&f)[3], const char* from) {
#pragma unroll
        for (int p = 0; p < 3; ++p) f[p] = *reinterpret_cast<const u32x4*>(from + 16 * p);
    };

    u32x4 a0[MB * 3], a1[MB * 3];
    load_x(xv[0], 0);
    load_x(xv[1], 1);
    load_a(a0);
    __builtin_amdgcn_sched_barrier(0);
    write_x(xv[0], lds);
    load_x(xv[0], 2);
    __builtin_amdgcn_sched_barrier(0);
    barrier();
    fetch(bf[0], mine);

    // One step = 32 channels.  While chunk t is multiplied, chunk t + 1 is split into its three parts (its loads were
    // issued two steps ago) and written to the other buffer, and the loads of chunk t + 3 are issued.
    auto step = [&](int t, u32x4 (&a)[MB * 3], u32x4 (&an)[MB * 3], float (&v)[IB][CH * PX]) {
        if (t + 1 < nchunks) wp += wstep;
        load_a(an);
        const char* cur = mine + (t & 1) * BUF;
        auto block = [&](auto nb_c) {
            constexpr int nb = decltype(nb_c)::value;
            if constexpr (nb + 1 < NB) fetch(bf[(nb + 1) & 1], cur + 48 * 16 * (nb + 1));
            constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};      // small products first
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, a[mb * 3 + PA[q]]), __builtin_bit_cast(bf16x8, bf[nb & 1][PB[q]]), acc[mb][nb], 0, 0, 0);
        };
        constexpr int HALF = NB / 2;
        static_range<0, HALF>(block);
        __builtin_amdgcn_sched_barrier(0);
        write_x(v, lds + ((t + 1) & 1) * BUF);
        static_range<HALF, NB>(block);
        // the arithmetic of the split runs in the shadow of the matrix instructions
#pragma unroll
        for (int i = 0; i < (NB - HALF) * 6 * MB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        load_x(v, t + 3);
        __builtin_amdgcn_sched_barrier(0);
        barrier();
        fetch(bf[0], mine + ((t + 1) & 1) * BUF);
    };
    for (int t = 0;;) {
        step(t, a0, a1, xv[1]);
        if (++t == nchunks) break;
        step(t, a1, a0, xv[0]);
        if (++t == nchunks) break;
    }

    // each partial sum is complete: write the block once.  Register i of a 16 x 16 block holds channel 4 grp + i of
    // pixel l16.  Sums that are not finite are marked.
    unsigned long long again = 0;
    static_assert(MB * NB * 4 <= 64, "one mark per output");
    auto write_y = [&](auto marked_c) {
        constexpr bool MARKED = decltype(marked_c)::value;  // the second time: marked outputs only
        const int l16 = opaque(lane) & 15, grp = opaque(lane) >> 4;
        if constexpr (VPX && !MARKED) {
            typedef float vec __attribute__((ext_vector_type(NB), aligned(4)));
            const int px = pixel_of(0, l16);                // ... and the next NB - 1
            if (px >= left_px) return;
            const int n = n0 + (p0 + px) / g.HW, r = (p0 + px) % g.HW;
            // at once where they lie in the row of y: beyond the image's pixels is its padding then
            const bool whole = r + NB <= g.HWy;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const int k0 = (kb16 + mb) * 16 + 4 * grp;
                float* yp = y + ((size_t)n * g.Ky + k0) * g.HWy + r;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    vec q;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        // (beyond the pixels that exist the inputs are what follows them: not a reason to do anything again)
                        if (px + nb < left_px && !(__builtin_fabsf(acc[mb][nb][i]) <= 3.402823466e38f)) again |= 1ull << ((nb * MB + mb) * 4 + i);
                        q[nb] = acc[mb][nb][i] * SPLIT_UNSCALE;
                    }
                    if (k0 + i >= g.K) continue;
                    if (whole) {
                        *reinterpret_cast<vec*>(yp + (size_t)i * g.HWy) = q;
                    } else {
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            if (px + nb < left_px) yp[(size_t)i * g.HWy + nb] = q[nb];
                    }
                }
            }
            return;
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int px = pixel_of(nb, l16);
            if (px >= left_px) continue;
            const int n = n0 + (p0 + px) / g.HW, r = (p0 + px) % g.HW;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const int k0 = (kb16 + mb) * 16 + 4 * grp, bit = (nb * MB + mb) * 4;
                if constexpr (!MARKED) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (!(__builtin_fabsf(acc[mb][nb][i]) <= 3.402823466e38f)) again |= 1ull << (bit + i);
                        acc[mb][nb][i] *= SPLIT_UNSCALE;
                    }
                }
                if (g.hwc) {
                    float* yp = y + ((size_t)n * g.HW + r) * g.K + k0;
                    if (!MARKED && g.vec_out && k0 + 3 < g.K) {
                        *reinterpret_cast<f32x4*>(yp) = acc[mb][nb];
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (k0 + i < g.K && (!MARKED || again >> (bit + i) & 1)) yp[i] = acc[mb][nb][i];
                    }
                } else {
                    float* yp = y + ((size_t)n * g.Ky + k0) * g.HWy + r;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (k0 + i < g.K && (!MARKED || again >> (bit + i) & 1)) yp[(size_t)i * g.HWy] = acc[mb][nb][i];
                }
            }
        }
    };
    write_y(std::false_type{});
    if (__builtin_amdgcn_ballot_w64(again != 0) == 0) return;

    // A wave with a marked output takes its whole block again on the fp32 matrix instructions, which hold their sums in
    // the same registers; the inputs come from memory.
    const int lane2 = opaque(lane), col16 = lane2 & 15, c0 = 8 * (lane2 >> 4);
    unsigned at[NB];                                        // this lane's pixels, first channel of its group
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int px = pixel_of(nb, col16), q = p0 + px, im = q / g.HW, r = q % g.HW;
        const int in = g.stride == 1 ? r : r / g.Q * g.stride * g.Win + r % g.Q * g.stride;
        at[nb] = px >= left_px ? OUTSIDE : g.hwc ? 4u * (unsigned)((im * g.HWin + in) * g.C + c0) : 4u * (unsigned)((im * g.C + c0) * g.HWin + in);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const u32x4* wq = wt + (size_t)group * g.w_image + (size_t)kb16 * 192 + lane2;
#pragma unroll 1
    for (int ch = 0; ch < nchunks; ++ch, wq += wstep) {
        float wv[MB][8];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) kept_eight(wq[mb * 192], wq[mb * 192 + 64], wq[mb * 192 + 128], wv[mb]);
        static_range<0, NB>([&](auto nb_c) {
            constexpr int nb = decltype(nb_c)::value;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = 32 * ch + j;                  // relative to the lane group's first
                v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                    rs, at[nb] != OUTSIDE && c + c0 < g.C ? (int)(at[nb] + c * (unsigned)cstep) : (int)OUTSIDE, 0, 0));
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[mb][j], v[j], acc[mb][nb], 0, 0, 0);
        });
    }
    write_y(std::true_type{});
}

template <int MB, int NB, int WM, int WN, int IN, bool VPX>
hipError_t launch_one(const float* x, const u32x4* wt, float* y, const SplitPointGeom& g, hipStream_t st)
{
    auto kern = split_point_kernel<MB, NB, WM, WN, IN, VPX>;
    constexpr size_t shm = 2 * 4 * 16 * NB * WN * 48 + 48;
    static_assert(shm <= 64 * 1024, "dynamic LDS without an opt-in");
    hipLaunchKernelGGL(kern, dim3(g.nbk * g.nbp * g.groups), dim3(64 * WM * WN), shm, st, x, wt, y, g);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_split_point(const float* x, const void* wt, float* y, const SplitPointGeom& g, hipStream_t st)
{
    // what the kernel assumes of its geometry
    const long long npix = 16LL * g.nb * g.wn, span = (g.HW - 1 + npix - 1) / g.HW + 1;
    if (g.Kb16 != g.nbk * g.mb * g.wm || (long long)g.nbp * npix < (long long)g.images * g.HW || (long long)g.images * g.HW >= (1LL << 31) - 1024 ||
        4 * (span < g.images ? span : g.images) * g.C * g.HWin >= (1LL << 31) || g.Kb16 * 16 < g.K ||
        (long long)g.nbk * g.nbp * g.groups > 0x7fffffffLL)
        return hipErrorInvalidValue;
    if (g.in == SPLIT_IN_CHANNELS && (!g.hwc || g.C % 4)) return hipErrorInvalidValue;
    if (g.in == SPLIT_IN_PIXELS && (g.hwc || g.stride != 1 || (g.images > 1 && g.HW % split_point_pixels(g.in)))) return hipErrorInvalidValue;
    const u32x4* w = static_cast<const u32x4*>(wt);
    // NB neighbouring pixels per lane (VPX) unless they can cross into another image.  16 planes of 512 x 12544 x 512: 580 ->
    // 545 us, 16 of 512 x 1024 x 512 47.9 -> 44.1, 64 images of 17 x 17, 768 -> 192: 46.1 -> 41.9; with the crossing groups
    // taken apart 64 images of 49 pixels, 512 -> 512, 19.7 -> 22.6, of 90 pixels 27.2 -> 29.4.
    const bool vec = !g.hwc && (g.images == 1 || g.HW % g.nb == 0);
#define IOLB_POINT_CASE(M_, N_, A_, B_)                                                                              \
    if (g.mb == M_ && g.nb == N_ && g.wm == A_ && g.wn == B_) {                                                      \
        if (g.in == SPLIT_IN_CHANNELS) return launch_one<M_, N_, A_, B_, SPLIT_IN_CHANNELS, false>(x, w, y, g, st);  \
        if (g.in == SPLIT_IN_PIXELS)                                                                                 \
            return vec ? launch_one<M_, N_, A_, B_, SPLIT_IN_PIXELS, true>(x, w, y, g, st)                           \
                       : launch_one<M_, N_, A_, B_, SPLIT_IN_PIXELS, false>(x, w, y, g, st);                         \
        return vec ? launch_one<M_, N_, A_, B_, SPLIT_IN_SINGLE, true>(x, w, y, g, st)                               \
                   : launch_one<M_, N_, A_, B_, SPLIT_IN_SINGLE, false>(x, w, y, g, st);                             \
    }
    IOLB_SPLIT_POINT_SHAPES(IOLB_POINT_CASE)
#undef IOLB_POINT_CASE
    return hipErrorInvalidValue;
}

}  // namespace iolb
