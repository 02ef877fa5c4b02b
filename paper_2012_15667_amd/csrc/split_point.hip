// 1 x 1 convolution (no padding), and the product step of unfused Winograd, on the 16-bit matrix cores at fp32 precision
// (operands in two fp16 parts, split_mfma.h): per group of images that share kernels y[K][HW] = w[K][C] x[C][HW], a
// transformed plane of Winograd being such a group of its own.
//
// A step is 32 channels.  The inputs of chunk t + 1 are split and written to one LDS buffer while chunk t is multiplied
// from the other; their loads are issued three chunks ahead and kept in registers, two neighbouring pixels per load where
// the layout has them.  Every pixel has a scale of its own: its image's largest value in the block, from the first 32 channels and a few more, but at
// most 512 times the largest of the pixel's own sample.  Sums are judged, and some computed again, as in direct_split.hip: those of a lane's
// four pixels together, or where these are of two images (a plane of 7 x 7 sub-domains) those of one with the pixels of the lane beside it.
// One to three alone are below their line so often that nearly every wave looked closer: product of 512 -> 512 at 14 x 14, batch 64, F(2 x 2)
// 113 us, with the lane beside it 103, without lines per kernel 91; all of 768 -> 192 at 17 x 17 35.1 and, without, 34.0.  The split's
// arithmetic is placed between the matrix instructions, three vector
// instructions after each, where it costs little (a 16-bit matrix instruction leaves the vector pipeline free; measured:
// eight vector instructions per 32-cycle matrix instruction 1433 against 1631 TFLOP/s).  wt is not declared restrict on
// purpose: loads of memory known not to change were moved down past the barrier to their use, which undid the prefetch.
//
// What bounds it: operands on their way in, about 20 bytes per clock and compute unit (a block of z channels by npix pixels needs
// 128 z + 128 npix bytes per 32 channels), and the latency of small layers' steps.  16 planes of 512 x 12544 x 512 (F(2x2)), 256 x 64
// blocks: 840 us on the fp32 instructions, 541 in three bf16 parts, 396 = 266 TFLOP/s in two fp16 parts.  1 x 1, 768 -> 192 at 17 x 17,
// batch 64, whole call: 66, 43.4, 35.6 us; 320 -> 224 at 170 x 170, batch 22 578 -> 454.  Zero pixels that each looked for their image's
// largest value cost 12 us of the 17 x 17 layer: now a wave does it once.
// Measured with three parts and taken back: the weights of chunk t + 2 loaded before the inputs of chunk t + 3, so that these have two steps
// to arrive (the same product 545 -> 573 us).
//
// A column of a wave's 16 x 16 blocks is 16 pixels; block nb of the wave takes every NB-th pixel from nb on (VPX), so that a
// lane holds NB neighbours of each output channel and stores them at once.
#include "kernels.h"
#include "split_mfma.h"
#include "split_weights.h"

#include <type_traits>

namespace iolb {

namespace {

template <int MB, int NB, int WM, int WN, int IN, bool VPX>
__global__ void __launch_bounds__(64 * WM * WN, 2)
split_point_kernel(const float* __restrict__ x, const u32x4* wt, float* y, SplitPointGeom g, const float* __restrict__ w, Divisor by_per)
{
    constexpr int T = 64 * WM * WN, NPIX = 16 * NB * WN, PLANE = 4 * NPIX * 16, BUF = 2 * PLANE;
    // an input item: CH channels of PX neighbouring pixels
    constexpr int PX = split_point_pixels(IN), CH = IN == SPLIT_IN_PIXELS ? 4 : 8;
    constexpr int ITEMS = 32 / CH * NPIX / PX, IB = (ITEMS + T - 1) / T;
    extern __shared__ u32x4 lds16[];
    // two buffers, each the h of all pixels and then the l; room that nobody reads; per pixel the largest value in the sample that sets
    // its scale, and of all its channels, scaled, and that of its image; its scale; what undoes the kernels' scales;
    // shares of their facts, then their lines
    char* const lds = reinterpret_cast<char*>(lds16);
    unsigned* const sample = reinterpret_cast<unsigned*>(lds + 2 * BUF + PLANE + 16);
    unsigned* const most = sample + NPIX;
    unsigned* const images = most + NPIX;
    unsigned* const scales = images + NPIX;
    float* const kback = reinterpret_cast<float*>(scales + NPIX);
    KernelFacts* const shares = reinterpret_cast<KernelFacts*>(kback + 16 * MB * WM);
    KernelLine* const lines = reinterpret_cast<KernelLine*>(shares);
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
    // images that have a scale of their own: which of them, in the block, a pixel is of (of a transformed plane g.HW is all of the batch)
    const int i0 = __builtin_amdgcn_readfirstlane(pix0 % g.per);
    const bool two_images = g.per >= NPIX, one_image = i0 + NPIX <= g.per;
    auto image_in = [&](int px) {
        const int one = i0 + px >= g.per, any = by_per.of(i0 + px);
        return two_images ? one : any;
    };

    const size_t image_floats = (size_t)g.C * g.HWin;
    const int span = __builtin_amdgcn_readfirstlane((p0 + NPIX - 1) / g.HW + 1);              // images the block touches
    const int have = (group + 1) * g.images - n0;
    const unsigned long long xbase = reinterpret_cast<unsigned long long>(x + (size_t)n0 * image_floats);
    // (the builtin returns a signed int: the halves have to be unsigned before they are put together)
    const unsigned xlo = __builtin_amdgcn_readfirstlane((unsigned)xbase), xhi = __builtin_amdgcn_readfirstlane((unsigned)(xbase >> 32));
    const unsigned range = __builtin_amdgcn_readfirstlane((unsigned)(4 * image_floats * (span < have ? span : have)));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>((unsigned long long)xhi << 32 | xlo), 0, (int)range, 0x00020000);

    // the input items of this thread
    // Column l16 of a wave's block nb is pixel 16 nb + l16, or NB l16 + nb (VPX): pixels are kept in LDS in the order in which
    // the blocks read them.  Pairs of pixels are then written with half the bank conflicts (16 bytes from lane to lane, not 32).
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
            dst[i] = (unsigned)(16 * (c_in[i] / 8 * NPIX + slot_of(px)) + (c_in[i] & 4) * 2);
            if (px < left_px) {
                const int q = p0 + px, im = q / g.HW, r = q % g.HW;
                const int in = g.stride == 1 ? r : r / g.Q * g.stride * g.Win + r % g.Q * g.stride;
                src[i] = g.hwc ? 4u * (unsigned)((im * g.HWin + in) * g.C + c_in[i]) : 4u * (unsigned)((im * g.C + c_in[i]) * g.HWin + in);
            }
        }
    }
    const int cstep = g.hwc ? 4 : 4 * g.HWin;
    constexpr int NEXT_PX = VPX ? 16 * 16 : 16;             // LDS bytes from a pixel to the next of its item

    f32x4 acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nchunks = (g.C + 31) >> 5;
    const int kb16 = kb * (MB * WM) + wm_i * MB;
    const size_t wstep = (size_t)g.Kb16 * 128;
    const u32x4* const group_w = wt + (size_t)group * g.w_image;
    const u32x4* wp = group_w + (size_t)kb16 * 128 + lane;

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
    float scale[IB][PX], top[IB][PX];                       // of the items' pixels: the scale; the largest value so far, scaled
    auto write_x = [&](const float (&v)[IB][CH * PX], char* buf) {
#pragma unroll
        for (int i = 0; i < IB; ++i) {
            char* d = (dst[i] == 2 * BUF ? lds : buf) + dst[i];
            if constexpr (CH == 8) {
                u32x4 h, l;
                top[i][0] = __builtin_fmaxf(top[i][0], half_eight(v[i], scale[i][0], h, l));
                *reinterpret_cast<u32x4*>(d) = h;
                *reinterpret_cast<u32x4*>(d + PLANE) = l;
            } else {
#pragma unroll
                for (int p = 0; p < PX; ++p) {
                    u32x2 h, l;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const float a = v[i][p * 4 + 2 * j] * scale[i][p], b = v[i][p * 4 + 2 * j + 1] * scale[i][p];
                        unsigned hj, lj;
                        half_pair(a, b, hj, lj);
                        h[j] = hj; l[j] = lj;
                        top[i][p] = __builtin_fmaxf(__builtin_fmaxf(top[i][p], __builtin_fabsf(a)), __builtin_fabsf(b));
                    }
                    // (an item that does not exist writes all its pixels to the same spare place)
                    char* dp = d + (dst[i] == 2 * BUF ? 0 : NEXT_PX * p);
                    *reinterpret_cast<u32x2*>(dp) = h;
                    *reinterpret_cast<u32x2*>(dp + PLANE) = l;
                }
            }
        }
    };
    auto load_a = [&](u32x4 (&a)[MB * 2]) {
#pragma unroll
        for (int j = 0; j < MB * 2; ++j) a[j] = wp[j * 64];
    };
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    const char* const mine = lds + 16 * (grp * NPIX + wn_i * NB * 16 + l16);
    u32x4 bf[2][2];
    auto fetch = [&](u32x4 (&f)[2], const char* from) {
        f[0] = *reinterpret_cast<const u32x4*>(from);
        f[1] = *reinterpret_cast<const u32x4*>(from + PLANE);
    };

    u32x4 a0[MB * 2], a1[MB * 2];
    load_x(xv[0], 0);
    // for the sample beside the first 32 channels one more value per item, from the others
    float spread[IB];
#pragma unroll
    for (int i = 0; i < IB; ++i) {
        const int c = 32 * (int)((unsigned)(37 * (i * T + tid) & 63) * (unsigned)nchunks >> 6);
        spread[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, src[i] != OUTSIDE && c + c_in[i] < g.C ? (int)(src[i] + (unsigned)c * (unsigned)cstep) : (int)OUTSIDE, 0, 0));
    }
    static_assert(16 * MB * WM <= T && 3 * NPIX <= T, "one kernel, one of the pixels' three values per thread");
    float my_kback = 0.f;
    constexpr int Z = 16 * MB * WM;
    const float* const group_scales = reinterpret_cast<const float*>(group_w + (size_t)nchunks * wstep);
    if (tid < Z) my_kback = group_scales[kb * Z + tid];
    // Blocks of several images whose lanes hold pixels of more than one judge single sums, by each kernel's own line (which others ask for
    // only where one for all kernels does not do).
    const bool of_one_image = i0 + (left_px < NPIX ? (int)left_px : NPIX) <= g.per, lane_of_one = of_one_image || (VPX && g.per % NB == 0);
    FactsShare<16> share;
    if (!lane_of_one) share.load(reinterpret_cast<const KernelFacts*>(group_scales + 16 * g.Kb16) + kb * Z + tid % Z, tid / Z, T / Z, g.pieces, 16 * g.Kb16);
    load_x(xv[1], 1);
    load_a(a0);
    if (tid < 3 * NPIX) sample[tid] = 0;                    // (most and images follow)
    __builtin_amdgcn_sched_barrier(0);
    barrier();
    // A pixel's scale follows from the largest value of its image's pixels in the block (a few channels of sparse data say little about the
    // others), but is at most 512 times its own (so that it is never too small for it).  Other images do not change its outputs.
    auto item_px = [&](int i) { return (i * T + tid) % (NPIX / PX) * PX; };
    auto exists = [&](int i) { return i * T + tid < ITEMS; };
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int p = 0; p < PX; ++p) {
            unsigned m = p == 0 ? finite_bits(spread[i]) : 0u;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const unsigned a = finite_bits(xv[0][i][p * CH + j]);
                m = a > m ? a : m;
            }
            if (exists(i) && m && item_px(i) + p < left_px) atomicMax(sample + item_px(i) + p, m);
        }
    if (tid < Z) kback[tid] = my_kback;
    if (!lane_of_one && tid < T / Z * Z) shares[tid] = share.sum();
    barrier();
    static_assert(NPIX <= 64, "a lane per pixel");
    if (!lane_of_one && tid < Z) lines[tid] = kernel_line(all_shares<Z, T / Z>(shares, tid));
    unsigned all = 0;
    if (one_image) {
        all = wave_max(lane < NPIX ? sample[lane] : 0u);
    } else {
        if (tid < NPIX && tid < left_px) atomicMax(images + image_in(tid), sample[tid]);
        barrier();
    }
    auto scale_of = [&](int px) {
        const unsigned m = sample[px], image = one_image ? all : images[image_in(px)];
        // (bits of floats: 3 << 23 less is an eighth, 9 << 23 more is 512 times)
        const unsigned eighth = image < 4u << 23 ? 0u : image - (3u << 23), most_m = m + (9u << 23);
        return half_scale_bits(m == 0 ? eighth : image < m ? m : image < most_m ? image : most_m);
    };
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int p = 0; p < PX; ++p) {
            const unsigned bits = scale_of(item_px(i) + p);
            scale[i][p] = __uint_as_float(bits);
            if (exists(i)) scales[item_px(i) + p] = bits;       // (the same from every channel's items)
            top[i][p] = 0.f;
        }
    __builtin_amdgcn_sched_barrier(0);
    write_x(xv[0], lds);
    load_x(xv[0], 2);
    __builtin_amdgcn_sched_barrier(0);
    barrier();
    fetch(bf[0], mine);

    // One step = 32 channels.  While chunk t is multiplied, chunk t + 1 is split into its parts (its loads were
    // issued two steps ago) and written to the other buffer, and the loads of chunk t + 3 are issued.
    auto step = [&](int t, u32x4 (&a)[MB * 2], u32x4 (&an)[MB * 2], float (&v)[IB][CH * PX]) {
        if (t + 1 < nchunks) wp += wstep;
        load_a(an);
        const char* cur = mine + (t & 1) * BUF;
        auto block = [&](auto nb_c) {
            constexpr int nb = decltype(nb_c)::value;
            if constexpr (nb + 1 < NB) fetch(bf[(nb + 1) & 1], cur + 16 * 16 * (nb + 1));
            constexpr int PA[3] = {1, 0, 0}, PB[3] = {0, 1, 0};      // small products first
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                        __builtin_bit_cast(f16x8, a[mb * 2 + PA[q]]), __builtin_bit_cast(f16x8, bf[nb & 1][PB[q]]), acc[mb][nb], 0, 0, 0);
        };
        constexpr int HALF = NB / 2;
        static_range<0, HALF>(block);
        __builtin_amdgcn_sched_barrier(0);
        write_x(v, lds + ((t + 1) & 1) * BUF);
        static_range<HALF, NB>(block);
        // the arithmetic of the split runs in the shadow of the matrix instructions
#pragma unroll
        for (int i = 0; i < (NB - HALF) * 3 * MB; ++i) {
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
    // pixel l16.  Where all sums are finite, no pixel is too small for its scale and no kernel's sums are too small, they are only
    // written; otherwise outputs for which that is not so are marked, and written a second time.
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int p = 0; p < PX; ++p)
            if (exists(i)) atomicMax(most + item_px(i) + p, __float_as_uint(top[i][p]));
    barrier();
    unsigned long long again = 0;
    static_assert(MB * NB * 4 <= 64, "one mark per output");
    float back[NB], inputs[NB];
    f32x4 kb4[MB];
    bool bad = false;
    const float all_norm = HALF_LINE * __builtin_amdgcn_sqrtf(g.pieces * (g.raw == SPLIT_RAW_ROWS ? HALF_PIECE : HALF_PIECE_PLANE)), all_root = HALF_LINE * __builtin_amdgcn_sqrtf((float)g.C);
    auto kernel_exists = [&](int mb, int i) { return (kb16 + mb) * 16 + 4 * grp + i < g.K; };
    const bool whole = left_px >= NPIX;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int px = pixel_of(nb, l16);
        back[nb] = half_unscale(scales[px]);
        inputs[nb] = px < left_px ? __uint_as_float(most[px]) : 0.f;
        bad |= __float_as_uint(inputs[nb]) - 1 < __float_as_uint(HALF_LEAST) - 1;
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) kb4[mb] = *reinterpret_cast<const f32x4*>(kback + (wm_i * MB + mb) * 16 + 4 * grp);
    // Nearly always a lane's pixels are judged together, or where they are of several images each by itself, and all is well.  (This way lies by
    // itself: instructions come from memory here.  The last block of an image, whose last lanes have few pixels, judges those of 16 lanes.)
    auto all_well = [&](auto closer_c) {
        constexpr bool CLOSER = decltype(closer_c)::value;
        auto line_at = [&](int mb, int i, float input) {
            return CLOSER ? line_of(lines[(wm_i * MB + mb) * 16 + 4 * grp + i], input) : all_norm + all_root * input;
        };
        if (__builtin_expect(VPX | of_one_image, 1)) {
            bool other = bad, apart = false;                // apart: pixels of two images
            float input = 0.f;
            const float first = of_one_image & !whole ? __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(back[0]))) : back[0];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                input = __builtin_fmaxf(input, inputs[nb]);
                other |= (back[nb] != first) & (pixel_of(nb, l16) < left_px);
            }
            if (of_one_image & !whole) input = row_largest(input);
            // (fewer than four: with the three lanes beside it, as below; all of one scale, then)
            const int mine = of_one_image ? 0 : image_in(pixel_of(0, l16));
            if (NB < 4 && lane_of_one) {
                const bool there = pixel_of(0, l16) < left_px;
                other |= there & (quad_largest(there ? back[0] : 0.f, mine) != back[0]);
                input = quad_largest(input, mine);
            }
            // (a lane of two images: each one's pixels, and those of the lanes beside it; of more, single ones)
            bool of_first[NB], of_last[NB], before = false, after = false;
            if (!lane_of_one) {
                const bool two = g.per >= NB - 1;
                other = bad;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const bool there = pixel_of(nb, l16) < left_px;
                    of_first[nb] = there & (two ? image_in(pixel_of(nb, l16)) == image_in(pixel_of(0, l16)) : nb == 0);
                    of_last[nb] = there & !of_first[nb];
                    other |= (of_first[nb] & (back[nb] != back[0])) | (of_last[nb] & (back[nb] != back[NB - 1])) | (!two & (nb > 0) & (nb + 1 < NB) & there);
                    apart |= of_last[nb];
                }
                before = apart & (l16 > 0) & (image_in(pixel_of(0, l16) - 1) == image_in(pixel_of(0, l16)));
                after = apart & (l16 < 15) & (pixel_of(NB, l16) < left_px) & (image_in(pixel_of(NB, l16)) == image_in(pixel_of(NB - 1, l16)));
                const float there[4] = {lane_before(back[NB - 1]), lane_after(back[0]), lane_before(input), lane_after(input)};
                before &= there[0] == back[0];
                after &= there[1] == back[NB - 1];
                if (before) input = __builtin_fmaxf(input, there[2]);
                if (after) input = __builtin_fmaxf(input, there[3]);
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float m = 0.f;
                    if (lane_of_one & whole) {
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) m = __builtin_elementwise_maximum(m, __builtin_fabsf(acc[mb][nb][i]));
                        if (NB < 4) m = quad_largest(m, mine);
                        other |= !(m <= FINITE);
                    } else if (lane_of_one) {
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) m = __builtin_elementwise_maximum(m, pixel_of(nb, l16) < left_px ? __builtin_fabsf(acc[mb][nb][i]) : 0.f);
                        if (NB < 4) m = quad_largest(m, mine);
                        if (of_one_image) m = row_largest(m);
                        other |= !(m <= FINITE);
                    } else {
                        float last = 0.f;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) {
                            m = __builtin_elementwise_maximum(m, of_first[nb] ? __builtin_fabsf(acc[mb][nb][i]) : 0.f);
                            last = __builtin_elementwise_maximum(last, of_last[nb] ? __builtin_fabsf(acc[mb][nb][i]) : 0.f);
                        }
                        other |= !(m <= FINITE) | !(last <= FINITE);
                        const float from = lane_before(apart ? last : m), to = lane_after(m);
                        if (before) m = __builtin_elementwise_maximum(m, from);
                        if (after) last = __builtin_elementwise_maximum(last, to);
                        m = apart && last < m ? last : m;
                    }
                    other |= !(m >= line_at(mb, i, input)) & kernel_exists(mb, i) & (input > 0.f);
                }
            return __builtin_amdgcn_ballot_w64(other) == 0;
        } else if constexpr (!VPX) {
            bool other = bad, same[NB][NB];
            float input = 0.f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                input = __builtin_fmaxf(input, inputs[nb]);
#pragma unroll
                for (int o = 0; o < NB; ++o) {
                    same[nb][o] = (image_in(pixel_of(o, l16)) == image_in(pixel_of(nb, l16))) & (pixel_of(o, l16) < left_px);
                    other |= (back[nb] != back[o]) & same[nb][o];
                }
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float line = line_at(mb, i, input);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        float m = 0.f;
#pragma unroll
                        for (int o = 0; o < NB; ++o) m = __builtin_elementwise_maximum(m, same[nb][o] ? __builtin_fabsf(acc[mb][o][i]) : 0.f);
                        other |= ((!(m >= line) & kernel_exists(mb, i) & (inputs[nb] > 0.f)) | !(m <= FINITE)) & same[nb][nb];
                    }
                }
            return __builtin_amdgcn_ballot_w64(other) == 0;
        } else {
            return false;
        }
    };
    bool fine = lane_of_one ? all_well(std::false_type{}) : false;
    if (__builtin_expect(!fine, 0)) {
        if (lane_of_one) wave_lines<MB>(reinterpret_cast<const KernelFacts*>(group_scales + 16 * g.Kb16) + kb16 * 16, g.pieces, 16 * g.Kb16, lane, lines + wm_i * (16 * MB));
        fine = all_well(std::true_type{});
    }
    if (__builtin_expect(!fine, 0)) {
    int image[NB];
    float size[NB];
    const bool ragged = of_one_image && !whole;
    const int judging = lane_of_one ? JUDGE_LANE : JUDGE_MIXED;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const bool there = pixel_of(nb, l16) < left_px;
        image[nb] = there ? image_in(pixel_of(nb, l16)) : -1;
        size[nb] = there ? back[nb] : 0.f;
    }
    // Pixels that are judged together have scales of their own: size, a pixel's against that of the brightest of them (0: no output).  The
    // largest input of them, by that scale, makes the line; where all are zero there is none.
    Joins joins = {};
    auto of_group = [&](const float (&v)[NB], float (&to)[NB]) {
        float all = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) all = __builtin_fmaxf(all, v[nb]);
        if (NB < 4) all = quad_largest(all, of_one_image ? 0 : image[0]);
        if (ragged) all = row_largest(all);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float mine = all;
            if (judging == JUDGE_MIXED) {
                mine = 0.f;
#pragma unroll
                for (int other = 0; other < NB; ++other) mine = image[other] == image[nb] ? __builtin_fmaxf(mine, v[other]) : mine;
            }
            to[nb] = mine;
        }
        if (judging == JUDGE_MIXED) {
            const float before = lane_before(to[NB - 1]), after = lane_after(to[0]);
#pragma unroll
            for (int nb = NB - 1; nb >= 0; --nb) {
                if (joins.before & (image[nb] == image[0])) to[nb] = __builtin_fmaxf(to[nb], before);
                if (joins.after & (image[nb] == image[NB - 1])) to[nb] = __builtin_fmaxf(to[nb], after);
            }
        }
    };
    bool lost[NB], zero[NB];
    {
        float brightest[NB];
        of_group(size, brightest);
        if (VPX && judging == JUDGE_MIXED) {
            const int l16 = opaque(lane) & 15, px0 = pixel_of(0, l16), px1 = pixel_of(NB, l16);
            const float before = lane_before(brightest[NB - 1]), after = lane_after(brightest[0]);
            const bool apart = image[NB - 1] != image[0];
            joins.before = apart & (l16 > 0) & (image[0] >= 0) & (before == brightest[0]) && image_in(px0 - 1) == image[0];
            joins.after = apart & (l16 < 15) & (px1 < left_px) & (after == brightest[NB - 1]) && image_in(px1) == image[NB - 1];
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            lost[nb] = __float_as_uint(inputs[nb]) - 1 < __float_as_uint(HALF_LEAST) - 1;
            zero[nb] = inputs[nb] == 0.f;
            size[nb] = size[nb] > 0.f ? size[nb] * half_unscale(__float_as_uint(brightest[nb])) : 0.f;      // (powers of two)
            inputs[nb] *= size[nb];
        }
        float largest[NB];
        of_group(inputs, largest);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) inputs[nb] = largest[nb];
    }
    // otherwise each output for itself; zero inputs have lost nothing
    {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (image[nb] >= 0 && (lost[nb] || !(__builtin_fabsf(acc[mb][nb][i]) <= FINITE)) && (kb16 + mb) * 16 + 4 * (opaque(lane) >> 4) + i < g.K)
                        again |= 1ull << ((nb * MB + mb) * 4 + i);
        unsigned group = 0;                                 // bits of the nb that are judged together
        judge_sums<MB, NB>(judging, ragged, image, 0, !of_one_image,
                           [&](int mb, int nb, int i) { return __builtin_fabsf(acc[mb][nb][i]) <= FINITE ? __builtin_fabsf(acc[mb][nb][i]) * size[nb] : 0.f; },
                           [&](auto in) {
                               group = 0;
#pragma unroll
                               for (int nb = 0; nb < NB; ++nb) group |= in(nb) && !zero[nb] ? 1u << nb : 0u;
                           },
                           [&](int mb, int i, float m) {
                               const int k = 4 * (opaque(lane) >> 4) + i;
                               if ((kb16 + mb) * 16 + k >= g.K) return;
                               const KernelLine line = lines[(wm_i * MB + mb) * 16 + k];
#pragma unroll
                               for (int nb = 0; nb < NB; ++nb)
                                   if ((group >> nb & 1) & !(m >= line_of(line, inputs[nb]))) again |= 1ull << ((nb * MB + mb) * 4 + i);
                           },
                           joins);
    }
    }
    // all of them; the second time those that were marked
    auto write_y = [&](auto marked_c) {
        constexpr bool MARKED = decltype(marked_c)::value;
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
                    for (int nb = 0; nb < NB; ++nb) q[nb] = acc[mb][nb][i] * back[nb] * kb4[mb][i];
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
                if constexpr (!MARKED) acc[mb][nb] = acc[mb][nb] * back[nb] * kb4[mb];
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
    if (__builtin_expect(fine || __builtin_amdgcn_ballot_w64(again != 0) == 0, 1)) return;

    // Few marked outputs of an image are sums of their own, a lane one channel in 64 (image by image: what others hold decides nothing).
    const RawKernels raw(w, g.raw, g.m, group, g.C, g.K);
    {
        constexpr int FEW = 16;
        unsigned long long many = 0;
        while (const unsigned long long lanes = __builtin_amdgcn_ballot_w64(again != 0)) {
            const int src = __builtin_ctzll(lanes);
            const int nb0 = __builtin_amdgcn_readlane((int)(__builtin_ctzll(again | 1ull << 63) / (4 * MB)), src);
            const int im = image_in(pixel_of(nb0, src & 15));
            unsigned long long own = 0;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) own |= image_in(pixel_of(nb, opaque(lane) & 15)) == im ? again & (((1ull << (4 * MB - 1) << 1) - 1) << (nb * MB * 4)) : 0;
            again &= ~own;
            if (wave_sum((float)__popcll(own)) > FEW) { many |= own; continue; }
            while (const unsigned long long left = __builtin_amdgcn_ballot_w64(own != 0)) {
                const int at = __builtin_ctzll(left);
                const int bit = __builtin_amdgcn_readlane(__builtin_ctzll(own | 1ull << 63), at);
                if (lane == at) own &= own - 1;
                const int k = (kb16 + bit / 4 % MB) * 16 + 4 * (at >> 4) + (bit & 3), q = p0 + pixel_of(bit / (4 * MB), at & 15), r = q % g.HW;
                const size_t n = n0 + q / g.HW, in = g.stride == 1 ? r : r / g.Q * g.stride * g.Win + r % g.Q * g.stride;
                const float* xp = x + n * image_floats + (g.hwc ? in * g.C : in);
                float sum = 0.f;
                // (eight loads at a time: their latency is what this costs)
#pragma unroll 1
                for (int c0 = lane; c0 < g.C; c0 += 8 * 64) {
                    float v[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) v[j] = xp[(size_t)(c0 + 64 * j < g.C ? c0 + 64 * j : 0) * (cstep / 4)];
#pragma unroll
                    for (int j = 0; j < 8; ++j) sum = __builtin_fmaf(c0 + 64 * j < g.C ? v[j] : 0.f, raw.at(k, c0 + 64 * j), sum);
                }
                sum = wave_sum(sum);
                if (lane == at) y[g.hwc ? (n * g.HW + r) * g.K + k : (n * g.Ky + k) * g.HWy + r] = sum;
            }
        }
        again = many;
        if (__builtin_amdgcn_ballot_w64(again != 0) == 0) return;
    }

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
#pragma unroll 1
    for (int ch = 0; ch < nchunks; ++ch) {
        float wv[MB][8];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < 8; ++j) wv[mb][j] = raw.at((kb16 + mb) * 16 + col16, 32 * ch + c0 + j);
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
hipError_t launch_one(const float* x, const u32x4* wt, const float* w, float* y, const SplitPointGeom& g, hipStream_t st)
{
    auto kern = split_point_kernel<MB, NB, WM, WN, IN, VPX>;
    constexpr size_t NPIX = 16 * NB * WN, shm = 5 * 4 * NPIX * 16 + 16 + 16 * NPIX + 64 * MB * WM + 512 * WM * WN;
    static_assert(shm <= 64 * 1024, "dynamic LDS without an opt-in");
    hipLaunchKernelGGL(kern, dim3(g.nbk * g.nbp * g.groups), dim3(64 * WM * WN), shm, st, x, wt, y, g, w, Divisor(g.per));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_split_point(const float* x, const void* wt, const float* w_given, float* y, const SplitPointGeom& g, hipStream_t st)
{
    // what the kernel assumes of its geometry
    const long long npix = 16LL * g.nb * g.wn, span = (g.HW - 1 + npix - 1) / g.HW + 1;
    if (g.Kb16 != g.nbk * g.mb * g.wm || (long long)g.nbp * npix < (long long)g.images * g.HW || (long long)g.images * g.HW >= (1LL << 31) - 1024 ||
        4 * (span < g.images ? span : g.images) * g.C * g.HWin >= (1LL << 31) || g.Kb16 * 16 < g.K ||
        (long long)g.nbk * g.nbp * g.groups > 0x7fffffffLL || g.per < 1 || g.pieces < 1)
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
        if (g.in == SPLIT_IN_CHANNELS) return launch_one<M_, N_, A_, B_, SPLIT_IN_CHANNELS, false>(x, w, w_given, y, g, st);  \
        if (g.in == SPLIT_IN_PIXELS)                                                                                 \
            return vec ? launch_one<M_, N_, A_, B_, SPLIT_IN_PIXELS, true>(x, w, w_given, y, g, st)                           \
                       : launch_one<M_, N_, A_, B_, SPLIT_IN_PIXELS, false>(x, w, w_given, y, g, st);                         \
        return vec ? launch_one<M_, N_, A_, B_, SPLIT_IN_SINGLE, true>(x, w, w_given, y, g, st)                               \
                   : launch_one<M_, N_, A_, B_, SPLIT_IN_SINGLE, false>(x, w, w_given, y, g, st);                             \
    }
    IOLB_SPLIT_POINT_SHAPES(IOLB_POINT_CASE)
#undef IOLB_POINT_CASE
    return hipErrorInvalidValue;
}

}  // namespace iolb
