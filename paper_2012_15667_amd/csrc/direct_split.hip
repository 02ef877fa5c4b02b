// Direct convolution on the 16-bit matrix cores at fp32 precision (operands in two fp16 parts, of few channels and small layers in
// three of bf16: split_mfma.h), dataflow of Sec. 5.2: a workgroup keeps the partial sums of b images * ty rows * tx columns by 16 MB WM output channels in
// registers for the whole channel loop and writes them once.
//
// The channel loop runs in chunks of 8, 16 or 32 channels (8 ch8).  Of a chunk the input tile is in LDS, per pixel and
// group of eight channels 16 bytes per part (two parts in planes of their own, three one after the other), in two buffers: while one chunk is multiplied the next
// is loaded to registers, split and written to the other buffer, a batch of items per matrix step, with one barrier
// per chunk.  A matrix step contracts four units of (tap, eight channels) in one v_mfma_f32_16x16x32 per product
// of parts: the four lane groups of the instruction read the window pixel of their own unit, whose LDS offset comes
// from a table, so one kernel serves every kernel extent, stride and padding.  Sixteen lanes read 16 bytes each 16 or 48
// bytes apart: every LDS bank once.  With a stride the columns are stored by residue class, so that this holds there too.
// The weights (split once per call, in the order of the steps) go from the L2 straight into registers: each wave has
// channels of its own, so through LDS they would only be written and read once more.
//
// Two parts: the scales (split_mfma.h) are of a kernel, and of an image in a block, from a sample of its first loads and 64 values
// spread over the channels, known before the first of them is split.  What the split finds of each pixel's largest value is kept in
// LDS; after the last step every wave looks through it for pixels that are too small for the scale, and at the largest of each
// kernel's sums over a lane's pixels, and computes outputs again whose window has no larger values, or whose kernel's sums are
// too small for what its operands may have lost: few of an image as fp32 sums of their own, more by taking the wave's block again on the
// fp32 instructions.  Nearly always all is well by one line for all kernels, from bounds; only otherwise is each kernel's own line
// computed, from what the weights' launch tells of it.  The scales and one barrier more cost 1.2 us of a workgroup's life, the look at
// the kernels' sums 0.3 - 0.5 (64 -> 64 at 56 x 56, batch 32 33.4 and 34.3 us, 256 -> 256, batch 64 602 and 605; with each kernel's own line
// there always, by v_dot2 beside the matrix instructions, 36.3 and 609).  Measured whole calls, three
// bf16 parts / two fp16 parts: 3x3, 256 -> 256 at 56 x 56, batch 64 927 / 595 us (398 TFLOP/s of fp32 products; register-only 646),
// 64 -> 64 at 56 x 56, batch 32 50 / 35, 128 -> 256 at 28 x 28, stride 2 57 / 41, 5x5, 96 -> 256 at 27 x 27, batch 16, channels
// innermost 76 / 57; 80 drawn layers 1.17 in the mean.
// What bounds it: the matrix cores are busy 0.6 of the cycles; the rest is LDS reads (85 bytes per clock and unit), weight loads (24
// through the L2) and the first loads and last stores of a round.  Twice the items per batch of staging: equal.
// With three parts (whole call on the fp32 instructions 1900 us, 934 - 953) measured on that layer: blocks of 32 x 112 per wave 1041 us (kernel),
// 64 x 64 with the weights read by two waves 1137, eight waves per workgroup 1046, chunks of 16 channels 1123; row pitch in
// LDS without the padding of split_derive 1068 against 1024; input loads whose descriptor or offset the compiler kept in
// vector registers (a loop over the lanes per load) 1073 against 1041.  Sums apart per step (APART) for all layers: error
// 1.8e-7 in place of 7.6e-7, 1129 us: kept for the few-channel layers only.
// Loads come back in the order they were issued, so a step that waits for weights waits for the inputs issued before them
// too, which come from further away: weights two or three steps ahead (AHEAD) give those as many steps to arrive.  One step
// ahead on blocks of more than eight 16 x 16 per wave: 64 -> 64 at 56 x 56, batch 32 48.5 us (two: 47.5, whole calls), 256 ->
// 256 at 56 x 56, batch 64 943 (908).
// Layers of one round of workgroups start and end together: of the 44 us a workgroup of 64 -> 64, batch 32, lives, 5.4
// pass before its first matrix step and 4.7 at its stores.  So the first loads go out before anything is waited for, and
// extents are divided by with a multiplication (64 -> 64 49.7 -> 48.5 us; 128 -> 256, stride 2 58.4 -> 55.6).
// Small layers (split_own) take no weights kernel before them: each workgroup reads the rows of its channels as they lie, cuts
// them into parts in LDS and multiplies from there (OWN; 16 -> 16 at 14 x 14, one image, 10.6 -> 8.2 us a call, 6.6 of them
// the GPU's).
#include "kernels.h"
#include "split_mfma.h"
#include "split_weights.h"

#include <type_traits>

namespace iolb {

namespace {

// Buffer of a block's images, first one n0: loads beyond them return zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t image_buffer(const float* x, const SplitGeom& g, int n0)
{
    const unsigned img = (unsigned)((long long)g.C * g.H * g.W * 4);
    const int images = g.N - n0 < g.b ? g.N - n0 : g.b;
    const unsigned long long xbase = reinterpret_cast<unsigned long long>(x + (size_t)n0 * g.C * g.H * g.W);
    // (the builtin returns a signed int: the halves have to be unsigned before they are put together)
    const unsigned xlo = __builtin_amdgcn_readfirstlane((unsigned)xbase), xhi = __builtin_amdgcn_readfirstlane((unsigned)(xbase >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((unsigned long long)xhi << 32 | xlo), 0,
                                             (int)__builtin_amdgcn_readfirstlane(img * (unsigned)images), 0x00020000);
}

template <int MB, int NB, int WM, int WN, bool VEC, bool APART, bool OWN, bool TWO>
__global__ void __launch_bounds__(64 * WM * WN, 2)
split_conv_kernel(const float* __restrict__ x, const u32x4* wt, float* y, SplitGeom given, SplitDivisors dv, SplitOwn own)
{
    // All of it is read here.  The compiler would otherwise read field by field where they are used, one wait after the other (33 scalar loads
    // before the first matrix step, and not 17: 64 -> 64 at 56 x 56, batch 32, 33.9 us and 33.5).
    SplitGeom read;
#pragma unroll
    for (unsigned i = 0; i < (TWO ? sizeof(read) / 4 : 0); ++i) reinterpret_cast<int*>(&read)[i] = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(&given)[i]);
    const SplitGeom& g = TWO ? read : given;
    extern __shared__ u32x4 lds16[];
    char* const lds = reinterpret_cast<char*>(lds16);
    constexpr int T = 64 * WM * WN;
    constexpr int IB = SPLIT_BATCH;
    static_assert(!TWO || (!APART && !OWN), "two fp16 parts, or three of bf16");
    constexpr int PARTS = TWO ? 2 : 3, PX = split_pixel_bytes(PARTS), WBLOCK = 64 * PARTS;
    // read here, once: loads of their own in the branches of a loop with diverging exits, which the compiler would make of
    // later uses, would count as values that differ between lanes
    const int CH8 = g.ch8, C = g.C, cstep = g.cstep;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm_i = wave % WM, wn_i = wave / WM;

    // consecutive workgroup ids are dealt round-robin to the 8 XCDs; remap so that each XCD (one L2) works on a
    // contiguous range of blocks, whose channel blocks share the same input tile
    int bid;
    {
        const int nblk = gridDim.x, q = nblk >> 3, r = nblk & 7, xcd = blockIdx.x & 7;
        bid = xcd * q + (xcd < r ? xcd : r) + ((int)blockIdx.x >> 3);
    }
    // channel blocks of the same pixels are neighbours, unless the kernels do not fit an L2 (k_outer): then an XCD stays with
    // one channel block
    const int pixel_blocks = g.nbx * g.nby * g.nbn;
    int kb, x0, y0, n0;
    if (dv.small) {
        const int a = g.k_outer ? dv.pixel_blocks.of(bid) : dv.nbk.of(bid);
        kb = g.k_outer ? a : bid - a * g.nbk;
        bid = g.k_outer ? bid - a * pixel_blocks : a;
        const int b = dv.nbx.of(bid), c = dv.nby.of(b);
        x0 = (bid - b * g.nbx) * g.tx;
        y0 = (b - c * g.nby) * g.ty;
        n0 = c * g.b;
    } else {
        kb = g.k_outer ? bid / pixel_blocks : bid % g.nbk;
        bid = g.k_outer ? bid % pixel_blocks : bid / g.nbk;
        x0 = bid % g.nbx * g.tx; bid /= g.nbx;
        y0 = bid % g.nby * g.ty;
        n0 = bid / g.nby * g.b;
    }
    // (divisions run on the vector unit: back to scalars, so that everything derived from them stays scalar)
    kb = __builtin_amdgcn_readfirstlane(kb);
    x0 = __builtin_amdgcn_readfirstlane(x0);
    y0 = __builtin_amdgcn_readfirstlane(y0);
    n0 = __builtin_amdgcn_readfirstlane(n0);

    const int RS = g.R * g.S;
    const int steps = (RS * CH8 + 3) >> 2;                  // matrix steps of a chunk: four units each
    const int items = CH8 * g.halo;
    const int im_bytes = g.yh * g.rowb, plane = g.b * im_bytes, group_bytes = split_planes(PARTS) * plane, buf_bytes = CH8 * group_bytes;
    // (two parts: l lies `plane` bytes after h)
    float* const kback = reinterpret_cast<float*>(lds + g.nbuf * buf_bytes);     // TWO: what undoes the scales of the block's kernels
    KernelLine* const lines = reinterpret_cast<KernelLine*>(kback + (TWO ? 16 * MB * WM : 0));           // TWO: of the kernels, where asked for
    int* const koff = reinterpret_cast<int*>(lines + (TWO ? 16 * MB * WM : 0));  // [4 * steps]
    uint2* const table = reinterpret_cast<uint2*>(koff + ((4 * steps + 1) & ~1));      // [items]
    // TWO: the largest value of each staged pixel over the channels, scaled; of each image in the sample (one image: of each wave)
    unsigned* const most = reinterpret_cast<unsigned*>(table + items);
    unsigned* const sample = most + g.halo;

    const int nchunks = __builtin_amdgcn_readfirstlane((C + 8 * CH8 - 1) / (8 * CH8));
    const int total = nchunks * steps;
    // weights of matrix step t: [t][16-channel block][part][lane]
    const int kb16 = kb * (MB * WM) + wm_i * MB;
    const size_t wstep = (size_t)g.Kb16 * WBLOCK;           // 16-byte pieces per step
    const u32x4* wp = wt + (size_t)kb16 * WBLOCK + lane;

    const __amdgpu_buffer_rsrc_t rs = image_buffer(x, g, n0);

    // where item `it` of the input tile comes from and where it goes
    const int gy0 = y0 * g.stride - g.pad, gx0 = x0 * g.stride - g.pad_w;
    auto place = [&](int it) {
        const int per = g.yh * g.rowp;
        const int c8 = dv.halo.of(it), hp = it - c8 * g.halo, im = dv.per.of(hp), rem = hp - im * per;
        const int iy = dv.rowp.of(rem), ix = rem - iy * g.rowp, ix_col = dv.esx.of(ix);
        // with a stride beyond the kernel's extent only the rows and columns that some window covers are staged
        const int gy = gy0 + iy + dv.esy.of(iy) * (g.stride - g.esy), gx = gx0 + ix + ix_col * (g.stride - g.esx);
        uint2 e;
        // (no branches: five of these stand between a workgroup's start and its last first load)
        const bool inside = (n0 + im < g.N) & (ix < g.xh) & ((unsigned)gy < (unsigned)g.H) & ((unsigned)gx < (unsigned)g.W);
        const int pixel = gy * g.W + gx;
        e.x = inside ? 4u * (unsigned)(g.hwc ? (im * g.H * g.W + pixel) * C + c8 * 8 : (im * C + c8 * 8) * g.H * g.W + pixel) : OUTSIDE;
        e.y = (unsigned)(c8 * group_bytes + im * im_bytes + iy * g.rowb + PX * ((ix - ix_col * g.esx) * g.colw + ix_col));
        // c8 in the low bits of the LDS offset (a multiple of 16, below 2^18); of two parts the image above, later its scale, a float
        e.y |= (unsigned)c8;
        if constexpr (TWO) e.y |= (unsigned)im << 23;
        return e;
    };

    // staging of chunk ch: an item's eight channels to registers, later its parts to LDS
    auto load_item = [&](float (&v)[8], uint2 e, int ch) {
        const int c0 = ch < nchunks ? ch * 8 * CH8 : 0, have = ch < nchunks ? C - c0 : 0;
        const int left = have - (int)(e.y & 15) * 8;          // channels of this group that exist
        if constexpr (VEC) {
            // channels innermost, C a multiple of 4 and x 16-byte aligned: two 16-byte loads
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rs, left > 4 * h ? (int)e.x + 16 * h : (int)OUTSIDE, c0 * 4, 0);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[4 * h + j] = __uint_as_float(q[j]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                // the scalar offset stays inside the buffer, whatever the lanes do
                const int cj = c0 + j < C ? c0 + j : C - 1;
                v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, left > j ? (int)e.x : (int)OUTSIDE, cj * cstep, 0));
            }
        }
    };
    static_assert(16 * NB * WN < 511, "images of a block, in nine bits beside no item");
    auto largest = [&]() {                                  // of a block's only image
        unsigned m = sample[0];
#pragma unroll
        for (int i = 1; i < WM * WN; ++i) m = sample[i] > m ? sample[i] : m;
        return m;
    };
    unsigned only = 0;                                      // its scale
    auto with_scale = [&](unsigned dst) {
        unsigned scale = only;
        if (g.b > 1) scale = half_scale_bits(sample[dst == ~0u ? 0 : dst >> 23]);
        return dst == ~0u ? dst : (dst & 0x7fffffu) | scale;
    };
    auto write_item = [&](const float (&v)[8], unsigned dst, char* buf, int it) {
        if constexpr (TWO) {
            u32x4 h, l;
            const float m = half_eight(v, __uint_as_float(dst & 0x7f800000u), h, l);
            if (dst != ~0u) {
                char* d = buf + (dst & 0x7ffff0u);
                *reinterpret_cast<u32x4*>(d) = h;
                *reinterpret_cast<u32x4*>(d + plane) = l;
                atomicMax(most + (it - (int)(dst & 15) * g.halo), __float_as_uint(m));
            }
            return;
        }
        u32x4 h, m, l;
        split_eight(v, h, m, l);
        if (dst != ~0u) {
            u32x4* d = reinterpret_cast<u32x4*>(buf + (dst & ~15u));
            d[0] = h; d[1] = m; d[2] = l;
        }
    };
    // a batch: IB items per thread, loads now, split and LDS writes one slot later.  A thread's own items: it alone reads
    // what it put in the table.
    float xv[IB][8];
    unsigned xdst[IB];
    const int batches = __builtin_amdgcn_readfirstlane((items + T * IB - 1) / (T * IB));
    auto load_batch = [&](int ch, int b) {
#pragma unroll
        for (int i = 0; i < IB; ++i) {
            const int it = (b * IB + i) * T + tid;
            uint2 e = {OUTSIDE, ~0u};
            if (it < items) e = table[it];
            xdst[i] = e.y;
            load_item(xv[i], e, ch);
        }
    };
    auto write_batch = [&](char* buf, int b) {
#pragma unroll
        for (int i = 0; i < IB; ++i) write_item(xv[i], xdst[i], buf, (b * IB + i) * T + tid);
    };
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // Everything the first steps need is on its way before the first of it is waited for: the first FIRST batches of chunk 0
    // as their places in the table are computed, the weights, chunk 1.  The rest of the tables is computed meanwhile.
    constexpr int FIRST = MB * NB >= 8 ? 2 : 1;
    float fv[FIRST][IB][8];
    unsigned fdst[FIRST][IB];
    auto place_batch = [&](float (&v)[IB][8], unsigned (&dst)[IB], int b) {
#pragma unroll
        for (int i = 0; i < IB; ++i) {
            const int it = (b * IB + i) * T + tid;
            uint2 e = {OUTSIDE, ~0u};
            if (it < items) {
                e = place(it);
                table[it] = e;
            }
            dst[i] = e.y;
            load_item(v[i], e, 0);
        }
    };
#pragma unroll
    for (int f = 0; f < FIRST; ++f) place_batch(fv[f], fdst[f], f);
    __builtin_amdgcn_sched_barrier(0);
    // Two parts: for the sample that sets the inputs' scales, beside the first batches, some values spread over the channels, of the
    // pixels of the first items, of several images over all of them; what undoes the kernels' scales.
    float spread = 0.f, my_kback = 0.f;
    unsigned spread_image = 0;
    constexpr int Z = 16 * MB * WM;
    if constexpr (TWO) {
        static_assert(Z <= T, "one kernel per thread");
        if (g.b > 1 || wave == 0) {
            uint2 e = {OUTSIDE, 0};
            if (g.b > 1) e = place(tid * items / T);
            else if (tid < items) e = table[tid];
            const int c = ((tid & 15) * nchunks >> 4) * 8 * CH8 + (tid >> 4 & 7);
            spread_image = e.y >> 23;
            const bool exists = e.x != OUTSIDE && c + (int)(e.y & 15) * 8 < C;
            spread = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, exists ? (int)(e.x + (unsigned)c * (unsigned)cstep) : (int)OUTSIDE, 0, 0));
        }
        for (int i = tid; i < g.halo; i += T) most[i] = 0;
        if (g.b > 1) {
            for (int i = tid; i < g.b; i += T) sample[i] = 0;
        }
        if (tid < Z) my_kback = reinterpret_cast<const float*>(wt + (size_t)total * wstep)[kb * Z + tid];
        __builtin_amdgcn_sched_barrier(0);
    }
    u32x4* const parts = reinterpret_cast<u32x4*>(lds + split_tables_bytes(g));     // a workgroup's own kernels (OWN)
    // Weights of the next AHEAD steps are on their way while a step multiplies: a step of a small block is shorter than
    // the latency of its loads.  A step issues first the weights, then the inputs.
    constexpr int AHEAD = OWN ? 1 : MB == 1 ? 3 : 2;
    u32x4 a[AHEAD + 1][MB * PARTS];
    auto load_weights = [&](u32x4 (&f)[MB * PARTS], int t) {
        if constexpr (OWN) {
            const u32x4* from = parts + ((t < total ? t : 0) * (MB * WM) + wm_i * MB) * 192 + lane;
#pragma unroll
            for (int j = 0; j < MB * PARTS; ++j) f[j] = from[j * 64];
            return;
        }
        if (t > 0 && t < total) wp += wstep;                // past the last step: read again, not used
#pragma unroll
        for (int j = 0; j < MB * PARTS; ++j) f[j] = wp[j * 64];
    };
    if constexpr (!OWN) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) load_weights(a[i], i);
    }
    __builtin_amdgcn_sched_barrier(0);
    // (Asked for in any case, as zeros where there is no second chunk, these loads let the first steps wait for fewer of them; that cost
    // layers of one chunk 1 - 4 %, and inputs in single floats with channels innermost up to 6: 411 -> 22 at 129 x 90, stride 2, batch 43
    // 706 us, 753 so; 17 -> 249 at 58 x 58 57.0 and 58.4.  Over 2500 drawn layers the branch is 0.7 % the better one, 3 - 4 % the worse
    // on 20; only the narrow blocks that read four channels at a time, 0.5 % the other way, go without.)
    if (nchunks > 1 || (VEC && MB * NB <= 2)) load_batch(1, 0);
    __builtin_amdgcn_sched_barrier(0);

    // LDS byte offset of unit (tap, channel group) relative to a pixel's window corner
    for (int u = tid; u < 4 * steps; u += T) {
        const int tap = dv.ch8.of(u), c8 = u - tap * CH8;
        int off = 0;
        if (tap < RS) {
            const int r = dv.S.of(tap), s = tap - r * g.S, s_col = dv.esx.of(s);
            off = c8 * group_bytes + r * g.rowb + PX * ((s - s_col * g.esx) * g.colw + s_col);
        }
        koff[u] = off;
    }
    // its own kernels (OWN): from w, whose rows for these channels are one stretch, to LDS, one float between rows; from there
    // the parts, in the order of the steps
    const int row_w = C * RS;
    if constexpr (OWN) {
        float* const rows = reinterpret_cast<float*>(parts + nchunks * steps * (MB * WM * 192));
        constexpr int PER = 8;
        const float* w = reinterpret_cast<const float*>(wt);
        const int k0 = kb * Z, have = (g.K - k0 < Z ? g.K - k0 : Z) * row_w;
        for (int e0 = tid; e0 < Z * row_w + tid; e0 += T * PER) {
            float v[PER];
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int e = e0 + i * T;
                v[i] = w[e < have ? (size_t)k0 * row_w + e : 0];
                v[i] = e < have ? v[i] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int e = e0 + i * T;
                if (e < Z * row_w) rows[e + own.row.of(e)] = v[i];
            }
        }
        barrier();
        for (int p = tid; p < nchunks * steps * (MB * WM * 64); p += T) {
            const int block = (p >> 6) % (MB * WM), t = (p >> 6) / (MB * WM), ch = own.steps.of(t);
            const int unit = (t - ch * steps) * 4 + (p >> 4 & 3), tap = dv.ch8.of(unit), c0 = (ch * CH8 + unit - tap * CH8) * 8;
            const int r = dv.S.of(tap), tw = own.transposed ? (tap - r * g.S) * g.R + r : tap;
            const float* from = rows + (block * 16 + (p & 15)) * (row_w + 1) + c0 * RS + tw;
            unsigned short q[3][8];
#pragma unroll
            for (int j = 0; j < 8; ++j) split_kept(tap < RS && c0 + j < C ? from[j * RS] : 0.f, q[0][j], q[1][j], q[2][j]);
            store_parts(parts + (p >> 6) * 192 + (p & 63), q);
        }
    }

    // pixels of this lane
    const int txy = g.tx * g.ty, npix = g.b * txy;
    int pbase[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int slot = (wn_i * NB + nb) * 16 + l16;
        const int pix = slot < npix ? slot : npix - 1;
        const int im = dv.txy.of(pix), rem = pix - im * txy, py = dv.tx.of(rem), px = rem - py * g.tx;
        pbase[nb] = im * im_bytes + py * g.esy * g.rowb + PX * px;
    }

    __builtin_amdgcn_sched_barrier(0);
    if constexpr (TWO) {
        // scales of the images, from the first batches and the spread values
        unsigned mine[FIRST][IB];
#pragma unroll
        for (int f = 0; f < FIRST; ++f)
#pragma unroll
            for (int i = 0; i < IB; ++i) mine[f][i] = largest_of(fv[f][i]);
        unsigned all = finite_bits(spread);
        if (g.b > 1) {
            barrier();
            if (all) atomicMax(sample + spread_image, all);
#pragma unroll
            for (int f = 0; f < FIRST; ++f)
#pragma unroll
                for (int i = 0; i < IB; ++i)
                    if (mine[f][i]) atomicMax(sample + (fdst[f][i] >> 23), mine[f][i]);      // (an item that does not exist is zeros)
        } else {
#pragma unroll
            for (int f = 0; f < FIRST; ++f)
#pragma unroll
                for (int i = 0; i < IB; ++i) all = mine[f][i] > all ? mine[f][i] : all;
            all = wave_max(all);
            if (lane == 0) sample[wave] = all;
        }
        barrier();
        only = half_scale_bits(largest());
#pragma unroll
        for (int f = 0; f < FIRST; ++f)
#pragma unroll
            for (int i = 0; i < IB; ++i) {
                fdst[f][i] = with_scale(fdst[f][i]);
                if (fdst[f][i] != ~0u) table[(f * IB + i) * T + tid].y = fdst[f][i];
            }
#pragma unroll
        for (int i = 0; i < IB; ++i) xdst[i] = fdst[0][i];                       // (those of the second chunk's first batch, if there is one)
    }
#pragma unroll
    for (int f = 0; f < FIRST; ++f)
#pragma unroll
        for (int i = 0; i < IB; ++i) write_item(fv[f][i], fdst[f][i], lds, (f * IB + i) * T + tid);
    for (int b = FIRST; b < batches; ++b) {
        place_batch(fv[0], fdst[0], b);
#pragma unroll
        for (int i = 0; i < IB; ++i) {
            const int it = (b * IB + i) * T + tid;
            if constexpr (TWO) {
                fdst[0][i] = with_scale(fdst[0][i]);
                if (fdst[0][i] != ~0u) table[it].y = fdst[0][i];
            }
            write_item(fv[0][i], fdst[0][i], lds, it);
        }
    }
    if constexpr (TWO) {
        if (tid < Z) kback[tid] = my_kback;
    }
    barrier();
    if constexpr (OWN) load_weights(a[0], 0);

    f32x4 acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

    u32x4 bf[2][PARTS];
    auto fetch = [&](u32x4 (&f)[PARTS], const char* from) {
#pragma unroll
        for (int p = 0; p < PARTS; ++p) f[p] = *reinterpret_cast<const u32x4*>(from + (TWO ? plane : 16) * p);
    };
    int ch = 0, k = 0, t = 0;
    int ko = koff[grp];
    fetch(bf[0], lds + ko + pbase[0]);
    // One matrix step: four units (tap, channel group) for every block of the wave.  The pixels come from LDS one block
    // ahead, across steps too.
    auto step = [&](const u32x4 (&w0)[MB * PARTS], u32x4 (&wn)[MB * PARTS]) {
        const bool chunk_end = k + 1 == steps;
        load_weights(wn, t + AHEAD);
        const char* bp = lds + split_buffer(ch, g.nbuf) * buf_bytes;
        const int kn = koff[4 * (chunk_end ? 0 : k + 1) + grp];
        auto block = [&](auto nb_c) {
            constexpr int nb = decltype(nb_c)::value;
            if constexpr (nb + 1 < NB) fetch(bf[(nb + 1) & 1], bp + ko + pbase[nb + 1]);
            else                       fetch(bf[(nb + 1) & 1], bp + kn + pbase[0]);
            // the products of parts that reach fp32 precision, smallest first: six, of two parts three
            constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
            f32x4 sum[MB];
#pragma unroll
            for (int q = TWO ? 3 : 0; q < 6; ++q)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    if constexpr (TWO) {
                        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            __builtin_bit_cast(f16x8, w0[mb * PARTS + PA[q]]), __builtin_bit_cast(f16x8, bf[nb & 1][PB[q]]), acc[mb][nb], 0, 0, 0);
                        continue;
                    }
                    f32x4& to = APART ? sum[mb] : acc[mb][nb];
                    to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, w0[mb * PARTS + PA[q]]), __builtin_bit_cast(bf16x8, bf[nb & 1][PB[q]]),
                        APART && q == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : to, 0, 0, 0);
                }
            if constexpr (APART) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[mb][nb] += sum[mb];
            }
        };
        constexpr int HALF = NB / 2;
        static_range<0, HALF>(block);
        // Loads come back in the order they were issued.  Where the paths with and without input loads meet, the
        // compiler would have to assume the worst and wait for every load at the next use of a weight: the two paths
        // stay apart until each has waited for the weights of the next step.
        constexpr int LATER = MB * PARTS * (AHEAD - 1), LOADS = (VEC ? 2 : 8) * IB;
        if (k < batches && ch + 1 < nchunks) {
            write_batch(lds + split_buffer(ch + 1, g.nbuf) * buf_bytes, k);
            const bool more = k + 1 < batches;
            load_batch(more ? ch + 1 : ch + 2, more ? k + 1 : 0);
            static_range<HALF, NB>(block);
            if constexpr (!OWN) __builtin_amdgcn_s_waitcnt(0x0F70 | ((LATER + LOADS) & 15) | ((LATER + LOADS) >> 4) << 14);
        } else {
            static_range<HALF, NB>(block);
            if constexpr (!OWN) __builtin_amdgcn_s_waitcnt(0x0F70 | (LATER & 15) | (LATER >> 4) << 14);
        }
        if constexpr (NB & 1) {
#pragma unroll
            for (int p = 0; p < PARTS; ++p) bf[0][p] = bf[1][p];
        }
        ko = kn;
        ++k;
        const bool done = ++t == total;
        if (chunk_end && !done) {                           // (one chunk has one buffer: there is no next one to read)
            barrier();
            k = 0;
            ++ch;
            fetch(bf[0], lds + split_buffer(ch, g.nbuf) * buf_bytes + ko + pbase[0]);
        }
        return done;
    };
    // AHEAD + 1 copies, so that every step names its registers
    bool done = false;
    while (!done)
        static_range<0, AHEAD + 1>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value;
            if (!done) done = step(a[i], a[(i + AHEAD) % (AHEAD + 1)]);
        });

    // each partial sum is complete: write the block once.  Register i of a 16 x 16 block holds channel 4 grp + i of
    // pixel l16.
    const size_t PQ = (size_t)g.P * g.Q;
    unsigned long long again = 0;                           // outputs that are computed once more
    static_assert(MB * NB * 4 <= 64, "one mark per output");
    // what undoes the scales (one image in a block: its own)
    float back = 1.f;
    f32x4 kb4[MB];
    bool fine;
    int image[NB], first_image = 0, last_image = 0, judging = JUDGE_LANE;
    bool ragged = false;                                    // some pixels of the block are no outputs
    auto image_of = [&](int nb) {
        const int slot = (wn_i * NB + nb) * 16 + (opaque(lane) & 15);
        return dv.txy.of(slot < npix ? slot : npix - 1);
    };
    if constexpr (TWO) {
        back = half_unscale(half_scale_bits(largest()));
        // pixels whose channels are all too small for their scale, and not all zeros: the windows they are in are looked at below
        bool small = false;
        unsigned brightest = 0;
        for (int i = lane; i < g.halo; i += 64) {
            small |= most[i] - 1 < __float_as_uint(HALF_LEAST) - 1;
            brightest = most[i] > brightest ? most[i] : brightest;
        }
        const float inputs = __uint_as_float(wave_max(brightest));
        // Whether all sums are finite and no kernel's too small, by the largest input: mostly so, and then they are only written.
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) kb4[mb] = *reinterpret_cast<const f32x4*>(kback + (wm_i * MB + mb) * 16 + 4 * grp);
        // First by a line for all kernels, then by each one's own.  A kernel's sums that are judged together: judge_sums.
        bool bad;
        ragged = (y0 + g.ty > g.P) | (x0 + g.tx > g.Q) | (n0 + g.b > g.N);
        // (The way of most workgroups lies by itself: instructions come from memory here.  Slots beyond the pixels of a whole block of one image
        // hold the last of them again.)
        const bool whole = (g.b == 1) & !ragged;
        if (__builtin_expect(!whole, 0)) {
            first_image = dv.txy.of(wn_i * NB * 16 < npix ? wn_i * NB * 16 : npix - 1);
            last_image = dv.txy.of((wn_i + 1) * NB * 16 < npix ? (wn_i + 1) * NB * 16 - 1 : npix - 1);
            judging = g.b == 1 ? JUDGE_LANE : last_image - first_image < MOST_IMAGES ? JUDGE_IMAGES : JUDGE_QUADS;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int slot = (wn_i * NB + nb) * 16 + l16, im = dv.txy.of(slot), rem = slot - im * txy, row = dv.tx.of(rem);
                image[nb] = (slot < npix) & (n0 + im < g.N) & (y0 + row < g.P) & (x0 + rem - row * g.tx < g.Q) ? im : -1;
            }
        }
        const float all_kernels = HALF_LINE * (__builtin_amdgcn_sqrtf(own.facts * HALF_PIECE) + __builtin_amdgcn_sqrtf((float)(C * RS)) * inputs);
        auto all_well = [&](auto closer_c) {
            constexpr bool closer = decltype(closer_c)::value;
            bad = small;
            auto see = [&](int mb, int i, float m) {
                const float line = closer ? line_of(lines[(wm_i * MB + mb) * 16 + 4 * grp + i], inputs) : all_kernels;
                bad |= (!(m >= line) & ((kb16 + mb) * 16 + 4 * grp + i < g.K)) | !(m <= FINITE);
            };
            if (__builtin_expect(whole, 1)) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float m = 0.f;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) m = __builtin_elementwise_maximum(m, __builtin_fabsf(acc[mb][nb][i]));
                        if constexpr (NB < 4) m = quad_largest(m, 0);
                        see(mb, i, m);
                    }
            } else {
                bool any = false;
                judge_sums<MB, NB>(judging, ragged, image, first_image, last_image, [&](int mb, int nb, int i) { return __builtin_fabsf(acc[mb][nb][i]); },
                                   [&](auto in) {
                                       any = false;
#pragma unroll
                                       for (int nb = 0; nb < NB; ++nb) any |= in(nb);
                                       if (judging == JUDGE_LANE) any = __builtin_amdgcn_ballot_w64(any) != 0;
                                   },
                                   [&](int mb, int i, float m) { see(mb, i, any || !(m <= FINITE) ? m : FINITE); });
            }
            return __builtin_amdgcn_ballot_w64(bad) == 0;
        };
        fine = all_well(std::false_type{});
        if (__builtin_expect(!fine, 0)) {
            wave_lines<MB>(reinterpret_cast<const KernelFacts*>(reinterpret_cast<const float*>(wt + (size_t)total * wstep) + 16 * g.Kb16) + kb16 * 16, own.facts,
                           16 * g.Kb16, lane, lines + wm_i * (16 * MB));
            fine = all_well(std::true_type{});
        }
    } else {
        float m = 0.f;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int i = 0; i < 4; ++i) m = __builtin_elementwise_maximum(m, __builtin_fabsf(acc[mb][nb][i]));
        fine = __builtin_amdgcn_ballot_w64(!(m <= FINITE)) == 0;
    }
    // Otherwise each output for itself: sums that are not finite; those whose window has no value that is large enough, and not only
    // zeros; those of kernels whose finite sums are all too small for it.
    if (__builtin_expect(!fine, 0)) {
        const int l16 = opaque(lane) & 15, grp = opaque(lane) >> 4;
        unsigned window[NB], exists = 0;
        int corner[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int slot = (wn_i * NB + nb) * 16 + l16, im = dv.txy.of(slot), rem = slot - im * txy, row = dv.tx.of(rem), col = rem - row * g.tx;
            const bool there = (slot < npix) & (n0 + im < g.N) & (y0 + row < g.P) & (x0 + col < g.Q);
            exists |= there ? 1u << nb : 0u;
            image[nb] = there ? im : -1;
            corner[nb] = there ? (im * g.yh + row * g.esy) * g.rowp + col * g.esx : 0;
            window[nb] = 0;
        }
        if constexpr (TWO)
            for (int r = 0; r < g.R; ++r)
                for (int s = 0; s < g.S; ++s)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const unsigned m = most[corner[nb] + r * g.rowp + s];
                        window[nb] = m > window[nb] ? m : window[nb];
                    }
        const int kernels = g.K - kb16 * 16 - 4 * grp;      // that exist from this lane's first on
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const bool lost = TWO && window[nb] - 1 < __float_as_uint(HALF_LEAST) - 1;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if ((exists >> nb & 1) & (lost | !(__builtin_fabsf(acc[mb][nb][i]) <= FINITE)) & (mb * 16 + i < kernels))
                        again |= 1ull << ((nb * MB + mb) * 4 + i);
        }
        if constexpr (TWO) {
            unsigned group = 0;                             // bits of the nb that are judged together
            judge_sums<MB, NB>(judging, ragged, image, first_image, last_image,
                               [&](int mb, int nb, int i) { return __builtin_fabsf(acc[mb][nb][i]) <= FINITE ? __builtin_fabsf(acc[mb][nb][i]) : 0.f; },
                               [&](auto in) {
                                   group = 0;
#pragma unroll
                                   for (int nb = 0; nb < NB; ++nb) group |= in(nb) && window[nb] != 0 ? 1u << nb : 0u;
                               },
                               [&](int mb, int i, float m) {
                                   if (mb * 16 + i >= kernels) return;
                                   const KernelLine line = lines[(wm_i * MB + mb) * 16 + 4 * grp + i];
#pragma unroll
                                   for (int nb = 0; nb < NB; ++nb)
                                       if ((group >> nb & 1) & !(m >= line_of(line, __uint_as_float(window[nb])))) again |= 1ull << ((nb * MB + mb) * 4 + i);
                               });
        }
    }
    // all of them; the second time those that were marked
    auto write_y = [&](auto marked_c) {
        constexpr bool MARKED = decltype(marked_c)::value;
        const int l16 = opaque(lane) & 15, grp = opaque(lane) >> 4;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int slot = (wn_i * NB + nb) * 16 + l16;
            const int im = dv.txy.of(slot), rem = slot - im * txy, row = dv.tx.of(rem), py = y0 + row, px = x0 + rem - row * g.tx;
            if (slot >= npix || n0 + im >= g.N || py >= g.P || px >= g.Q) continue;
            if constexpr (TWO && !MARKED)
                if (g.b > 1) back = half_unscale(half_scale_bits(sample[im]));
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const int k0 = (kb16 + mb) * 16 + 4 * grp, bit = (nb * MB + mb) * 4;
                if constexpr (!MARKED) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (TWO) acc[mb][nb][i] = acc[mb][nb][i] * back * kb4[mb][i];
                        else               acc[mb][nb][i] *= SPLIT_UNSCALE;
                    }
                }
                if (g.hwc) {
                    float* yp = y + (((size_t)(n0 + im) * g.P + py) * g.Q + px) * g.K + k0;
                    if (!MARKED && g.vec_out && k0 + 3 < g.K) {
                        *reinterpret_cast<f32x4*>(yp) = acc[mb][nb];
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (k0 + i < g.K && (!MARKED || again >> (bit + i) & 1)) yp[i] = acc[mb][nb][i];
                    }
                } else {
                    float* yp = y + ((size_t)(n0 + im) * g.K + k0) * PQ + (size_t)py * g.Q + px;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (k0 + i < g.K && (!MARKED || again >> (bit + i) & 1)) yp[(size_t)i * PQ] = acc[mb][nb][i];
                }
            }
        }
    };
    write_y(std::false_type{});
    if (__builtin_expect(fine || __builtin_amdgcn_ballot_w64(again != 0) == 0, 1)) return;

    // Few marked outputs of an image are sums of their own, a wave's lanes one channel each: so single sums that are small by chance, where
    // few are judged together, or windows of one small value cost 1 - 2 us and not a block.  (Image by image: what other images hold
    // decides nothing.)
    if constexpr (TWO) {
        constexpr int FEW = 16;
        unsigned long long many = 0;
        while (const unsigned long long lanes = __builtin_amdgcn_ballot_w64(again != 0)) {
            const int src = __builtin_ctzll(lanes);
            const int nb0 = __builtin_amdgcn_readlane((int)(__builtin_ctzll(again | 1ull << 63) / (4 * MB)), src);
            const int image = dv.txy.of((wn_i * NB + nb0) * 16 + (src & 15));
            unsigned long long mine = 0;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) mine |= image_of(nb) == image ? again & (((1ull << (4 * MB - 1) << 1) - 1) << (nb * MB * 4)) : 0;
            again &= ~mine;
            if (wave_sum((float)__popcll(mine)) > FEW) { many |= mine; continue; }
            while (const unsigned long long left = __builtin_amdgcn_ballot_w64(mine != 0)) {
                const int at = __builtin_ctzll(left);
                const int bit = __builtin_amdgcn_readlane(__builtin_ctzll(mine | 1ull << 63), at);
                if (lane == at) mine &= mine - 1;
                const int nb = bit / (4 * MB), k = (kb16 + bit / 4 % MB) * 16 + 4 * (at >> 4) + (bit & 3);
                const int rem = (wn_i * NB + nb) * 16 + (at & 15) - image * txy, row = rem / g.tx, n = n0 + image, py = y0 + row, px = x0 + rem % g.tx;
                // (a lane takes every 64th of channels and taps, eight at a time: the latency of their loads is what this costs)
                const float *xp = x + (size_t)n * C * g.H * g.W, *wp1 = own.w + (size_t)k * C * RS;
                const int gy1 = py * g.stride - g.pad, gx1 = px * g.stride - g.pad_w;
                float sum = 0.f;
#pragma unroll 1
                for (int e0 = lane; e0 < RS * C; e0 += 8 * 64) {
                    float v[8], u[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int e = e0 + 64 * j, c = e / RS, tap = e - c * RS;                     // as the kernel lies
                        const int r = own.transposed ? tap % g.R : tap / g.S, s = own.transposed ? tap / g.R : tap - r * g.S;
                        const int gy = gy1 + r, gx = gx1 + s;
                        const bool inside = (e < RS * C) & (gy >= 0) & (gy < g.H) & (gx >= 0) & (gx < g.W);
                        v[j] = xp[inside ? (size_t)c * (cstep / 4) + (g.hwc ? ((size_t)gy * g.W + gx) * C : (size_t)gy * g.W + gx) : 0];
                        v[j] = inside ? v[j] : 0.f;
                        u[j] = wp1[inside ? e : 0];
                        u[j] = inside ? u[j] : 0.f;
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) sum = __builtin_fmaf(v[j], u[j], sum);
                }
                sum = wave_sum(sum);
                if (lane == at) y[g.hwc ? (((size_t)n * g.P + py) * g.Q + px) * g.K + k : ((size_t)n * g.K + k) * PQ + (size_t)py * g.Q + px] = sum;
            }
        }
        again = many;
        if (__builtin_amdgcn_ballot_w64(again != 0) == 0) return;
    }

    // A wave with a marked output takes its whole block again on the fp32 matrix instructions, which hold their sums in
    // the same registers: in the same steps, four units of eight channels, the inputs from memory, those of the next 16
    // pixels while the present ones are multiplied.  Bound by the latency of a step's loads, at most once per wave: 64 -> 64
    // at 56 x 56, batch 8, all inputs NaN 40 -> 89 us (one output at a time in its lane: 3081), one NaN 53 (1234); 256 ->
    // 256 at 56 x 56, batch 64, all NaN 3516 against 1891 on the fp32 tile.
    // (a descriptor of its own: kept through the matrix loop, the first one would end in vector registers)
    const __amdgpu_buffer_rsrc_t rs2 = image_buffer(x, g, __builtin_amdgcn_readfirstlane(opaque(n0)));
    const int lane2 = opaque(lane), col16 = lane2 & 15, unit0 = lane2 >> 4;
    int cy[NB], cx[NB], ci[NB];                             // window corner and image of this lane's pixels
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int slot = (wn_i * NB + nb) * 16 + col16, pix = slot < npix ? slot : npix - 1, rem = pix % txy;
        ci[nb] = pix / txy;
        cy[nb] = gy0 + rem / g.tx * g.stride;
        cx[nb] = gx0 + rem % g.tx * g.stride;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const u32x4* wq = OWN ? parts + wm_i * (MB * 192) + lane2 : wt + (size_t)kb16 * 192 + lane2;
    const size_t next_w = OWN ? MB * WM * 192 : wstep;
#pragma unroll 1
    for (int s = 0; s < total; ++s, wq += next_w) {
        const int unit = s % steps * 4 + unit0, tap = unit / CH8, c0 = (s / steps * CH8 + unit % CH8) * 8;
        const int r = tap / g.S, col = tap % g.S;
        float wv[MB][8], v[2][8];
        auto load_v = [&](float (&to)[8], int cyn, int cxn, int cin) {
            const int gy = cyn + r, gx = cxn + col;
            const bool inside = tap < RS && n0 + cin < g.N && gy >= 0 && gy < g.H && gx >= 0 && gx < g.W;
            const unsigned at = g.hwc ? 4u * (unsigned)(((cin * g.H + gy) * g.W + gx) * C + c0) : 4u * (unsigned)(((cin * C + c0) * g.H + gy) * g.W + gx);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                to[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs2, inside && c0 + j < C ? (int)(at + j * (unsigned)cstep) : (int)OUTSIDE, 0, 0));
        };
        load_v(v[0], cy[0], cx[0], ci[0]);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if constexpr (TWO) {
                // the kernels as the caller holds them: their two parts are not always all of them
                const int k0 = (kb16 + mb) * 16 + col16, tw = own.transposed ? col * g.R + r : tap;
                const float* from = own.w + ((size_t)(k0 < g.K ? k0 : 0) * C + c0) * RS + tw;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool exists = tap < RS && k0 < g.K && c0 + j < C;
                    wv[mb][j] = exists ? from[(size_t)j * RS] : 0.f;
                }
            } else {
                kept_eight(wq[mb * 192], wq[mb * 192 + 64], wq[mb * 192 + 128], wv[mb]);
            }
            if constexpr (MB > 2) __builtin_amdgcn_sched_barrier(0);       // all pieces at once would not fit the registers
        }
        static_range<0, NB>([&](auto nb_c) {
            constexpr int nb = decltype(nb_c)::value;
            if constexpr (nb + 1 < NB) load_v(v[(nb + 1) & 1], cy[nb + 1], cx[nb + 1], ci[nb + 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[mb][j], v[nb & 1][j], acc[mb][nb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    write_y(std::true_type{});
}

// w[K][C][R][S] -> the operands of the matrix steps, [chunk][step][16-channel block][part][lane][8 values].  A workgroup per 16
// kernels, `octets` groups of eight channels and up to 16 taps (all of them, or slices of 16), whose pieces its threads take
// one each: rows of w are read as they lie, 16 floats and more at a time, and go through LDS.  Bound by latency: a load, an
// LDS pass and a store one after the other (gathered in single floats, 256 -> 256 kernels of 3 x 3 took 7.4 us, now 5.7; 7 x
// 7 and 11 x 11 on three channels 62 -> 58 and 49.2 -> 46.8 whole calls).
constexpr int SLICE = 16, ROW = 8 * SLICE;                 // taps of a slice; floats of a kernel in LDS
template <bool TWO>
__global__ void __launch_bounds__(256)
split_weights_kernel(const float* __restrict__ w, u32x4* __restrict__ wt, int K, int C, int R, int S, int ch8, int steps, int Kb16,
                     int octets, int all_octets, int slices, int transposed)
{
    constexpr int PITCH = ROW + 1, ROWS = 16, MINE = ROWS / 4;
    __shared__ unsigned scales[ROWS];                       // TWO: scale of each kernel, lowest bit: too small or too large for it here
    __shared__ float rows[ROWS * PITCH];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = blockIdx.x % Kb16, rest = blockIdx.x / Kb16, first = rest / slices * octets, t0 = rest % slices * SLICE;
    const int RS = R * S, taps = 4 * steps / ch8, k0 = kb * 16;
    const int ts = slices > 1 ? SLICE : RS;                 // taps of a channel in LDS
    const int channels = C - first * 8 < octets * 8 ? C - first * 8 : octets * 8;
    const long long from0 = (long long)k0 * C * RS + (long long)first * 8 * RS + t0;
    float v[2][MINE], some[MINE];
    if constexpr (TWO) {
        const int row = C * RS, at = (int)((long long)row * (lane >> 2) >> 4) + (lane & 3);
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const int k = k0 + wave * MINE + j;
            const bool exists = k < K && at < row;
            some[j] = w[exists ? (size_t)k * row + at : 0];
            some[j] = exists ? some[j] : 0.f;
        }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int e = lane + 64 * c, row = slices > 1 ? e / SLICE * RS + e % SLICE : e;
        // (kernels, channels and taps that only fill a block up are not there to be read)
        const bool here = slices > 1 ? e / SLICE < channels && t0 + e % SLICE < RS : e < channels * RS;
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const int k = wave * MINE + j;
            const bool exists = here && k0 + k < K;
            v[c][j] = w[exists ? from0 + (long long)k * C * RS + row : 0];
            v[c][j] = exists ? v[c][j] : 0.f;
        }
    }
    if constexpr (TWO) {
        // A kernel's scale follows from 64 of its values, 16 runs of four spread over it: the same in each of its workgroups.
        float* const kback = reinterpret_cast<float*>(wt + (size_t)steps * (all_octets / ch8) * Kb16 * 128);
        KernelFacts* const facts = reinterpret_cast<KernelFacts*>(kback + 16 * Kb16) + (size_t)rest * 16 * Kb16 + k0;
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const int k = wave * MINE + j;
            unsigned here = __float_as_uint(__builtin_fabsf(v[0][j])), there = __float_as_uint(__builtin_fabsf(v[1][j]));
            here = here > there ? here : there;
            const unsigned scale = half_scale_bits(wave_max(finite_bits(some[j])));
            here = wave_max(here);
            const float a = v[0][j] * __uint_as_float(scale), b = v[1][j] * __uint_as_float(scale);
            const float squares = wave_sum(__builtin_fmaf(a, a, b * b));
            const int small = __popcll(__builtin_amdgcn_ballot_w64(v[0][j] != 0.f && __builtin_fabsf(a) < HALF_LEAST)) +
                              __popcll(__builtin_amdgcn_ballot_w64(v[1][j] != 0.f && __builtin_fabsf(b) < HALF_LEAST));
            if (lane == 0) {
                facts[k] = {squares, (float)small};
                // (of fewer than 32 values here some are all small now and then: left to the sums)
                scales[k] = scale + ((here != 0 && channels * ts >= 32 && __uint_as_float(here) * __uint_as_float(scale) < HALF_LEAST) || !(squares <= HALF_PIECE));
                if (first == 0 && t0 == 0) kback[k0 + k] = half_unscale(scale);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int j = 0; j < MINE; ++j) rows[(wave * MINE + j) * PITCH + lane + 64 * c] = v[c][j];
    __syncthreads();
    const int k = tid & 15, mine = slices > 1 ? SLICE : taps, t = t0 + (tid >> 4) % mine, o = (tid >> 4) / mine, octet = first + o;
    if (o >= octets || octet >= all_octets || t >= taps) return;
    const float* from = rows + k * PITCH + o * 8 * ts + t - t0;
    if constexpr (TWO) {
        // (a kernel that does not fit its scale: NaN in place of its parts here, which every sum of it shows)
        const float scale = __uint_as_float(scales[k] & ~1u);
        const unsigned poison = scales[k] & 1 ? 0x7e007e00u : 0u;
        float g8[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) g8[j] = t < RS ? from[j * ts] : 0.f;
        u32x4 h, l;
        half_eight(g8, scale, h, l);
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] |= poison;
        const int tap = transposed && t < RS ? t % R * S + t / R : t, unit = tap * ch8 + octet % ch8;
        u32x4* to = wt + ((size_t)(octet / ch8 * steps + (unit >> 2)) * Kb16 + kb) * 128 + (unit & 3) * 16 + k;
        to[0] = h;
        to[64] = l;
        return;
    }
    unsigned short p[3][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) split_kept(t < RS ? from[j * ts] : 0.f, p[0][j], p[1][j], p[2][j]);
    const int tap = transposed && t < RS ? t % R * S + t / R : t;
    const int unit = tap * ch8 + octet % ch8;
    store_parts(wt + ((size_t)(octet / ch8 * steps + (unit >> 2)) * Kb16 + kb) * 192 + (unit & 3) * 16 + k, p);
}

template <int MB, int NB, int WM, int WN, bool VEC, bool APART, bool OWN, bool TWO>
hipError_t launch_one(const float* x, const u32x4* wt, float* y, const SplitGeom& g, const SplitDivisors& dv, const SplitOwn& own, hipStream_t st)
{
    auto kern = split_conv_kernel<MB, NB, WM, WN, VEC, APART, OWN, TWO>;
    const size_t shm = split_lds_bytes(g, OWN);
    if (shm > 64 * 1024) {
        const hipError_t e = allow_large_lds((const void*)kern);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(g.nbk * g.nbx * g.nby * g.nbn), dim3(64 * WM * WN), shm, st, x, wt, y, g, dv, own);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_split_weights(const float* w, void* wt, int K, int C, int R, int S, int ch8, int Kb16, int parts, bool transposed, hipStream_t st)
{
    if (ch8 != 1 && ch8 != 2 && ch8 != 4) return hipErrorInvalidValue;
    const SplitPieces p = split_pieces(C, R * S, ch8);
    const long long blocks = (long long)p.pieces * Kb16;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    // the room of three parts, 3072 bytes per unit, holds two, the scales and the facts
    static_assert(SLICE == 16);
    if (parts == 2 && 2048LL * (p.octets / ch8) * p.steps + 64 + 128LL * p.pieces > 3072LL * (p.octets / ch8) * p.steps) return hipErrorInvalidValue;
    hipLaunchKernelGGL(parts == 2 ? split_weights_kernel<true> : split_weights_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, w, (u32x4*)wt, K, C, R, S, ch8, p.steps,
                       Kb16, p.per, p.octets, p.slices, transposed ? 1 : 0);
    return hipGetLastError();
}

// At most eight channels (ch8 = 1): each step's products are summed from zero before they are added to the running
// sum, which is then rounded once per step and not six times.  Such layers ran on plain FMAs or short fp32 chains
// before, which round less than six bf16 products per step would; they are not bound by the matrix cores.
template <bool VEC>
static hipError_t launch_shape(const float* x, const u32x4* wt, float* y, const SplitGeom& g, const SplitDivisors& dv, bool own, const SplitOwn& o, hipStream_t st)
{
#define IOLB_SPLIT_IS(M_, N_, A_, B_) (g.mb == M_ && g.nb == N_ && g.wm == A_ && g.wn == B_)
#define IOLB_SPLIT_TWO_CASE(M_, N_, A_, B_) \
    if (g.parts == 2 && IOLB_SPLIT_IS(M_, N_, A_, B_)) return launch_one<M_, N_, A_, B_, VEC, false, false, true>(x, wt, y, g, dv, o, st);
#define IOLB_SPLIT_CASE(M_, N_, A_, B_) \
    if (g.parts == 3 && !own && IOLB_SPLIT_IS(M_, N_, A_, B_)) return launch_one<M_, N_, A_, B_, VEC, APART, false, false>(x, wt, y, g, dv, o, st);
#define IOLB_SPLIT_OWN_CASE(M_, N_, A_, B_) \
    if (own && IOLB_SPLIT_IS(M_, N_, A_, B_)) return launch_one<M_, N_, A_, B_, VEC, APART, true, false>(x, wt, y, g, dv, o, st);
    if (g.ch8 == 1) {
        constexpr bool APART = true;
        IOLB_SPLIT_FEW_SHAPES(IOLB_SPLIT_CASE)
        IOLB_SPLIT_OWN_FEW_SHAPES(IOLB_SPLIT_OWN_CASE)
    } else {
        constexpr bool APART = false;
        IOLB_SPLIT_SHAPES(IOLB_SPLIT_TWO_CASE)
        IOLB_SPLIT_SMALL_SHAPES(IOLB_SPLIT_CASE)
        IOLB_SPLIT_OWN_SHAPES(IOLB_SPLIT_OWN_CASE)
    }
#undef IOLB_SPLIT_OWN_CASE
#undef IOLB_SPLIT_CASE
#undef IOLB_SPLIT_TWO_CASE
#undef IOLB_SPLIT_IS
    return hipErrorInvalidValue;
}

hipError_t launch_split_conv(const float* x, const void* wt, const float* w_given, float* y, const SplitGeom& g, bool own, bool transposed, hipStream_t st)
{
    // what the kernel assumes of its geometry
    if (g.b * g.tx * g.ty > 16 * g.nb * g.wn || split_lds_bytes(g, own) > 160 * 1024 || g.Kb16 != g.nbk * g.mb * g.wm ||
        (split_chunks(g) > 1 && split_batches(g) > split_steps(g)) || g.nbuf < (split_chunks(g) > 1 ? 2 : 1) || g.nbuf > 2 || (g.ch8 != 1 && g.ch8 != 2 && g.ch8 != 4) ||
        4LL * g.b * g.C * g.H * g.W >= (1LL << 31) || g.cstep != (g.hwc ? 4 : 4 * g.H * g.W) || (g.vec_in && (!g.hwc || g.C % 4)) || (g.parts != 2 && g.parts != 3) || (g.parts == 2 && (g.ch8 == 1 || own)))
        return hipErrorInvalidValue;
    const u32x4* w = static_cast<const u32x4*>(wt);
    SplitDivisors dv;
    SplitOwn o;
    if (!split_divisors(g, transposed, &dv, &o)) return hipErrorInvalidValue;
    o.w = w_given;
    return g.vec_in ? launch_shape<true>(x, w, y, g, dv, own, o, st) : launch_shape<false>(x, w, y, g, dv, own, o, st);
}

}  // namespace iolb
