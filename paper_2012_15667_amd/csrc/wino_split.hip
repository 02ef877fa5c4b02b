// Winograd F(2 x 2, 3 x 3) and F(4 x 4, 3 x 3) in one kernel on the 16-bit matrix cores at fp32 precision (operands in two
// fp16 parts, of few channels in three of bf16: split_mfma.h).  A workgroup of eight waves takes TB sub-domains by Z kernels in every one
// of the (m + 2)^2 planes; the channel sums of all planes stay in registers until the last channel, so that V and M never leave the chip.
//
// A stage is 16 channels, one contraction of a 32x32x16 matrix instruction.  Each thread transforms TB / 32 windows of inputs
// (loaded one stage ahead) and puts V in LDS in fp32, in one of two buffers; each wave multiplies PL / 8 planes: it cuts its V
// into parts between the matrix instructions of the plane before, and takes the transformed kernels, already in parts, from
// the L2 into registers some units ahead.  Each V is cut once and each kernel part read once per workgroup.
//
// Two parts: inputs are scaled before their transform, per image of the block by a sample of its first stage and a few channels more;
// kernels per kernel, their planes brought to the same size.  A sub-domain whose windows are all too small for the scale, like a sum that
// is not finite, has its block taken again; so has one of whose sums in a plane none reaches the line of its kernel (split_mfma.h), from the
// parts, and where these do not hold the kernel, from the caller's.  Lines and looking at them cost 1 us of 50 (256 -> 256 at 14 x 14).
//
// What bounds it, F(4 x 4), 32 x 64, 128 -> 128 at 112 x 112, batch 64: of the 46 us that a block lives, 10 pass before its first product
// and 9 after its last, with one block on a unit; a stage takes 3.4, 1.7 of them products and waiting for kernel parts (147 KB from the L2), the rest
// the transform.  (Kernel parts from one place in place of the L2's: 2 % less; no scales: 1 %.)  Whole calls, fp32 way / three
// bf16 parts / this: that layer 859 / 581 / 496 us (119 TFLOP/s of the planes' products), F(4 x 4) 256 -> 256 at 14 x 14 87 / 60 / 52,
// F(2 x 2) 64 -> 64 at 28 x 28, batch 8 (three parts) 19.8 / 13.2.
// Channel sums through LDS two at a time, and no division by the planes' scales: 506 -> 496.
// Registers: F(4 x 4), 32 x 64 has 253 and spills 47 - 62 scalar ones, most of them of what is taken again; three parts 256 and spill 5
// vector ones (24 bytes a lane; 13 and 44 where columns are read one by one).
// A block that is taken again is so by all its waves, stage by stage without overlap: one such block adds its time (256 -> 256 at 14 x 14, F(4 x 4)
// 52 -> 178 us, 128 -> 128 at 56 x 56, batch 8, F(2 x 2) 35 -> 101), and where the caller's kernels are read in it, which is not tuned, several
// times that (channels and kernels balanced by 1e3: 490 and 390).  With three parts, of which one NaN cost 64 -> 155 us: the next stage's inputs
// and the next unit's kernels on their way in it gave 133, but one or two more registers were spilled and large finite layers took 0.5 %
// longer: not kept.
// Measured and not kept: four waves of twice the planes each; transform and loads spread between the matrix instructions
// of every wave in place of the two phases below (F(4 x 4), 256 -> 256 at 56 x 56 521 -> 666: 26 registers spilled);
// differences of the cut by v_dot2 (equal).
#include "kernels.h"
#include "split_mfma.h"
#include "split_weights.h"
#include "wino_mats.h"
#include "wino_transform.h"

namespace iolb {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
// M outputs of a row, at any float
template <int M> using row_of = float __attribute__((ext_vector_type(M), aligned(4)));

// B v for one column of a window, with the sums that two rows of B share taken once
template <int M>
__device__ __forceinline__ void input_transform_1d(float (&v)[M + 2])
{
    if constexpr (M == 2) {
        const float d0 = v[0], d1 = v[1], d2 = v[2], d3 = v[3];
        v[0] = d0 - d2; v[1] = d1 + d2; v[2] = d2 - d1; v[3] = d1 - d3;
    } else {
        const float d0 = v[0], d1 = v[1], d2 = v[2], d3 = v[3], d4 = v[4], d5 = v[5];
        v[0] = __builtin_fmaf(4.f, d0, __builtin_fmaf(-5.f, d2, d4));
        const float p = __builtin_fmaf(-4.f, d2, d4), q = __builtin_fmaf(-4.f, d1, d3);
        v[1] = p + q; v[2] = p - q;
        const float r = d4 - d2, t = d3 - d1;
        v[3] = __builtin_fmaf(2.f, t, r); v[4] = __builtin_fmaf(-2.f, t, r);
        v[5] = __builtin_fmaf(4.f, d1, __builtin_fmaf(-5.f, d3, d5));
    }
}
// A v: n values in, M out
template <int M>
__device__ __forceinline__ void output_transform_1d(const float (&v)[M + 2], float (&o)[M])
{
    if constexpr (M == 2) {
        o[0] = v[0] + v[1] + v[2];
        o[1] = v[1] - v[2] - v[3];
    } else {
        const float a = v[1] + v[2], b = v[1] - v[2], c = v[3] + v[4], d = v[3] - v[4];
        o[0] = v[0] + a + c;
        o[1] = __builtin_fmaf(2.f, d, b);
        o[2] = __builtin_fmaf(4.f, c, a);
        o[3] = __builtin_fmaf(8.f, d, b) + v[5];
    }
}

// Whether this lane's bit of a wave-uniform mask is set: a select reads the mask as it is.
__device__ __forceinline__ bool by_lane(unsigned long long mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

template <int M, int TB, int Z, int COLS, int PARTS>
__global__ void __launch_bounds__(512, M == 2 && TB == 32 && Z == 32 ? 4 : 2)
wino_split_kernel(const float* __restrict__ x, const u32x4* wt, float* __restrict__ y, WinoSplitGeom g, WinoSplitDivisors dv, const float* __restrict__ w_raw,
                  int raw)
{
    constexpr int n = M + 2, PL = n * n, ZB = Z / 32, TBB = TB / 32;
    constexpr int FP = PL / 8, LP = PL % 8;                  // whole planes per wave, planes left over: 4 ZB units for 8 waves
    constexpr int UNITS = FP * ZB + (LP ? 1 : 0);            // units (32 kernels of a plane) per wave
    constexpr int D = UNITS % 3 == 0 ? 3 : UNITS == 4 ? 2 : UNITS;       // units of kernels in flight
    constexpr int WIN = TB / 32;                             // windows per thread and stage
    constexpr int VBUF = PL * TB * 64;
    constexpr bool TWO = PARTS == 2;                         // operands in two fp16 parts, else in three of bf16
    constexpr unsigned UNIT = 1024u * PARTS;                 // bytes of a unit
    static_assert(LP == 0 || LP == 4, "left-over planes");
    // Inputs are scaled so that V, up to 100 and 4 times as large in F(4 x 4) and F(2 x 2), has the room above it that other operands have.
    // What a transform rounds off is not less than what V's parts lose, at most 2^-25, where a window has a value of 2^-5 and 2^-2.
    constexpr int TOP = M == 4 ? 3 : 7;
    constexpr float LEAST = M == 4 ? 0.03125f : 0.25f;
    // Sums are judged as split_mfma.h tells, the outputs of a sub-domain together: unmarked errors are 2^-21 of the largest of them, 2^-18 in
    // F(4 x 4) (in the root mean square; the transforms round off 2^-22 and 2^-19).
    constexpr float LINE = M == 4 ? HALF_LINE / 8 : HALF_LINE;
    extern __shared__ u32x4 lds16[];
    char* const lds = reinterpret_cast<char*>(lds16);
    // behind the buffers: whether a block is taken again; what undoes the kernels' scales; per image of the block the largest value of the
    // sample that sets its scale; per sub-domain the largest value of its windows, scaled; what the kernels' lines follow from
    int* const any = reinterpret_cast<int*>(lds + wino_split_buffers(M, TB));
    float* const kback = reinterpret_cast<float*>(any + 4);
    unsigned* const sample = reinterpret_cast<unsigned*>(kback + Z);
    unsigned* const most = sample + TB;
    KernelLine* const lines = reinterpret_cast<KernelLine*>(most + TB);
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int bid;
    {
        const int nblk = gridDim.x, q = nblk >> 3, r = nblk & 7, xcd = blockIdx.x & 7;
        bid = xcd * q + (xcd < r ? xcd : r) + ((int)blockIdx.x >> 3);
    }
    // an XCD stays with one block of kernels, whose parts its L2 holds
    const int kb = __builtin_amdgcn_readfirstlane(dv.small ? dv.nbt.of(bid) : bid / g.nbt);
    const int t0 = (bid - kb * g.nbt) * TB;
    const int per_image = g.th * g.tw, plane_in = g.H * g.W;
    auto image_of = [&](int t) { return dv.small ? dv.per_image.of(t) : t / per_image; };
    // a sub-domain's image, row and column
    auto place = [&](int t, int& img, int& ti, int& tj) {
        img = image_of(t);
        const int in = t - img * per_image;
        ti = dv.small ? dv.tw.of(in) : in / g.tw;
        tj = in - ti * g.tw;
    };
    const int img0 = __builtin_amdgcn_readfirstlane(image_of(t0));

    // inputs: byte offsets from the first image's window origin at (-pad, -pad)
    const int shift = g.pad * (g.W + 1);
    const size_t image = (size_t)g.C * plane_in;
    const int last_t = t0 + TB < g.tiles ? t0 + TB : g.tiles;
    const int span = __builtin_amdgcn_readfirstlane(image_of(last_t - 1) + 1 - img0);
    const unsigned long long xb = reinterpret_cast<unsigned long long>(x) + 4 * (img0 * image) - 4ull * shift;
    const unsigned xlo = __builtin_amdgcn_readfirstlane((unsigned)xb), xhi = __builtin_amdgcn_readfirstlane((unsigned)(xb >> 32));
    const unsigned xrange = __builtin_amdgcn_readfirstlane(wino_split_range(g, span));
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((unsigned long long)xhi << 32 | xlo), 0, (int)xrange, 0x00020000);
    const unsigned ubytes = __builtin_amdgcn_readfirstlane((unsigned)g.chunks * (unsigned)g.Kb32 * (UNIT * PL));
    const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4*>(wt), 0, (int)ubytes, 0x00020000);

    // this thread's windows: a wave takes 4 channels of 16 sub-domains, a row of 16 lanes each.  A lane loads the M columns
    // under its sub-domain's own place; the two border columns are its neighbours', those of lanes 0 and 15 are loaded.
    const int c0w = TB == 32 ? (wave >> 1) * 4 : (wave >> 2) * 8;
    const int tloc = (TB == 32 ? wave & 1 : wave & 3) * 16 + (lane & 15), cl = c0w + (lane >> 4);
    unsigned long long rowok[n], colok[M], left, right, edge;            // by lane: one register pair each, as the selects read them
    unsigned xoff, eoff;
    int image_in;                                           // of the block
    bool tile_exists;
    {
        const int t = t0 + tloc, tt = t < g.tiles ? t : t0;
        int img, ti, tj;
        place(tt, img, ti, tj);
        image_in = img - img0;
        tile_exists = t < g.tiles;
        const int h0 = ti * M - g.pad, w0 = tj * M - g.pad;
        auto lanes = [](bool v) { return __builtin_amdgcn_ballot_w64(v); };
#pragma unroll
        for (int i = 0; i < n; ++i) rowok[i] = lanes(t < g.tiles && h0 + i >= 0 && h0 + i < g.H);
#pragma unroll
        for (int j = 0; j < M; ++j) colok[j] = COLS == WINO_COLS_WHOLE ? ~0ull : lanes(w0 + 1 + j >= 0 && w0 + 1 + j < g.W);
        // (pad >= 1: beyond the first and the last sub-domain of a row there are zeros)
        left = lanes(tj > 0); right = lanes(tj + 1 < g.tw);
        const int e16 = lane & 15, we = w0 + (e16 == 0 ? 0 : M + 1);
        edge = lanes((e16 == 0 ? tj > 0 : e16 == 15 && tj + 1 < g.tw) && we >= 0 && we < g.W);
        xoff = 4u * (unsigned)(shift + (int)((img - img0) * (int)image) + (lane >> 4) * plane_in + h0 * g.W + w0);
        eoff = xoff + ((lane & 15) == 0 ? 0 : 4 * (M + 1));
    }
    typedef float Windows[WIN][n][n];                       // loads in flight: column 0 the edge, then the M own columns
    const int nst = g.chunks;
    auto load_x = [&](Windows& wx, int s) {
        static_range<0, WIN>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const int c0 = 16 * s + c0w + 4 * i;
            const unsigned long long have = __builtin_amdgcn_ballot_w64(16 * s + cl + 4 * i < g.C);
            static_range<0, n>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                const int so = wino_split_offset<COLS>(g, c0, r);
                const unsigned long long row = have & rowok[r];
                wx[i][r][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, (int)(by_lane(row & edge) ? eoff : OUTSIDE), so, 0));
                if constexpr (COLS != WINO_COLS_SINGLE && M == 4) {
                    const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)((by_lane(row) ? xoff : OUTSIDE) + 4), so, 0);
#pragma unroll
                    for (int j = 0; j < 4; ++j) wx[i][r][j + 1] = __uint_as_float(q[j]);
                } else if constexpr (COLS != WINO_COLS_SINGLE) {
                    const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(rx, (int)((by_lane(row) ? xoff : OUTSIDE) + 4), so, 0);
#pragma unroll
                    for (int j = 0; j < 2; ++j) wx[i][r][j + 1] = __uint_as_float(q[j]);
                } else {
#pragma unroll
                    for (int j = 0; j < M; ++j)
                        wx[i][r][j + 1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, (int)((by_lane(row & colok[j]) ? xoff : OUTSIDE) + 4 * (j + 1)), so, 0));
                }
            });
        });
    };
    // V in LDS: [plane][four channels][sub-domain][4]
    const int vw = cl / 4 * (TB * 16) + tloc * 16 + (cl & 3) * 4;
    float xs = 1.f, top = 0.f;                              // this thread's image's scale; the largest value of its windows, scaled
    auto transform = [&](Windows& wx, char* vb) {
        static_range<0, WIN>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if constexpr (COLS == WINO_COLS_CUT)
#pragma unroll
                for (int r = 0; r < n; ++r)
#pragma unroll
                    for (int j = 1; j < M; ++j) wx[i][r][j + 1] = by_lane(colok[j]) ? wx[i][r][j + 1] : 0.f;
            if constexpr (TWO)
#pragma unroll
                for (int r = 0; r < n; ++r)
#pragma unroll
                    for (int j = 0; j <= M; ++j) wx[i][r][j] *= xs;
#pragma unroll
            for (int r = 0; r < n; ++r) {
                const int e = __float_as_int(wx[i][r][0]);
                // row_shr:1 and row_shl:1: lanes without such a neighbour keep the edge
                const float lf = __int_as_float(__builtin_amdgcn_update_dpp(e, __float_as_int(wx[i][r][M]), 0x111, 0xf, 0xf, false));
                const float rg = __int_as_float(__builtin_amdgcn_update_dpp(e, __float_as_int(wx[i][r][1]), 0x101, 0xf, 0xf, false));
                wx[i][r][0] = by_lane(left) ? lf : 0.f;
                wx[i][r][n - 1] = by_lane(right) ? rg : 0.f;
                if constexpr (TWO)
#pragma unroll
                    for (int j = 0; j < n; ++j) top = __builtin_fmaxf(top, __builtin_fabsf(wx[i][r][j]));
            }
#pragma unroll
            for (int j = 0; j < n; ++j) {
                float c[n];
#pragma unroll
                for (int r = 0; r < n; ++r) c[r] = wx[i][r][j];
                input_transform_1d<M>(c);
#pragma unroll
                for (int r = 0; r < n; ++r) wx[i][r][j] = c[r];
            }
            char* d = vb + vw + i * (TB * 16);
#pragma unroll
            for (int r = 0; r < n; ++r) {
                input_transform_1d<M>(wx[i][r]);
#pragma unroll
                for (int j = 0; j < n; ++j) *reinterpret_cast<float*>(d + (r * n + j) * (TB * 64)) = wx[i][r][j];
            }
        });
    };
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // kernels: plane p of this wave, unit zb of it; the left-over unit
    const int xplane = 8 * FP + (ZB == 2 ? wave >> 1 : wave & 3), xzb = ZB == 2 ? wave & 1 : 0;
    const bool has_extra = LP && (ZB == 2 || wave < 4);
    const unsigned pstride = (unsigned)g.chunks * (unsigned)g.Kb32 * UNIT;
    auto unit_at = [&](int u, int s) {                      // byte offset of unit u (a constant) of stage s
        const unsigned at = (unsigned)(s * g.Kb32 + kb * ZB) * UNIT;
        if (LP && u == UNITS - 1) return at + (unsigned)xplane * pstride + xzb * UNIT;
        return at + (unsigned)(wave * FP + u / ZB) * pstride + u % ZB * UNIT;
    };
    u32x4 a[D][PARTS];
    auto load_u = [&](u32x4 (&f)[PARTS], unsigned at) {
#pragma unroll
        for (int p = 0; p < PARTS; ++p) f[p] = __builtin_amdgcn_raw_buffer_load_b128(ru, lane * 16 + 1024 * p, (int)at, 0);
    };

    f32x16 acc[FP][ZB][TBB], accx[TBB];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
#pragma unroll
            for (int p = 0; p < FP; ++p)
#pragma unroll
                for (int z = 0; z < ZB; ++z)
#pragma unroll
                    for (int b = 0; b < TBB; ++b) acc[p][z][b][i] = 0.f;
#pragma unroll
            for (int b = 0; b < TBB; ++b) accx[b][i] = 0.f;
        }
    };
    // the eight channels of this lane's half, of tile l32 (+ 32 b), of a plane
    const int r0 = half * (TB * 32) + l32 * 16;
    auto fetch = [&](float (&v)[8], const char* vplane, int b) {
        const f32x4 lo = *reinterpret_cast<const f32x4*>(vplane + r0 + b * 512), hi = *reinterpret_cast<const f32x4*>(vplane + r0 + TB * 16 + b * 512);
#pragma unroll
        for (int j = 0; j < 4; ++j) { v[j] = lo[j]; v[4 + j] = hi[j]; }
    };
    // Plane by plane; the next plane's operands are read and cut into parts between the matrix instructions of this one,
    // the unit after next is loaded part by part as the registers fall free.
    constexpr int PLANES = FP + (LP ? 1 : 0);
    auto multiply = [&](int s, const char* vb) {
        const int next = s + 1 < nst ? s + 1 : s;
        auto plane_at = [&](int p) { return vb + (LP && p == FP ? xplane : wave * FP + p) * (TB * 64); };
        u32x4 b[2][TBB][PARTS];
        f32x4 v[2];
        // pieces of four channels: 2 TBB of a plane
        auto fetch4 = [&](f32x4& o, int p, int piece) {
            o = *reinterpret_cast<const f32x4*>(plane_at(p) + r0 + (piece & 1) * (TB * 16) + (piece >> 1) * 512);
        };
        auto cut4 = [&](u32x4 (&o)[TBB][PARTS], const f32x4& f, int piece) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                unsigned part[3];
                if constexpr (TWO) half_pair(f[2 * j], f[2 * j + 1], part[0], part[1]);
                else               split_pair(f[2 * j], f[2 * j + 1], part[0], part[1], part[2]);
#pragma unroll
                for (int q = 0; q < PARTS; ++q) o[piece >> 1][q][2 * (piece & 1) + j] = part[q];
            }
        };
        static_range<0, TBB>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            fetch4(v[0], 0, 2 * t);
            fetch4(v[1], 0, 2 * t + 1);
            cut4(b[0], v[0], 2 * t);
            cut4(b[0], v[1], 2 * t + 1);
        });
        static_range<0, PLANES>([&](auto pc) {
            constexpr int p = decltype(pc)::value;
            constexpr bool EXTRA = LP && p == FP;
            constexpr int Z1 = EXTRA ? 1 : ZB;               // units of the plane here
            if (EXTRA && !has_extra) return;
            static_range<0, Z1>([&](auto zc) {
                constexpr int z = decltype(zc)::value, u = EXTRA ? UNITS - 1 : p * ZB + z, un = u + D;
                constexpr bool MORE = p + 1 < PLANES;
                constexpr int PIECES = MORE ? 2 * TBB / Z1 : 0;          // pieces of the next plane cut here
                __builtin_amdgcn_sched_barrier(0);
                static_range<0, PIECES>([&](auto ic) { fetch4(v[decltype(ic)::value & 1], p + 1, z * PIECES + decltype(ic)::value);
                                                       if constexpr (PIECES > 2) cut4(b[(p + 1) & 1], v[decltype(ic)::value & 1], z * PIECES + decltype(ic)::value); });
                if constexpr (PIECES <= 2)
                    static_range<0, PIECES>([&](auto ic) { cut4(b[(p + 1) & 1], v[decltype(ic)::value & 1], z * PIECES + decltype(ic)::value); });
                u32x4 (&f)[PARTS] = a[u % D];
                f32x16 (&c)[TBB] = EXTRA ? accx : acc[EXTRA ? 0 : p][EXTRA ? 0 : z];
                const bool load = !LP || un != UNITS - 1 || has_extra;
                const unsigned at = un < UNITS ? unit_at(un, s) : unit_at(un - UNITS, next);
                // the products, small ones first; each part of the kernels is loaded again after its last
                constexpr int PRODUCTS = TWO ? 3 : 6, PA[6] = {TWO ? 1 : 2, TWO ? 0 : 1, TWO ? 0 : 1, 0, 0, 0}, PB[6] = {0, 1, 0, 2, 1, 0};
                constexpr auto last = [](int q) { return q == 0 || q == 2 || q == 5; };
                static_range<0, PRODUCTS>([&](auto qc) {
                    constexpr int q = decltype(qc)::value;
#pragma unroll
                    for (int t = 0; t < TBB; ++t)
                        if constexpr (TWO)
                            c[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, f[PA[q]]), __builtin_bit_cast(f16x8, b[p & 1][t][PB[q]]), c[t], 0, 0, 0);
                        else
                            c[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f[PA[q]]), __builtin_bit_cast(bf16x8, b[p & 1][t][PB[q]]), c[t], 0, 0, 0);
                    if constexpr (last(q))
                        if (load) f[PA[q]] = __builtin_amdgcn_raw_buffer_load_b128(ru, lane * 16 + 1024 * PA[q], (int)at, 0);
                });
                // per matrix instruction its share of the vector work
                constexpr int VALU = ((TWO ? 6 : 26) * PIECES + PRODUCTS * TBB - 1) / (PRODUCTS * TBB) + 1;
#pragma unroll
                for (int i = 0; i < PRODUCTS; ++i) {
#pragma unroll
                    for (int t = 0; t < TBB; ++t) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        if constexpr (MORE) __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
                    }
                    if (last(i)) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };

    // Channel sums leave the registers 32 kernels at a time, through LDS: [plane][tile][kernel], 34 floats from tile to tile, so that a lane
    // writes and reads two kernels at once and 32 tiles reach every bank once; a thread then owns whole (kernel, tile) pairs.
    constexpr int PAIRS = 32 * TB / 512;
    static_assert(ZB * PAIRS <= 32, "one mark per pair");
    unsigned again = 0;                                      // pairs that are taken again
    bool again_root = false;                                 // (the second time: and once more those below what their kernel's small elements may have lost)
    auto finish = [&](auto marked_c) {
        constexpr bool MARKED = decltype(marked_c)::value;   // the second time: marked pairs only
        float* const m = reinterpret_cast<float*>(lds);
        static_range<0, ZB>([&](auto zc) {
            constexpr int z = decltype(zc)::value;
            if constexpr (z) barrier();
            auto put = [&](int plane, const f32x16 (&c)[TBB]) {
                const float scale = MARKED ? 1.f : TWO ? row_down<M>(plane / n) * row_down<M>(plane % n) : SPLIT_UNSCALE;
#pragma unroll
                for (int t = 0; t < TBB; ++t)
#pragma unroll
                    for (int i = 0; i < 16; i += 2)
                        *reinterpret_cast<f32x2*>(m + (plane * TB + 32 * t + l32) * 34 + 8 * (i >> 2) + (i & 3) + 4 * half) = f32x2{c[t][i] * scale, c[t][i + 1] * scale};
            };
            static_range<0, FP>([&](auto pc) { put(wave * FP + decltype(pc)::value, acc[decltype(pc)::value][z]); });
            if constexpr (LP != 0)
                if (has_extra && xzb == z) put(xplane, accx);
            barrier();
            const int tl = opaque(tid) % TB, t = t0 + tl;
            int img, ti, tj;
            place(t, img, ti, tj);
            const int h0 = ti * M, w0 = tj * M;
            float back = 1.f, input = 0.f;
            bool lost = false;
            if constexpr (TWO) {
                back = half_unscale(half_scale_bits<TOP>(sample[t < g.tiles ? img - img0 : 0]));
                input = __uint_as_float(most[tl]);
                lost = most[tl] - 1 < __float_as_uint(LEAST) - 1;
            }
#pragma unroll
            for (int i2 = 0; i2 < PAIRS / 2; ++i2) {
                const int kl2 = 2 * (tid / TB + i2 * (512 / TB));
                f32x2 both[n][n];
#pragma unroll
                for (int r = 0; r < n; ++r)
#pragma unroll
                    for (int j = 0; j < n; ++j) both[r][j] = *reinterpret_cast<const f32x2*>(m + ((r * n + j) * TB + tl) * 34 + kl2);
#pragma unroll
                for (int q2 = 0; q2 < 2; ++q2) {
                    const int kl = kl2 + q2, k = kb * Z + 32 * z + kl, bit = z * PAIRS + 2 * i2 + q2;
                    float v[n][n];
#pragma unroll
                    for (int r = 0; r < n; ++r)
#pragma unroll
                        for (int j = 0; j < n; ++j) v[r][j] = both[r][j][q2];
                    float h[n][M], o[M][M];
#pragma unroll
                    for (int r = 0; r < n; ++r) output_transform_1d<M>(v[r], h[r]);
#pragma unroll
                    for (int j = 0; j < M; ++j) {
                        float c[n], q[M];
#pragma unroll
                        for (int r = 0; r < n; ++r) c[r] = h[r][j];
                        output_transform_1d<M>(c, q);
#pragma unroll
                        for (int r = 0; r < M; ++r) o[r][j] = q[r];
                    }
                    if (t >= g.tiles || k >= g.K) continue;
                    if constexpr (MARKED) {
                        if (!(again >> bit & 1)) continue;
                        if (TWO && again_root) {
                            float largest = 0.f;
#pragma unroll
                            for (int r = 0; r < M; ++r)
#pragma unroll
                                for (int j = 0; j < M; ++j) largest = __builtin_elementwise_maximum(largest, __builtin_fabsf(o[r][j]));
                            // (sums that are not finite are what they are)
                            if (!(largest < lines[32 * z + kl].root * input * back * kback[32 * z + kl])) again &= ~(1u << bit);
                        }
                    } else {
                        // (every plane enters an output)
                        float largest = 0.f;
#pragma unroll
                        for (int r = 0; r < M; ++r)
#pragma unroll
                            for (int j = 0; j < M; ++j) largest = __builtin_elementwise_maximum(largest, __builtin_fabsf(o[r][j]));
                        bool bad = lost || !(largest <= FINITE);
                        if constexpr (TWO) {
                            const KernelLine line = lines[32 * z + kl];
                            bad |= input > 0.f && !(largest >= line_of(line, input));
                        }
                        if (bad) again |= 1u << bit;
                        if constexpr (TWO) {
                            const float kscale = kback[32 * z + kl];
#pragma unroll
                            for (int r = 0; r < M; ++r)
#pragma unroll
                                for (int j = 0; j < M; ++j) o[r][j] = o[r][j] * back * kscale;
                        }
                    }
                    float* yp = y + ((size_t)img * g.K + k) * ((size_t)g.P * g.Q) + (size_t)h0 * g.Q + w0;
#pragma unroll
                    for (int r = 0; r < M; ++r) {
                        if (h0 + r >= g.P) break;
                        if (w0 + M <= g.Q) {
                            row_of<M> v;
#pragma unroll
                            for (int j = 0; j < M; ++j) v[j] = o[r][j];
                            *reinterpret_cast<row_of<M>*>(yp + (size_t)r * g.Q) = v;
                        } else {
#pragma unroll
                            for (int j = 0; j < M; ++j)
                                if (w0 + j < g.Q) yp[(size_t)r * g.Q + j] = o[r][j];
                        }
                    }
                }
            }
        });
    };

    // Waves w and w + 4 share a SIMD.  The first transforms the next stage after it has multiplied this one, the second
    // before, so that one's vector work runs beside the other's matrix work: the second is one transform ahead and
    // meets the barrier between the two.
    const bool ahead = wave >= 4;
    Windows wx;
    {
        // before there are sums the registers hold two stages' windows: both are on their way before the first is waited for
        Windows first;
        load_x(first, 0);
        // for the sample beside the first stage a value of each sub-domain from other channels, a wave four of them; the kernels' scales
        float spread = 0.f, my_kback = 0.f;
        FactsShare<2> share;                                   // (of the kernels' facts, a piece per stage)
        if constexpr (TWO) {
            const int sc = wave * g.C >> 3;
            const unsigned long long have = __builtin_amdgcn_ballot_w64(sc + (lane >> 4) < g.C) & rowok[1] & colok[0];
            spread = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, (int)((by_lane(have) ? xoff : OUTSIDE) + 4), wino_split_offset<COLS>(g, sc, 1), 0));
            const float* const scales = reinterpret_cast<const float*>(reinterpret_cast<const char*>(wt) + (size_t)PL * pstride);
            if (tid < Z) my_kback = scales[kb * Z + tid];
            share.load(reinterpret_cast<const KernelFacts*>(scales + 32 * g.Kb32) + kb * Z + tid % Z, tid / Z, 512 / Z, nst, 32 * g.Kb32);
        }
        static_range<0, D>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            if (!LP || u < UNITS - 1 || has_extra) load_u(a[u], unit_at(u, 0));
        });
        load_x(wx, 1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (TWO) {
            if (tid < 2 * TB) sample[tid] = 0;                  // (most follows)
            barrier();
            unsigned largest = finite_bits(spread);
            static_range<0, WIN>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
#pragma unroll
                for (int r = 0; r < n; ++r)
#pragma unroll
                    for (int j = 0; j < M; ++j) {
                        const unsigned m = COLS == WINO_COLS_CUT && !by_lane(colok[j]) ? 0u : finite_bits(first[i][r][j + 1]);
                        largest = m > largest ? m : largest;
                    }
            });
            if (span == 1) {
                largest = wave_max(largest);
                if (lane == 0) atomicMax(sample, largest);
            } else if (tile_exists && largest) {
                atomicMax(sample + image_in, largest);
            }
            if (tid < Z) kback[tid] = my_kback;
            // (in the buffer that the second stage goes to)
            KernelFacts* const shares = reinterpret_cast<KernelFacts*>(lds + VBUF);
            static_assert(VBUF >= 512 * (int)sizeof(KernelFacts), "room for the shares");
            shares[tid] = share.sum();
            barrier();
            if (tid < Z) {
                const KernelLine line = kernel_line(all_shares<Z, 512 / Z>(shares, tid), LINE);
                constexpr float growth = input_growth<M>();
                lines[tid] = {line.norm, growth * line.root};
            }
            xs = __uint_as_float(half_scale_bits<TOP>(sample[image_in]));
        }
        transform(first, lds);
    }
    __builtin_amdgcn_sched_barrier(0);
    barrier();
    if (ahead) {
        if (1 < nst) transform(wx, lds + VBUF);
        load_x(wx, 2);
        __builtin_amdgcn_sched_barrier(0);
    }
    clear();
#pragma unroll 1
    for (int s = 0; s < nst; ++s) {
        multiply(s, lds + (s & 1) * VBUF);
        if (ahead) barrier();
        const int ts = ahead ? s + 2 : s + 1;
        if (ts < nst) {
            transform(wx, lds + (ts & 1) * VBUF);
            load_x(wx, ts + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!ahead) barrier();
    }
    if constexpr (TWO)
        if (tile_exists) atomicMax(most + tloc, __float_as_uint(top));
    if (tid == 0) *any = 0;
    barrier();
    finish(std::false_type{});
    barrier();
    if (again) *any = 1;
    barrier();
    if (__builtin_amdgcn_readfirstlane(*any) == 0) return;

    // The block again on the fp32 matrix instructions, from the same inputs.  Three parts hold all of a kernel, and so do two of most, unless they
    // are not finite: the caller's own is read then.  Sums that are below what the kernel's small elements may have lost are taken
    // once more, all of their kernels read from the caller's.
    xs = 1.f;
#pragma unroll 1
    for (bool careful = false;; careful = true) {
    clear();
#pragma unroll 1
    for (int s = 0; s < nst; ++s) {
        load_x(wx, s);
        transform(wx, lds);
        barrier();
        auto multiply4 = [&](int plane, int four, const float* w, f32x16 (&c)[TBB]) {
#pragma unroll
            for (int t = 0; t < TBB; ++t) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(lds + plane * (TB * 64) + r0 + four * (TB * 16) + t * 512);
#pragma unroll
                for (int j = 0; j < 4; ++j) c[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[j], v[j], c[t], 0, 0, 0);
            }
        };
        if constexpr (TWO) {
            static_range<0, ZB>([&](auto zc) {
                constexpr int z = decltype(zc)::value;
#pragma unroll 1
                for (int four = 0; four < 2; ++four) {
                    const int lane2 = opaque(lane), k = kb * Z + 32 * z + (lane2 & 31), c0 = 16 * s + 8 * (lane2 >> 5) + 4 * four;
                    float taps[4][9];
                    if (careful && raw == SPLIT_RAW_TAPS)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
#pragma unroll
                            for (int i = 0; i < 9; ++i) {
                                const bool exists = k < g.K && c0 + j < g.C;
                                taps[j][i] = w_raw[exists ? ((size_t)k * g.C + c0 + j) * 9 + i : 0];
                                taps[j][i] = exists ? taps[j][i] : 0.f;
                            }
                    auto unit = [&](int plane, f32x16 (&c)[TBB]) {
                        // (opaque: nothing of it is computed, and kept in scalar registers, through the loop above)
                        const int pl = __builtin_amdgcn_readfirstlane(opaque(plane + (four >> 1)));
                        const RawKernels kernels(w_raw, raw, M, pl, opaque(g.C), opaque(g.K));
                        float w[4];
                        bool whole = !careful;
                        if (!careful) {
                            const unsigned at = (unsigned)(s * g.Kb32 + kb * ZB + z) * UNIT + (unsigned)pl * pstride;
                            const u32x2 h = __builtin_amdgcn_raw_buffer_load_b64(ru, lane * 16 + 8 * four, (int)at, 0), l = __builtin_amdgcn_raw_buffer_load_b64(ru, lane * 16 + 8 * four + 1024, (int)at, 0);
                            const float back = kback[32 * z + l32] * (row_down<M>(pl / n) * row_down<M>(pl % n));
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                // (a bit_cast of an element of a vector reads its first one)
                                const unsigned hb = h[j / 2], lb = l[j / 2];
                                const f16x2 hj = __builtin_bit_cast(f16x2, hb), lj = __builtin_bit_cast(f16x2, lb);
                                w[j] = ((float)hj[j % 2] + (float)lj[j % 2]) * back;
                                whole = whole && __builtin_fabsf(w[j]) <= FINITE;
                            }
                        }
                        if (!whole)
#pragma unroll
                            for (int j = 0; j < 4; ++j) w[j] = careful && raw == SPLIT_RAW_TAPS ? kernels.of(taps[j]) : kernels.at(k, c0 + j);
                        multiply4(plane, four, w, c);
                    };
                    static_range<0, FP>([&](auto pc) { unit(wave * FP + decltype(pc)::value, acc[decltype(pc)::value][z]); });
                    if constexpr (LP != 0)
                        if (has_extra && xzb == z) unit(xplane, accx);
                }
            });
        } else {
            auto unit = [&](int u, int plane, f32x16 (&c)[TBB]) {
                u32x4 f[PARTS];
                float w[8];
                load_u(f, unit_at(u, s));
                kept_eight(f[0], f[1], f[PARTS - 1], w);
                multiply4(plane, 0, w, c);
                multiply4(plane, 1, w + 4, c);
            };
            static_range<0, FP * ZB>([&](auto uc) {
                constexpr int u = decltype(uc)::value;
                unit(u, wave * FP + u / ZB, acc[u / ZB][u % ZB]);
            });
            if constexpr (LP != 0)
                if (has_extra) unit(UNITS - 1, xplane, accx);
        }
        barrier();
    }
    if (tid == 0) *any = 0;
    again_root = !careful;
    finish(std::true_type{});
    if (!TWO || careful) return;
    barrier();
    if (again) *any = 1;
    barrier();
    if (__builtin_amdgcn_readfirstlane(*any) == 0) return;
    }
}

// What a lane's elements of a kernel in a plane tell, by the weight of its sums in an output.
__device__ __forceinline__ void add_weighted(KernelFacts& to, const KernelFacts& f, float weight)
{
    to.squares = __builtin_fmaf(weight * weight, f.squares, to.squares);
    to.small = __builtin_fmaf(weight * weight, f.small, to.small);
}
// All of a kernel's 16 channels, rows[row of planes][channels' half, kernel], in a fixed order.
template <int M>
__device__ __forceinline__ void store_facts(const KernelFacts (&rows)[M + 2][64], KernelFacts* to)
{
    __syncthreads();
    if (threadIdx.x >= 32) return;
    KernelFacts all = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < M + 2; ++i)
#pragma unroll
        for (int half = 0; half < 64; half += 32) {
            all.squares += rows[i][half + threadIdx.x].squares;
            all.small += rows[i][half + threadIdx.x].small;
        }
    to[threadIdx.x] = all;
}

// Kernels in two or three parts in the order of the kernel above: [plane][16 channels][32 kernels][part][lane][8 channels], and behind two
// parts what undoes the scales of 32 Kb32 kernels, and their facts, [16 channels][kernel].
// One workgroup per 16 channels of 32 kernels of w[K][C][3][3], a wave per row of the planes in turn.
template <int M, int PARTS>
__global__ void __launch_bounds__(256)
wino_split_weights(const float* __restrict__ w, u32x4* __restrict__ wt, int C, int K, int chunks, int Kb32)
{
    constexpr int n = M + 2, LEN = 16 * 9, PITCH = LEN + 1;
    __shared__ float rows[32 * PITCH];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kb = blockIdx.x % Kb32, ch = blockIdx.x / Kb32;
    const int have = C - ch * 16 < 16 ? (C - ch * 16) * 9 : LEN;
    __shared__ unsigned scales[32];
    __shared__ KernelFacts rows_facts[n][64];
    float some[8];                                          // each kernel's scale, the same in all of its workgroups
#pragma unroll
    for (int j = 0; j < 8; ++j) some[j] = PARTS == 2 ? sampled_value(w, kb * 32 + wave * 8 + j, K, C, lane) : 0.f;
    stage_kernels<32, 4, 3>(K > kb * 32 ? w + ((size_t)kb * 32 * C + ch * 16) * 9 : w, rows, wave, lane, C * 9LL, K - kb * 32, have, LEN, PITCH);
#pragma unroll
    for (int j = 0; j < (PARTS == 2 ? 8 : 0); ++j) {
        const unsigned s = half_scale_bits(wave_max(finite_bits(some[j])));
        if (lane == 0) scales[wave * 8 + j] = s;
    }
    __syncthreads();
    const float* mine = rows + (lane & 31) * PITCH + (lane >> 5) * 72;
    const unsigned scale = PARTS == 2 ? scales[lane & 31] : 0u;
    if (PARTS == 2 && ch == 0 && threadIdx.x < 32) reinterpret_cast<float*>(wt + (size_t)n * n * chunks * Kb32 * 128)[kb * 32 + threadIdx.x] = half_unscale(scale);
#pragma unroll 1
    for (int row = wave; row < n; row += 4) {
        float lg[8][3];                                     // this row of L g, for each channel
        kernel_row<M>(row, mine, lg);
        const float this_up = row_up<M>(row), this_weight = PARTS == 2 ? row_weight<M>(row) : 0.f;
        KernelFacts facts = {0.f, 0.f};
        static_for<n>([&](auto j) {
            constexpr int J = decltype(j)::value;
            if constexpr (PARTS == 3) {
                unsigned short p[3][8];
#pragma unroll
                for (int c = 0; c < 8; ++c) split_kept(kernel_element<M, J>(lg[c]), p[0][c], p[1][c], p[2][c]);
                store_parts(wt + (((size_t)(row * n + J) * chunks + ch) * Kb32 + kb) * 192 + lane, p);
                return;
            }
            constexpr float to_size = power_of_two(kernel_up<M>(J));
            const float up = __uint_as_float(scale) * this_up * to_size;
            float u[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) u[c] = kernel_element<M, J>(lg[c]) * up;
            const KernelFacts f = store_halves<32, false>(wt + (((size_t)(row * n + J) * chunks + ch) * Kb32 + kb) * 128 + lane, u, C - ch * 16, 3e38f);
            constexpr float weight = plane_weight<M>(J);
            add_weighted(facts, f, this_weight * weight);
        });
        if constexpr (PARTS == 2) rows_facts[row][lane] = facts;
    }
    if constexpr (PARTS == 2)
        store_facts<M>(rows_facts, reinterpret_cast<KernelFacts*>(reinterpret_cast<float*>(wt + (size_t)n * n * chunks * Kb32 * 128) + 32 * Kb32) + ((size_t)ch * Kb32 + kb) * 32);
}

// The same, to the same bits, from a caller's U[plane][C rounded up to 16][K rounded up to 32]: a wave per row of the planes.
template <int M, int PARTS>
__global__ void __launch_bounds__(64 * (M + 2))
wino_split_given(const float* __restrict__ U, u32x4* __restrict__ wt, int C, int K, int chunks, int Kb32)
{
    constexpr int n = M + 2;
    __shared__ KernelFacts rows_facts[n][64];
    const int lane = threadIdx.x & 63, row = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kb = blockIdx.x % Kb32, ch = blockIdx.x / Kb32;
    const int k = kb * 32 + (lane & 31), c0 = ch * 16 + (lane >> 5) * 8;
    const int rows = (C + 15) / 16 * 16, cols = (K + 31) / 32 * 32;
    const unsigned scale = PARTS == 2 ? scale_of_given<M, 32>(U, k, K, C, rows, cols, lane) : 0u;
    if (PARTS == 2 && ch == 0 && threadIdx.x < 32) reinterpret_cast<float*>(wt + (size_t)n * n * chunks * Kb32 * 128)[k] = half_unscale(scale);
    KernelFacts facts = {0.f, 0.f};
    float v[n][8];
#pragma unroll
    for (int j = 0; j < n; ++j)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const bool exists = k < K && c0 + c < C;
            v[j][c] = U[exists ? ((size_t)(row * n + j) * rows + c0 + c) * cols + k : 0];
            v[j][c] = exists ? v[j][c] : 0.f;
        }
    const float this_up = row_up<M>(row), this_weight = PARTS == 2 ? row_weight<M>(row) : 0.f;
    static_for<n>([&](auto j) {
        constexpr int J = decltype(j)::value;
        const size_t piece = ((size_t)(row * n + J) * chunks + ch) * Kb32 + kb;
        if constexpr (PARTS == 3) {
            unsigned short p[3][8];
#pragma unroll
            for (int c = 0; c < 8; ++c) split_kept(v[J][c], p[0][c], p[1][c], p[2][c]);
            store_parts(wt + piece * 192 + lane, p);
            return;
        }
        constexpr float to_size = power_of_two(kernel_up<M>(J));
            const float up = __uint_as_float(scale) * this_up * to_size;
        float u[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) u[c] = v[J][c] * up;
        const KernelFacts f = store_halves<32, false>(wt + piece * 128 + lane, u, C - ch * 16, 3e38f);
        constexpr float weight = plane_weight<M>(J);
        add_weighted(facts, f, this_weight * weight);
    });
    if constexpr (PARTS == 2) rows_facts[row][lane] = facts;
    if constexpr (PARTS == 2)
        store_facts<M>(rows_facts, reinterpret_cast<KernelFacts*>(reinterpret_cast<float*>(wt + (size_t)n * n * chunks * Kb32 * 128) + 32 * Kb32) + ((size_t)ch * Kb32 + kb) * 32);
}

template <int M, int TB, int Z, int COLS, int PARTS>
hipError_t launch_one(const float* x, const u32x4* wt, const float* w, int raw, float* y, const WinoSplitGeom& g, hipStream_t st)
{
    auto kern = wino_split_kernel<M, TB, Z, COLS, PARTS>;
    constexpr size_t shm = wino_split_buffers(M, TB) + 16 + 4 * Z + 8 * TB + 8 * Z;
    static_assert(shm <= 160 * 1024, "LDS");
    if (shm > 64 * 1024) {
        const hipError_t e = allow_large_lds((const void*)kern);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(g.nbt * g.nbk), dim3(512), shm, st, x, wt, y, g, wino_split_divisors(g), w, raw);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_wino_split_weights(const float* w, bool given, void* wt, const WinoSplitGeom& g, hipStream_t st)
{
    const long long blocks = (long long)g.chunks * g.Kb32;
    if (blocks >= (1LL << 25) || g.chunks * 16LL < g.C || g.Kb32 * 32LL < g.K) return hipErrorInvalidValue;
    u32x4* o = static_cast<u32x4*>(wt);
#define IOLB_CASE(M_, P_)                                                                                                                       \
    if (g.m == M_ && g.parts == P_) {                                                                                                           \
        if (given) hipLaunchKernelGGL((wino_split_given<M_, P_>), dim3((unsigned)blocks), dim3(64 * (M_ + 2)), 0, st, w, o, g.C, g.K, g.chunks, g.Kb32);  \
        else       hipLaunchKernelGGL((wino_split_weights<M_, P_>), dim3((unsigned)blocks), dim3(256), 0, st, w, o, g.C, g.K, g.chunks, g.Kb32); \
        return hipGetLastError();                                                                                                               \
    }
    IOLB_CASE(2, 2) IOLB_CASE(2, 3) IOLB_CASE(4, 2) IOLB_CASE(4, 3)
#undef IOLB_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_wino_split(const float* x, const void* wt, const float* w, bool given, float* y, const WinoSplitGeom& g, hipStream_t st)
{
    // what the kernel assumes of its geometry
    if (!wino_split_fits(g)) return hipErrorInvalidValue;
    const u32x4* u = static_cast<const u32x4*>(wt);
    const int cols = wino_split_cols(g), raw = given ? SPLIT_RAW_PLANES : SPLIT_RAW_TAPS;
#define IOLB_PARTS_CASE(M_, T_, Z_, P_)                                                                      \
    if (g.m == M_ && g.tb == T_ && g.z == Z_ && g.parts == P_)                                               \
        return cols == WINO_COLS_WHOLE ? launch_one<M_, T_, Z_, WINO_COLS_WHOLE, P_>(x, u, w, raw, y, g, st) \
               : cols == WINO_COLS_CUT ? launch_one<M_, T_, Z_, WINO_COLS_CUT, P_>(x, u, w, raw, y, g, st)   \
                                       : launch_one<M_, T_, Z_, WINO_COLS_SINGLE, P_>(x, u, w, raw, y, g, st);
#define IOLB_CASE(M_, T_, Z_) IOLB_PARTS_CASE(M_, T_, Z_, 2) IOLB_PARTS_CASE(M_, T_, Z_, 3)
    IOLB_WINO_SPLIT_SHAPES(IOLB_CASE)
#undef IOLB_PARTS_CASE
#undef IOLB_CASE
    return hipErrorInvalidValue;
}

}  // namespace iolb
