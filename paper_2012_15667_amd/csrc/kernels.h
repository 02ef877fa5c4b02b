// Internal launch interface between the C-ABI layer and the gfx950 kernels.
#ifndef IOLB_KERNELS_H
#define IOLB_KERNELS_H

#include <hip/hip_runtime.h>

#include <mutex>
#include <set>
#include <utility>

#include "iolbconv.h"

namespace iolb {

// Dynamic LDS above 64 KB needs an opt-in per kernel and device.  Done once for each pair; safe to call from
// several host threads.
inline hipError_t allow_large_lds(const void* kernel)
{
    static std::mutex guard;
    static std::set<std::pair<const void*, int>> done;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(guard);
    if (done.count({kernel, dev})) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess) done.insert({kernel, dev});
    return e;
}

// Geometry of one direct-convolution launch: the layer, the output sub-block b * tx * ty * z of
// Sec. 5.2 with its input tile xh * yh (x' * y' in the paper), and the block counts.
struct DirectGeom {
    int N, C, H, W, K, R, S, stride, pad, P, Q;   // pad: rows of zeros above and below
    int pad_w;                 // columns of zeros left and right (= pad except for conv_direct_pad2)
    int Kp;                    // MFMA path: K rounded up to a multiple of 32 (pitch of wt, extent of the z blocks)
    int b, tx, ty, z, alpha;
    int threads;               // workgroup size
    int waves_m, waves_n;      // MFMA path: wave grid; FMA path: channel groups, 1
    int per_thread;            // FMA path: output channels per lane
    int nbx, nby, nbn, nbk;    // blocks along W_out, H_out, batch, C_out
    int xh, yh, halo;          // input tile extents and elements per channel (b * yh * xh)
    int flat;                  // MFMA path, set by the launcher: input tile staged in flat 64-element chunks
    int w_transposed;          // weights are read with r and s exchanged: w[k][c][s'][r'] for this launch's (r', s')
    int hwc;                   // 0: x[N][C][H][W], y[N][K][P][Q];  1: x[N][H][W][C], y[N][P][Q][K]
};

// Re-layout w[K][C][R][S] -> wt[rows][Kp] (rows >= CRS = C*R*S, Kp >= K; rows beyond CRS and columns
// beyond K are zero) so that a stage's weight slab is a run of rows contiguous in K.
hipError_t launch_weight_relayout(const float* w, float* wt, int K, int Kp, int CRS, int rows, hipStream_t st);
// The same for a launch whose kernel extents (R, S) are the transposes of the stored weights' (S, R): row
// c*R*S + r*S + s of wt is taken from w[k][c][s][r].
hipError_t launch_weight_relayout_transposed(const float* w, float* wt, int K, int Kp, int C, int R, int S, int rows,
                                             hipStream_t st);

hipError_t launch_direct_fma(const float* x, const float* w, float* y, const DirectGeom& g, hipStream_t st);
// wt: re-laid-out weights with ceil(C/alpha)*alpha*R*S rows of g.Kp floats.
hipError_t launch_direct_mfma(const float* x, const float* wt, float* y, const DirectGeom& g, hipStream_t st);
// The same for the channels-innermost tensor layout (g.hwc = 1).
hipError_t launch_direct_mfma_hwc(const float* x, const float* wt, float* y, const DirectGeom& g, hipStream_t st);

// Direct convolution on the 16-bit matrix cores with operands in parts (direct_split.hip).
struct SplitGeom {
    int N, C, H, W, K, R, S, stride, pad, P, Q;
    int pad_w;
    int b, tx, ty;             // output sub-block: b images * ty rows * tx columns, at most 16 * nb * wn pixels
    int mb, nb, wm, wn;        // wave grid wm x wn, blocks of 16 channels x 16 pixels per wave mb x nb
    int ch8;                   // channels per chunk / 8: 1, 2 or 4
    int nbx, nby, nbn, nbk;    // blocks along W_out, H_out, batch, C_out
    int esy, esx;              // staged stride: min(stride, R), min(stride, S)
    int yh, xh;                // staged rows and columns per image
    int colw, rowp;            // columns of one residue class mod esx; elements of a staged row (esx * colw)
    int rowb;                  // bytes from one staged row to the next in LDS
    int halo;                  // b * yh * rowp
    int nbuf;                  // LDS buffers: 1 when the channels fit one chunk
    int Kb16;                  // 16-channel blocks, whole workgroup blocks
    int k_outer;               // blocks of one channel block are neighbours, not those of the same pixels
    int hwc, vec_in, vec_out;  // channels innermost; with 16-byte loads / stores of four channels
    int cstep;                 // bytes from an input channel to the next
    int parts;                 // of an operand: 3 of bf16, 2 of fp16
};
// Division by a number known on the host: exact for n * d < 2^31.  (The compiler's division takes some 40 instructions.)
struct Divisor {
    unsigned m;                // 2^31 / d, rounded down, + 1
    Divisor() = default;
    explicit Divisor(unsigned d) : m((1u << 31) / d + 1) {}
    __host__ __device__ int of(int n) const { return (int)((unsigned long long)((unsigned)n << 1) * m >> 32); }
};
// ... by the extents that the kernel divides by
struct SplitDivisors {
    Divisor ch8, halo, per, rowp, S, esx, esy, txy, tx;     // per: yh * rowp
    Divisor nbk, pixel_blocks, nbx, nby;                    // of workgroup ids, where small says that they are exact
    int small;
};
// ... and where workgroups prepare their own kernels (row: C * R * S; transposed: w[K][C][S][R])
struct SplitOwn {
    Divisor steps, row;
    int transposed;
    const float* w;            // the kernels as the caller holds them, for blocks that are taken again
    int facts;                 // pieces that a kernel's facts come in
};
constexpr int SPLIT_BATCH = 2;          // (pixel, 8 channels) items of the input tile that a thread stages at once
// The workgroup shapes that exist: blocks per wave (channels, pixels), wave grid (channels, pixels).  Of two with the same
// workgroup block and blocks per wave, which the planner's model cannot tell apart, there is one.
#define IOLB_SPLIT_SHAPES(X) \
    X(1, 2, 4, 1) X(1, 4, 4, 1) X(1, 8, 4, 1) X(2, 2, 4, 1) X(2, 4, 4, 1) X(2, 5, 4, 1) X(2, 7, 4, 1) X(2, 8, 4, 1) \
    X(3, 2, 4, 1) X(3, 4, 4, 1) X(4, 2, 4, 1)                                                                       \
    X(1, 2, 2, 2) X(1, 4, 2, 2) X(1, 7, 2, 2) X(1, 8, 2, 2) X(2, 5, 2, 2) X(2, 7, 2, 2) X(2, 8, 2, 2)             \
    X(3, 4, 2, 2) X(3, 5, 4, 1) X(3, 5, 2, 2)                                                                       \
    X(1, 1, 1, 4) X(1, 2, 1, 4) X(1, 4, 1, 4) X(1, 7, 1, 4) X(2, 7, 1, 4) X(3, 4, 1, 4)
// ... and those of them that small layers and short sums run in three parts
#define IOLB_SPLIT_SMALL_SHAPES(X) \
    X(1, 2, 4, 1) X(1, 4, 4, 1) X(2, 2, 4, 1) X(2, 4, 4, 1) X(2, 7, 4, 1) X(1, 2, 2, 2) X(1, 4, 2, 2) X(1, 8, 2, 2) X(1, 1, 1, 4)  \
    X(1, 2, 1, 4) X(1, 4, 1, 4) X(2, 8, 4, 1) X(3, 4, 4, 1) X(3, 4, 2, 2)
// ... and those for layers of at most eight channels (ch8 = 1)
#define IOLB_SPLIT_FEW_SHAPES(X) \
    X(1, 2, 4, 1) X(1, 4, 4, 1) X(1, 2, 2, 2) X(1, 4, 2, 2) X(2, 4, 2, 2) X(1, 2, 1, 4) X(1, 4, 1, 4) X(2, 4, 1, 4)
// ... and those with workgroups that prepare their own kernels
#define IOLB_SPLIT_OWN_SHAPES(X) X(1, 1, 1, 4) X(1, 2, 1, 4) X(1, 4, 1, 4) X(1, 2, 2, 2) X(1, 2, 4, 1)
#define IOLB_SPLIT_OWN_FEW_SHAPES(X) X(1, 2, 1, 4) X(1, 4, 1, 4)
inline int split_steps(const SplitGeom& g) { return (g.R * g.S * g.ch8 + 3) / 4; }
inline int split_chunks(const SplitGeom& g) { return (g.C + 8 * g.ch8 - 1) / (8 * g.ch8); }
inline int split_batches(const SplitGeom& g)
{
    const int per = 64 * g.wm * g.wn * SPLIT_BATCH;
    return (g.ch8 * g.halo + per - 1) / per;
}
// bytes in LDS of a pixel's eight channels: three parts one after the other; two in planes of their own, sixteen each
__host__ __device__ constexpr int split_pixel_bytes(int parts) { return parts == 2 ? 16 : 48; }
__host__ __device__ constexpr int split_planes(int parts) { return parts == 2 ? 2 : 1; }
// buffers of the input tile, offsets of the matrix steps' units, table of the input tile's elements, whole 16 bytes; of two parts
// also the kernels' scales and lines, the pixels' largest values and the images'
__host__ __device__ inline int split_two_bytes(const SplitGeom& g)
{
    return g.parts == 2 ? 64 * g.mb * g.wm + 128 * g.mb * g.wm + 4 * g.halo + 4 * (g.b > 4 ? g.b : 4) : 0;
}
__host__ __device__ inline int split_tables_bytes(const SplitGeom& g)
{
    const int steps = (g.R * g.S * g.ch8 + 3) / 4;
    return (g.nbuf * g.ch8 * split_planes(g.parts) * g.b * g.yh * g.rowb + 4 * ((4 * steps + 1) & ~1) + 8 * g.ch8 * g.halo + split_two_bytes(g) + 15) & ~15;
}
// ... and the parts and rows of a workgroup's own kernels
inline long long split_own_bytes(const SplitGeom& g)
{
    return (long long)split_chunks(g) * split_steps(g) * g.mb * g.wm * 3072 + 64LL * g.mb * g.wm * (g.C * g.R * g.S + 1LL);
}
inline long long split_lds_bytes(const SplitGeom& g, bool own = false)
{
    const long long tables = ((long long)g.nbuf * g.ch8 * split_planes(g.parts) * g.b * g.yh * g.rowb + 4 * ((4 * split_steps(g) + 1) & ~1) +
                              8LL * g.ch8 * g.halo + split_two_bytes(g) + 15) & ~15LL;
    return tables + (own ? split_own_bytes(g) : 0);
}
// The kernels' parts are written by workgroups of 16 kernels, some groups of eight channels and up to 16 taps: the pieces that what they tell
// of a kernel comes in (C in chunks of 8 ch8).
struct SplitPieces { int steps, octets, per, slices, pieces; };
inline SplitPieces split_pieces(int C, int RS, int ch8)
{
    SplitPieces p;
    p.steps = (RS * ch8 + 3) / 4;
    p.octets = (C + 8 * ch8 - 1) / (8 * ch8) * ch8;
    const int taps = 4 * p.steps / ch8;
    p.per = taps < 16 ? 16 / taps : 1;
    p.slices = (taps + 15) / 16;
    p.pieces = (p.octets + p.per - 1) / p.per * p.slices;
    return p;
}
inline int split_facts(int C, int RS, int ch8) { return split_pieces(C, RS, ch8).pieces; }
// What the kernel divides by.  Divided are items, units and pixels of a block (what is in LDS per item and unit bounds them by 2^15,
// their divisors too), and workgroup ids, where there are few enough.  False for a geometry beyond that.
inline bool split_divisors(const SplitGeom& g, bool transposed, SplitDivisors* dv, SplitOwn* own)
{
    if ((long long)g.ch8 * g.halo > 32768 || split_steps(g) * 4LL > 32768 || g.S > 32768) return false;
    const unsigned pixel_blocks = (unsigned)(g.nbx * g.nby * g.nbn);
    const bool small = (long long)pixel_blocks * g.nbk <= 32768;
    *dv = {Divisor(g.ch8), Divisor(g.halo), Divisor(g.yh * g.rowp), Divisor(g.rowp), Divisor(g.S), Divisor(g.esx), Divisor(g.esy), Divisor(g.tx * g.ty),
           Divisor(g.tx), Divisor(g.nbk), Divisor(pixel_blocks), Divisor(g.nbx), Divisor(g.nby), small};
    *own = {Divisor(split_steps(g)), Divisor(g.C * g.R * g.S), transposed ? 1 : 0, nullptr, split_facts(g.C, g.R * g.S, g.ch8)};
    return true;
}
// The input-tile buffer of a chunk: never one that split_lds_bytes does not count.
__host__ __device__ constexpr int split_buffer(int chunk, int nbuf) { return chunk & (nbuf - 1); }
static_assert(split_buffer(0, 1) == 0 && split_buffer(1, 1) == 0 && split_buffer(0, 2) == 0 && split_buffer(1, 2) == 1 && split_buffer(2, 2) == 0,
              "one buffer or two in turn");
// Room for the kernels, of which two parts with their exponents use less.  (What conv_direct_noalloc has room for follows from it.)
inline long long split_weight_bytes(const SplitGeom& g) { return (long long)split_chunks(g) * split_steps(g) * g.Kb16 * 3072; }
// Kernels in two or three parts in the order of the matrix steps, written from w[K][C][R][S] (transposed: w[K][C][S][R]); of two parts
// what undoes the scales of 16 Kb16 kernels follows, and their facts, [piece][kernel].
hipError_t launch_split_weights(const float* w, void* wt, int K, int C, int R, int S, int ch8, int Kb16, int parts, bool transposed, hipStream_t st);
// (own: the kernels themselves, transposed as above, in place of wt)
hipError_t launch_split_conv(const float* x, const void* wt, const float* w, float* y, const SplitGeom& g, bool own, bool transposed, hipStream_t st);

// 1 x 1 layers and the Winograd product on the same matrix cores (split_point.hip): per group of images that share
// kernels (all images of a layer; one transformed plane), y[K][HW] = w[K][C] x[C][HW] over the group's pixels.
struct SplitPointGeom {
    int groups, images;        // groups, images per group
    int C, K, Ky;              // Ky: channel planes per image of y (>= K)
    int HW, HWy, HWin, Win, Q, stride;   // output pixels per image, pitch of an output plane; input plane, row lengths and stride
    int mb, nb, wm, wn;        // wave grid wm x wn, blocks of 16 channels x 16 pixels per wave mb x nb
    int nbk, nbp;              // blocks along the channels, along a group's pixels
    int Kb16;                  // 16-channel blocks in the re-laid-out kernels
    long long w_image;         // 16-byte pieces from one group's kernels to the next
    int hwc, in, vec_out;      // in: how the inputs are read, below
    int raw, m;                // the kernels as the caller holds them, below; tile edge where they are transformed
    int per, pieces;           // pixels of an image that have one scale; pieces that a kernel's facts come in
};
// Inputs read in single floats; four channels at a time (channels innermost, C a multiple of 4, 16-byte aligned); two
// neighbouring pixels at a time (channels outermost, stride 1; blocks may run on into the next image only where HW is
// even).
// (the caller's kernels: w[K][C]; transformed w[plane][C rounded up to 16][K rounded up to 32]; w[K][C][3][3], to be transformed)
enum { SPLIT_RAW_ROWS = 0, SPLIT_RAW_PLANES = 1, SPLIT_RAW_TAPS = 2 };
enum { SPLIT_IN_SINGLE = 0, SPLIT_IN_CHANNELS = 1, SPLIT_IN_PIXELS = 2 };
constexpr int split_point_pixels(int in) { return in == SPLIT_IN_PIXELS ? 2 : 1; }
#define IOLB_SPLIT_POINT_SHAPES(X) X(1, 2, 4, 1) X(1, 4, 4, 1) X(2, 4, 4, 1) X(3, 4, 4, 1) X(4, 4, 4, 1)
// Room for a group's kernels in two parts, which they and what undoes their scales do not fill.
inline long long split_point_weight_bytes(const SplitPointGeom& g) { return (g.C + 31LL) / 32 * g.Kb16 * 3072; }
// wt: the kernels in two parts, per group [chunk][16-kernel block][part][lane] and behind them what undoes the scales of 16 Kb16 kernels
// and their facts, [piece][kernel];
// w: as the caller holds them (g.raw), for blocks that are taken again.
hipError_t launch_split_point(const float* x, const void* wt, const float* w, float* y, const SplitPointGeom& g, hipStream_t st);

// Thin layers (direct_thin.hip): 3 x 3 kernels, stride 1, C <= 4, plain NCHW tensors.  wk: K rows of
// direct_thin_row(C) floats (the 9 C elements of a kernel, zero-padded to whole 16-float pieces), 64-byte aligned,
// written from w by launch_direct_thin_rows.  Of g the layer, P, Q, pad and pad_w are used.
int direct_thin_row(int C);
hipError_t launch_direct_thin_rows(const float* w, float* wk, int K, int C, hipStream_t st);
hipError_t launch_direct_thin(const float* x, const float* wk, float* y, const DirectGeom& g, hipStream_t st);

// 1 x 1 convolution, no padding (pointwise_mfma.hip): per image y[K][HW] = w[K][C] x[C][HW] over the HW = P Q output
// pixels, whose inputs are the pixels (stride p, stride q) of the H x W planes.  A wave owns
// mbw x nbw blocks of 32 x 32 partial sums (z = 32 mbw channels by 32 nbw pixels of one image); a workgroup is
// `waves` waves on consecutive pixel ranges.  w: the kernels [K][Cw], Cw a multiple of 4 and 16-byte aligned rows
// (the caller's own w when C is a multiple of 4, else a copy with zeros in [C, Cw): launch_pointwise_weight_pad).
struct PointGeom {
    int N, C, HW, K;           // HW: output pixels per image
    int HWin, Win, Q, stride;  // input plane size and row length, output row length, stride (HWin = HW for stride 1)
    int Kp;                    // K rounded up to a multiple of z
    int Cw;                    // floats per kernel in w: C rounded up to a multiple of 4
    int z, mbw, nbw;
    int waves;                 // 4
    int alpha;                 // channels per stage: 16, 32 or 64 (twice the depth of the input ring)
    int tiles_per_image;       // ceil(HW / (32 nbw))
    int nbk;                   // Kp / z
    int npg;                   // workgroups along the pixels: ceil(N * tiles_per_image / waves)
};
hipError_t launch_pointwise_weight_pad(const float* w, float* wp, int K, int C, int Cw, hipStream_t st);
hipError_t launch_pointwise_mfma(const float* x, const float* w, float* y, const PointGeom& g, hipStream_t st);

// Winograd F(m x m, 3 x 3), unfused: kernel transform, input transform, batched product over the
// (m+2)^2 planes, output transform (steps 1-4 of Sec. 4.3).
struct WinoGeom {
    int N, C, H, W, K, m;
    int pad, P, Q;             // zero padding on every side; output extents P = H + 2 pad - 2, Q = W + 2 pad - 2
    int Cp;                    // C rounded up to whole stages: U and V carry zero rows for c in [C, Cp)
    int Kp;                    // K rounded up to a multiple of 32: U carries zero columns, M unused rows for k in [K, Kp)
    int CpU;                   // channel rows per plane of U (>= Cp; a caller-held U is padded to a multiple of 16)
    int th, tw;                // sub-domains along H_out and W_out
    int tiles;                 // N * th * tw
    int tiles_pitch;           // tiles rounded up to a whole number of blocks
    int tb, z, alpha;          // block: tb sub-domains by z channels of one plane
    int waves_m, waves_n;
};
hipError_t launch_wino_kernel_transform(const float* w, float* U, const WinoGeom& g, hipStream_t st);
// Input transform of x into V and, in the same launch, the kernels of the product: NONE (U is there already), PLAIN
// (U[xi][CpU][Kp] from w), or two fp16 parts for launch_split_point (groups = planes, Kb16 16-kernel blocks) from w
// (SPLIT) or from a caller's U[xi][C rounded up to 16][K rounded up to 32] in w's place (GIVEN).
enum { WINO_KERNELS_NONE, WINO_KERNELS_PLAIN, WINO_KERNELS_SPLIT, WINO_KERNELS_GIVEN };
hipError_t launch_wino_transforms(const float* x, float* V, const WinoGeom& g, const float* w, void* U, int kind, int Kb16, hipStream_t st);
hipError_t launch_wino_product(const float* U, const float* V, float* M, const WinoGeom& g, hipStream_t st);
hipError_t launch_wino_output_transform(const float* M, float* y, const WinoGeom& g, hipStream_t st);
// All four steps in one kernel, for C <= 4 with C * (m+2)^2 <= 128 (wino_fused.hip).  Its kernel-side
// factors are K rows of wino_fused_row(m, C) floats, Uk[k][xi * C + c], which launch_wino_fused_relayout
// makes from the plane-major U of launch_wino_kernel_transform.
int wino_fused_row(int m, int C);
hipError_t launch_wino_fused_relayout(const float* U, float* Uk, const WinoGeom& g, hipStream_t st);
hipError_t launch_wino_fused(const float* x, const float* Uk, float* y, const WinoGeom& g, hipStream_t st);

// All four steps in one matrix-core kernel for any channel count, m in {2, 4} (wino_fused_mfma.hip).  Its
// transformed kernels are U2[c / 2][xi][k][c % 2] with g.Cp rows (a multiple of g.alpha) and g.Kp columns (a
// multiple of g.z), written from w by launch_wino_kernel_transform_paired or re-laid out from a plane-major
// U[xi][rows][cols] by launch_wino_pair_relayout.  g.tb, g.z, g.alpha, g.waves_m, g.waves_n select the block.
hipError_t launch_wino_kernel_transform_paired(const float* w, float* U2, const WinoGeom& g, hipStream_t st);
hipError_t launch_wino_pair_relayout(const float* U, int rows, int cols, float* U2, const WinoGeom& g, hipStream_t st);
hipError_t launch_wino_fused_mfma(const float* x, const float* U2, float* y, const WinoGeom& g, hipStream_t st);
// The same with one wave per plane row and the input transform shared out over all threads (wino_fused_rows.hip).
hipError_t launch_wino_fused_rows(const float* x, const float* U2, float* y, const WinoGeom& g, hipStream_t st);

// All four steps in one kernel on the 16-bit matrix cores m in {2, 4} (wino_split.hip).
struct WinoSplitGeom {
    int N, C, H, W, K, m, pad, P, Q;
    int th, tw, tiles;         // sub-domains along H_out, W_out; in all
    int tb, z;                 // block: tb sub-domains by z kernels, every plane
    int nbt, nbk;              // blocks along the sub-domains, the kernels
    int chunks, Kb32;          // stages of 16 channels; 32-kernel blocks, whole workgroup blocks
    int parts;                 // of an operand: 3 of bf16, 2 of fp16
};
// ... and what it divides workgroup ids and sub-domains by, where small says that this is exact (per_image: th * tw)
struct WinoSplitDivisors {
    Divisor nbt, per_image, tw;
    int small;
};
inline WinoSplitDivisors wino_split_divisors(const WinoSplitGeom& g)
{
    const int per_image = g.th * g.tw;
    // (sub-domains of the last block may not exist: less than 64 of them)
    const bool small = (g.tiles + 64LL) * per_image < (1LL << 31) && (long long)g.nbt * g.nbk * g.nbt < (1LL << 31);
    return {Divisor(g.nbt), Divisor(per_image), Divisor(g.tw), small};
}
// LDS of its buffers: two of V, 64 bytes per plane and sub-domain, or the channel sums of 32 kernels, 34 floats
constexpr int wino_split_buffers(int m, int tb) { return (m + 2) * (m + 2) * tb * (34 * 4); }
#define IOLB_WINO_SPLIT_SHAPES(X) X(4, 32, 64) X(4, 32, 32) X(2, 64, 64) X(2, 32, 32)
inline long long wino_split_weight_bytes(const WinoSplitGeom& g) { return (g.m + 2LL) * (g.m + 2) * g.chunks * g.Kb32 * 3072; }
// Whether the kernel's 32-bit offsets reach: the images of a block, the kernels.
inline bool wino_split_fits(const WinoSplitGeom& g)
{
    const long long per = (long long)g.th * g.tw, span = (g.tb - 1 + per - 1) / per + 1;
    const long long images = span < g.N ? span : g.N;
    return g.pad >= 1 && 4 * (images * g.C * g.H * g.W + g.pad * (g.W + 1LL)) < (1LL << 31) && wino_split_weight_bytes(g) < (1LL << 31) && g.chunks == (g.C + 15) / 16 &&
           g.nbk * (g.z / 32) == g.Kb32 && g.Kb32 * 32LL >= g.K && (long long)g.nbt * g.tb >= g.tiles && (long long)g.nbt * g.nbk <= 0x7fffffffLL &&
           per * g.N == g.tiles && (long long)g.nbt * g.tb < (1LL << 31);
}
// Bytes of the buffer that a block's inputs are read from, `images` of them, from the first window's origin at (-pad, -pad) on.
__host__ __device__ inline unsigned wino_split_range(const WinoSplitGeom& g, int images)
{
    return 4u * ((unsigned)images * (unsigned)(g.C * g.H * g.W) + (unsigned)(g.pad * (g.W + 1)));
}
// How a lane's own columns are read: one by one; M at a time, those beyond the image's last column (in the last sub-domain of
// a row) zeroed afterwards; M at a time, all inside.  Images of so few rows that the last ones of every window lie below them are read
// one by one, too.  (Loads and stores of M floats need no more than the alignment of one; each float is checked against the buffer's
// range, the scalar offset included: measured with loads across the end of a range inside a larger buffer.)
enum { WINO_COLS_SINGLE, WINO_COLS_CUT, WINO_COLS_WHOLE };
inline int wino_split_cols(const WinoSplitGeom& g)
{
    return g.pad != 1 || g.H + g.pad < g.m + 2 ? WINO_COLS_SINGLE : g.W % g.m ? WINO_COLS_CUT : WINO_COLS_WHOLE;
}
// The scalar byte offset at which channel c0 (and the next three) and row r of the windows are loaded.  Never beyond the range of
// even one image: the hardware checks a lane's own offset against the range less this one, which must not wrap.  Rows that lie
// below every window's image (r >= H + pad; only read one by one) and channels that do not exist are masked in every lane.
template <int COLS>
__host__ __device__ inline int wino_split_offset(const WinoSplitGeom& g, int c0, int r)
{
    const int last = g.H + g.pad - 1, row = COLS == WINO_COLS_SINGLE && r > last ? last : r;
    return 4 * ((c0 < g.C ? c0 : 0) * (g.H * g.W) + row * g.W);
}
// The kernels in two (which do not fill their room) or three parts, from w[K][C][3][3] or (given) from a caller's U[plane][C rounded up to 16][K to 32].
hipError_t launch_wino_split_weights(const float* w, bool given, void* wt, const WinoSplitGeom& g, hipStream_t st);
// (w, given: what they were made from, for blocks that are taken again)
hipError_t launch_wino_split(const float* x, const void* wt, const float* w, bool given, float* y, const WinoSplitGeom& g, hipStream_t st);

// Ceiling probes (probe.hip).  The copy moves bytes / 16 16-byte pieces; the MFMA loop runs
// PROBE_MFMA_BLOCKS workgroups of four waves, each wave PROBE_ACC MFMAs (4096 flop each) per iteration, and
// writes PROBE_MFMA_BLOCKS * 256 floats to sink.
constexpr int PROBE_COPY_BLOCKS = 8192;
constexpr int PROBE_MFMA_BLOCKS = 1024;
constexpr int PROBE_ACC = 8;
hipError_t launch_probe_copy(const void* src, void* dst, size_t bytes, hipStream_t st);
hipError_t launch_probe_mfma(float* sink, int iters, hipStream_t st);
// Waves of two kinds side by side on every SIMD: `slots` waves per SIMD, slot s playing role (roles >> 2 s) & 3;
// ticks gets PROBE_SHARE_BLOCKS * 16 clock counts (one per wave, unused ones untouched), sink one float.
constexpr int PROBE_SHARE_BLOCKS = 256;
constexpr unsigned PROBE_ROLE_MFMA = 0, PROBE_ROLE_VALU = 1;
hipError_t launch_probe_share(unsigned long long* ticks, float* sink, int slots, unsigned roles, int iters, hipStream_t st);

}  // namespace iolb

#endif
