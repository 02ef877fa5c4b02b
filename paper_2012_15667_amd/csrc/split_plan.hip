// The block of a layer on the split matrix-core kernel (direct_split.hip): host only.
#include "split_plan.h"
#include "tune.h"

#include <algorithm>
#include <cmath>
#include <limits>
#include <vector>

namespace iolb {

bool split_derive(SplitGeom* g)
{
    g->esy = std::min(g->stride, g->R);
    g->esx = std::min(g->stride, g->S);
    const long long yh = (long long)(g->ty - 1) * g->esy + g->R, xh = (long long)(g->tx - 1) * g->esx + g->S;
    if (yh * xh * g->b > 8192) return false;
    g->yh = (int)yh;
    g->xh = (int)xh;
    g->colw = (g->xh + g->esx - 1) / g->esx;
    g->rowp = g->colw * g->esx;
    g->halo = g->b * g->yh * g->rowp;
    const int z = 16 * g->mb * g->wm;
    g->nbk = (g->K + z - 1) / z;
    g->Kb16 = g->nbk * g->mb * g->wm;
    g->nbx = (g->Q + g->tx - 1) / g->tx;
    g->nby = (g->P + g->ty - 1) / g->ty;
    g->nbn = (g->N + g->b - 1) / g->b;
    if ((long long)g->nbk * g->nbx * g->nby * g->nbn > 0x7fffffffLL) return false;
    // kernels of 3 MiB and more do not stay in an L2 of 4 MiB beside the inputs: then an XCD works on one channel block
    // at a time (512 -> 512 at 28 x 28, 14 MB of kernels: 1140 -> 1118 us; 256 -> 256 at 56 x 56, 3.5 MB: 1068 -> 1052;
    // 256 -> 512 at 28 x 28: equal).  Measured with three parts; the bytes are those of three parts in two as well, half as much
    // again as these take, so that in two parts the line lies at 2 MiB.
    g->k_outer = g->nbk > 1 && split_weight_bytes(*g) >= (3LL << 20);
    g->nbuf = split_chunks(*g) > 1 ? 2 : 1;
    if (g->b * g->tx * g->ty > 16 * g->nb * g->wn) return false;
    if (4LL * g->b * g->C * g->H * g->W >= (1LL << 31)) return false;
    g->cstep = g->hwc ? 4 : 4 * g->H * g->W;
    if (split_chunks(*g) > 1 && split_batches(*g) > split_steps(*g)) return false;
    // Sixteen lanes read 16 bytes each of consecutive pixels, 48 bytes apart (16 in two parts): that covers every LDS bank once.  A row
    // pitch that is congruent to the bytes of a tile row modulo the 256 bytes of the banks keeps it so across a row
    // end; taken where it does not cost a resident workgroup.
    const int px = split_pixel_bytes(g->parts);
    g->rowb = g->rowp * px;
    const long long tight = split_lds_bytes(*g);
    if (g->ty * g->b > 1) {
        int padded = g->rowb;
        while ((g->esy * padded - px * g->tx) % 256 && padded < g->rowb + 256) padded += 16;
        if ((g->esy * padded - px * g->tx) % 256 == 0) {
            SplitGeom t = *g;
            t.rowb = padded;
            const long long full = 160 * 1024;
            if (split_lds_bytes(t) <= full && std::min(full / split_lds_bytes(t), 2LL) == std::min(full / tight, 2LL)) g->rowb = padded;
        }
    }
    return split_lds_bytes(*g) <= 160 * 1024;
}

// Modelled clock cycles of a layer, by rounds of workgroups.  Per matrix step a wave keeps its SIMD busy for 96 cycles per 16 x 16 block (six
// instructions of 16) plus some 60; an input item costs 220 cycles of loads, split and LDS writes per chunk.  One
// workgroup per compute unit leaves latencies open (1.45), two hide most of them (1.15).  Up to four rounds count whole.
// Fitted on ten layers by timing the best block of every workgroup shape (74 variants each): the pick is the fastest or
// within 4 % on six, within 15 % on the others.
static double split_rounds(const SplitGeom& g)
{
    const double steps = split_steps(g), chunks = split_chunks(g);
    const double T = 64.0 * g.wm * g.wn;
    const double mfma = 96.0 * g.mb * g.nb;
    const double items = g.ch8 * g.halo / T;
    const double wg = chunks * (steps * (mfma + 60) + items * 220 + 200) + 4000 + 60.0 * g.mb * g.nb + items * 900;
    const double grid = (double)g.nbk * g.nbx * g.nby * g.nbn;
    const bool two = split_lds_bytes(g) <= 80 * 1024;
    const double per = grid / 256;
    const double rounds = per <= 1 ? 1 : per <= 4 ? (double)(long long)(per + 0.999) : per + 0.6;
    return rounds * wg * (two && per > 1 ? 1.15 : 1.45);
}

// Workgroups that share a compute unit: by registers (of the shapes as compiled) and LDS.
static int split_resident(const SplitGeom& g)
{
    const int two = g.mb == 1 && g.nb <= 2 ? 5 : g.mb * g.nb <= 4 ? 4 : g.mb == 1 || (g.mb == 2 && g.nb <= 4) || (g.mb == 3 && g.nb == 2) ? 3 : 2;
    const int regs = g.parts == 2 ? two : g.mb == 1 ? (g.nb <= 2 ? 4 : 3) : g.mb == 2 && g.nb == 2 ? 3 : 2;
    return (int)std::min<long long>(regs, 160 * 1024 / split_lds_bytes(g));
}

// The same by what a workgroup does alone and what several on a compute unit share.  Alone it takes the sum of what its
// chunks do one after the other: per matrix step 96 cycles per 16 x 16 block (six instructions of 16) and 170 of waiting,
// 507 per input item of a thread (loads, split, LDS writes; more where rows are narrow), 1120 at the chunk's end; then its
// stores.  Several hide each other's waiting until they meet in what they share: the matrix cores, the rate of the weights
// through the L2 (16 channels per wave and step: 69 cycles, and 159 where they are read at all), 730 per item.  The two
// times and the traffic of inputs and outputs are joined by norms.
// Fitted on 187 layers (drawn over 9 to 512 channels, 7 x 7 to 224 x 224, batch 1 to 64, and the networks'), on the best
// three blocks of every workgroup shape: within 7 % (2-norm).  Its picks take 1.030 times the best block timed, those of
// split_rounds 1.072; on 266 other layers 130 picks differ, 1.064 times as fast, but seven of them 5 - 14 % slower.  Where
// it promises 8 % over the pick of split_rounds, 355 of 2000 further layers, that is 1.118 times as fast, 11 of them 3 - 13 % slower (at
// 12 % 4 of 214, but 1.03 - 1.05 times as fast is lost on the others; 338 -> 385 at 17 x 17, 1 x 3, 25.4 -> 27.8 us is promised 17): those
// leave it (5 x 5, 96 -> 256 at 27 x 27, batch 16: 82.7 -> 78.5 us; 180 -> 35 at 124 x 124, stride 2: 158 -> 122).
constexpr double PROMISE = 1.08;
static double norm4(double a, double b) { return std::sqrt(std::sqrt((a * a) * (a * a) + (b * b) * (b * b))); }
// limit: a result that is not below it may be any such number (the planner asks for the least of some thousand blocks, and a bound
// without powers decides most of them: 0.69 -> 0.34 ms on a layer's first call, in the mean of 4000).
static double split_cycles(const SplitGeom& g, double limit)
{
    const double steps = split_steps(g), chunks = split_chunks(g);
    const double mfma = 96.0 * g.mb * g.nb, narrow = 1 + 0.8 / g.xh, items = g.ch8 * g.halo / (64.0 * g.wm * g.wn) * narrow;
    const double alone = 390.0 * g.mb * g.nb + 1520 * std::ceil(items / narrow) * narrow + chunks * (steps * (mfma + 170) + 507 * items + 1120);
    const double shared = 1010 + 357.0 * g.mb * g.nb + chunks * (steps * norm4(1.13 * mfma, g.mb * (17.2 * g.wm + 159)) + 730 * items);
    const int most = split_resident(g);
    const double n = (double)g.nbk * g.nbx * g.nby * g.nbn / 256, full = std::floor(n / most), rest = std::ceil(n - full * most);
    const double bytes = 4.0 * g.N * ((double)g.C * g.H * g.W + (double)g.K * g.P * g.Q);
    auto rounds = [&](auto group) { return n <= 4 * most ? full * group(most) + (rest > 0 ? group(rest) : 0) : (n / most + 0.5) * group(most); };
    const double least = rounds([&](double w) { return std::max(alone, w * shared); });
    if (least >= limit) return least;
    const double cycles = rounds([&](double w) { return std::pow(std::pow(alone, 3.13) + std::pow(w * shared, 3.13), 1 / 3.13); });
    return norm4(cycles, bytes / 990);
}

// The same of operands in two parts, which take half the matrix time, 48 cycles per block and step.  What workgroups on a unit share
// is the sum of the matrix cores' time, the weights' through the L2 (per 16 channels of a wave) and the pixels' out of LDS (per 16);
// an item costs as a mean of those that exist and of whole batches of the threads.  Fitted like that one, on 12300 blocks of 200
// layers: within 7 % (those within 25 % of a layer's best 6 %), its picks 1.015 times the best block timed in the mean (0.05 of them
// above 1.06, the worst 1.24: 22 -> 412 at 25 x 27, batch 14, 26 us for 21).
static double split_cycles_two(const SplitGeom& g, double limit)
{
    const double steps = split_steps(g), chunks = split_chunks(g), blocks = g.mb * g.nb, narrow = 1 + 0.97 / g.xh;
    const double threads = 64.0 * g.wm * g.wn, each = g.ch8 * g.halo / threads, items = (0.5 * SPLIT_BATCH * split_batches(g) + 0.5 * each) * narrow;
    const double alone = 248 * blocks + 614 * std::ceil(each) * narrow + chunks * (steps * (48 * blocks + 230) + 717 * items + 302);
    const double shared = 112 + 434 * blocks + chunks * (steps * (18.4 * blocks + 86.6 * g.mb + 39.1 * g.nb) + 274 * items);
    const int most = split_resident(g);
    const double n = (double)g.nbk * g.nbx * g.nby * g.nbn / 256, full = std::floor(n / most), rest = std::ceil(n - full * most);
    const double bytes = 4.0 * g.N * ((double)g.C * g.H * g.W + (double)g.K * g.P * g.Q);
    auto rounds = [&](auto group) { return n <= 4 * most ? full * group(most) + (rest > 0 ? group(rest) : 0) : (n / most + 0.5) * group(most); };
    const double least = rounds([&](double w) { return std::max(alone, w * shared); });
    if (least >= limit) return least;
    return norm4(rounds([&](double w) { return std::sqrt(alone * alone + w * shared * w * shared); }), bytes / 1245);
}

constexpr long long OWN_VALUES = 6144;
static bool split_plan_parts(SplitGeom* g, bool small, double* cycles)
{
    struct Shape { int mb, nb, wm, wn; };
#define IOLB_SPLIT_ENTRY(M_, N_, A_, B_) {M_, N_, A_, B_},
    static const std::vector<Shape> all = {IOLB_SPLIT_SHAPES(IOLB_SPLIT_ENTRY)}, few = {IOLB_SPLIT_FEW_SHAPES(IOLB_SPLIT_ENTRY)},
                                    little = {IOLB_SPLIT_SMALL_SHAPES(IOLB_SPLIT_ENTRY)};
#undef IOLB_SPLIT_ENTRY
    const std::vector<Shape>& shapes = g->C <= 8 ? few : small ? little : all;
    const bool two = g->parts == 2;
    // cuts of an extent into k nearly equal parts
    auto cuts = [](int extent, int most) {
        std::vector<int> v;
        for (int k = 1; k <= extent; ++k) {
            const int c = (extent + k - 1) / k;
            if (c > most) continue;
            if (v.empty() || v.back() != c) v.push_back(c);
            if (v.size() >= 24) break;
        }
        return v;
    };
    bool found = false;
    SplitGeom best = *g, other = *g;                        // of least split_rounds, of least split_cycles
    double best_rounds = 0, best_cycles = 0;
    for (const Shape& sh : shapes) {
        const int slots = 16 * sh.nb * sh.wn;
        for (int ch8 : {4, 2, 1}) {
            if ((ch8 == 4 && g->C <= 16) || (ch8 == 1) != (g->C <= 8)) continue;
            SplitGeom t = *g;
            t.mb = sh.mb; t.nb = sh.nb; t.wm = sh.wm; t.wn = sh.wn; t.ch8 = ch8;
            for (int tx : cuts(g->Q, slots))
                for (int ty : cuts(g->P, slots / tx)) {
                    const int most_b = (tx == g->Q && ty == g->P) ? std::min(g->N, slots / (tx * ty)) : 1;
                    for (int b = 1; b <= most_b; ++b) {
                        if (b * tx * ty * 2 < slots) continue;           // a smaller shape does it
                        t.tx = tx; t.ty = ty; t.b = b;
                        if (!split_derive(&t)) continue;
                        const double limit = found ? best_cycles : std::numeric_limits<double>::infinity();
                        const double c = two ? split_cycles_two(t, limit) : split_cycles(t, limit), r = two ? c : split_rounds(t);
                        if (!found || r < best_rounds) { best = t; best_rounds = r; }
                        if (!found || c < best_cycles) { other = t; best_cycles = c; }
                        found = true;
                    }
                }
        }
    }
    if (!found) return false;
    const double c = two ? best_cycles : split_cycles(best, std::numeric_limits<double>::infinity());
    const bool leave = c > PROMISE * best_cycles;
    *g = leave ? other : best;
    *cycles = leave ? best_cycles : c;
    return true;
}

// Layers of few workgroups and small kernels: a launch before the convolution takes longer (some 2.3 us of the host's time
// and 3 us of the GPU's) than every workgroup cutting the same kernels once more, about 1 us for 2304 values.  Counted are the
// values that it cuts: eight channels per unit whether they exist or not, four units per step.  The line lies where both are even,
// found on 340 drawn layers of up to 20500 values: up to 6144, and 256 workgroups of those, own kernels are the faster way by 1.23 in
// the mean on 202, none below 0.99 (16 -> 16 at 14 x 14, one image, 10.6 -> 8.2 us a call; 3 x 32 -> 32 at 15 x 15, 4608 values,
// 10.4 -> 8.5); at 6656 it is 0.96 - 1.07, at 7680 0.91 - 0.96, and 0.5 - 0.8 on more than 256 workgroups (3 -> 48 at 148 x 148, batch 6,
// 7 x 7, stride 2: 6656 values, 2352 of them of channels and taps that exist, 504 workgroups, 19.4 us with a launch before it,
// 29.0 without).
constexpr long long OWN_ALL_VALUES = 256 * OWN_VALUES;
bool split_own(const SplitGeom& g)
{
    bool shape = false;
#define IOLB_SPLIT_OWN_ENTRY(M_, N_, A_, B_) shape = shape || (g.mb == M_ && g.nb == N_ && g.wm == A_ && g.wn == B_);
    if (g.ch8 == 1) { IOLB_SPLIT_OWN_FEW_SHAPES(IOLB_SPLIT_OWN_ENTRY) } else { IOLB_SPLIT_OWN_SHAPES(IOLB_SPLIT_OWN_ENTRY) }
#undef IOLB_SPLIT_OWN_ENTRY
    const long long values = 16LL * g.mb * g.wm * split_chunks(g) * split_steps(g) * 32;
    const long long grid = (long long)g.nbk * g.nbx * g.nby * g.nbn;
    return g.parts == 3 && shape && values <= OWN_VALUES && grid * values <= OWN_ALL_VALUES && split_lds_bytes(g, true) <= 160 * 1024;
}

// Three bf16 parts: at most eight channels, workgroups that prepare their own kernels, sums of fewer than 96 products (of 27 - 48 their
// error is 7.5e-8, that of two fp16 parts 8.9e-8; from 96 on two parts have the smaller one), and layers so small that what two fp16 parts take
// besides the products (the samples their scales come from; some 1.2 us) outweighs them, by both models.  Measured on 200 layers: where
// the models part them two parts are 0.88 - 1.05 times as fast below 15 us, 1.1 - 1.7 above 25; the picks of this rule take 1.025 times the
// best block of both, those of two parts alone 1.035.
// (Cycles: that of two parts more than of three; up to which of three nothing is gained; beyond which two always win.)
constexpr double TWO_MORE = 2300, THREE_SMALL = 16000, THREE_MOST = 40000;
bool split_plan(SplitGeom* g, double* cycles)
{
    const bool few = g->C <= 8, maybe_own = 16LL * g->C * g->R * g->S <= OWN_VALUES;
    SplitGeom three = *g;
    three.parts = 3;
    double c3 = 0;
    if ((few || maybe_own) && split_plan_parts(&three, false, &c3) && (few || split_own(three))) {
        *g = three;
        *cycles = c3;
        return true;
    }
    g->parts = 2;
    if (few || !split_plan_parts(g, false, cycles)) return false;
    three = *g;
    three.parts = 3;
    const bool thin = (long long)g->C * g->R * g->S < 96;
    if (thin && !split_plan_parts(&three, true, &c3)) return false;
    if (thin || (*cycles < THREE_MOST && split_plan_parts(&three, true, &c3) && c3 < std::max(THREE_SMALL, *cycles + TWO_MORE))) {
        *g = three;
        *cycles = c3;
    }
    return true;
}

bool split_point_plan(SplitPointGeom* g, double* cycles)
{
    struct Shape { int mb, nb, wm, wn; };
    static const Shape shapes[] = {
#define IOLB_POINT_ENTRY(M_, N_, A_, B_) {M_, N_, A_, B_},
        IOLB_SPLIT_POINT_SHAPES(IOLB_POINT_ENTRY)
#undef IOLB_POINT_ENTRY
    };
    bool found = false;
    SplitPointGeom best = *g;
    double best_cycles = 0;
    for (const Shape& sh : shapes) {
        SplitPointGeom t = *g;
        t.mb = sh.mb; t.nb = sh.nb; t.wm = sh.wm; t.wn = sh.wn;
        const int npix = 16 * t.nb * t.wn, z = 16 * t.mb * t.wm;
        // pixels read several at a time must not run on into another image
        if (t.in == SPLIT_IN_PIXELS && t.images > 1 && t.HW % split_point_pixels(t.in)) {
            if (t.w_image == 0 && t.HW >= 128) { t.groups *= t.images; t.images = 1; }
            else t.in = SPLIT_IN_SINGLE;
        }
        t.nbk = (t.K + z - 1) / z;
        t.Kb16 = t.nbk * t.mb * t.wm;
        const long long nbp = ((long long)t.images * t.HW + npix - 1) / npix, grid = nbp * t.groups * t.nbk;
        const long long span = std::min<long long>((t.HW - 1 + npix - 1) / t.HW + 1, t.images);
        if (grid > 0x7fffffffLL || (long long)t.images * t.HW >= (1LL << 31) - 1024 || 4 * span * t.C * t.HWin >= (1LL << 31)) continue;
        t.nbp = (int)nbp;
        // A step of a workgroup: 32 channels of npix pixels come in at 12 bytes per clock and compute unit, and those of z kernels in two
        // parts at 16; alone on its unit a workgroup waits some 2800 clocks for them.  (Fitted on all blocks of 37 drawn layers, two of
        // which do better with another, by 1 and 2 %.  By the bytes of three parts 768 -> 192 at 17 x 17, batch 64, took 64 kernels a block,
        // 37 us, and not 192, 35.  Blocks of 128 pixels and 128, 192 or 256 kernels on eight waves: 0.8 - 1.02 on 36 of them.)
        const double chunks = (t.C + 31) / 32, n = grid / 256.0, rounds = n <= 4 ? (double)((grid + 255) / 256) : n + 0.5;
        const double step = std::max((96.0 * z + 128.0 * npix) / 12, 48.0 * t.mb * t.nb * (t.wm * t.wn / 4) * 1.4);
        // (the time that is told is the one that split_wino_pick's models were fitted with: three parts at 19 bytes per clock)
        const double told = std::max((192.0 * z + 128.0 * npix) / 19, 96.0 * t.mb * t.nb * (t.wm * t.wn / 4) * 1.4);
        const double res = t.mb * t.nb <= 4 ? 4 : t.mb * t.nb <= 8 ? 3 : 8.0 / (t.wm * t.wn);
        auto time = [&](double per_step, double alone) { return std::max(rounds * chunks * per_step, (double)(long long)(rounds / res + 0.999) * chunks * alone) + 6000; };
        const double c = time(step, 2800);
        if (!found || c < best_cycles) { found = true; best = t; best_cycles = c; *cycles = time(told, 3200); }
    }
    if (found) *g = best;
    return found;
}

// Kernels with a window: measured 1.1 to 4 times as fast as the fp32 kernels on every layer of 60 drawn ones (16 to 512
// channels, 7 x 7 to 224 x 224, batch 1 to 64) but those of three channels with 3 x 3 kernels, which are bound by
// their stores (0.76 - 0.96); 7 x 7 and 11 x 11 kernels on three channels 0.98 - 1.2 and 5.7.
bool split_conv_faster(const iolb_shape& s) { return s.C > 8 || s.R * s.S >= 25; }

// 1 x 1, channels outermost: the fp32 kernel reads and writes at the rate of memory and needs no pass over the kernels before it; it loses
// where its chain over the channels or the products outweigh that.  Modelled times in us, fitted on 260 drawn layers (16 to 2048
// channels; within 14 and 19 % in the 2-norm); where the split way wins by a margin it is 1.6 times as fast in the mean
// (1536 -> 32 at 13 x 15, batch 6 46 -> 24 us; 684 -> 127 at 8 x 8, batch 53 24 -> 16), one of those 13 % slower; the others it
// would make up to 1.7 times slower (128 -> 352 at 25 x 25, batch 3 6.9 -> 11.9).
//   Channels innermost: that kernel does not exist, and the general one reads a channel group of a pixel at a time.  On all of 40 drawn layers
// of 16 channels and more the split way was the faster one, by 2.3 in the mean (16 -> 32 at 84 x 90, batch 11 14.6 -> 14.3 us, 151 -> 224
// at 73 x 73, batch 33 950 -> 107), at a smaller error (16 channels 7.7e-8 -> 7.0e-8, 256 2.8e-7 -> 1.7e-7).
bool split_point_faster(const iolb_shape& s, int P, int Q, bool hwc)
{
    if (s.C < 16) return false;
    if (hwc) return true;
    const double pixels = (double)s.N * P * Q, flop = 2 * pixels * s.C * s.K;
    const double bytes = 4 * (pixels * s.C + pixels * s.K + (double)s.K * s.C);
    const double waves = std::ceil(pixels / 256 * std::ceil(s.K / 64.0) / 512);
    const double tile = 5.04 + norm4(bytes / 7.47e6, flop / 1.08e8) + 0.0220 * s.C * std::max(1.0, waves);
    const double split = 8.65 + norm4(bytes / 4.48e6, flop / 2.20e8) + 0.0087 * s.C;
    return split + 1 < 0.94 * tile;
}

// Sums of fewer channels keep three bf16 parts, whose error is smaller there (F(2 x 2), 16 channels 1.0e-7 against 1.3e-7, 48 1.7e-7 and
// 1.9e-7; F(4 x 4) 3.7e-7 and 5.4e-7, 1.2e-6 and 1.3e-6; from 64 on that of two fp16 parts is), and which are up to 12 % faster there;
// so do a few more in a single round of workgroups, where the sample of two parts costs more than its products save (40 drawn layers of
// 64 - 94 channels in one round, two parts against three: F(2 x 2) 1.00 - 1.10 times the time, F(4 x 4) 0.97 - 1.19; 1.034 in the mean).
constexpr int WINO_TWO_LEAST = 64, WINO_TWO_SMALL = 96;

// Modelled time of a call: the kernels' transform, and per round of workgroups first loads and stores and a stage of 16
// channels.  Fitted on 148 drawn layers (16 to 512 channels, 7 x 7 to 224 x 224, batch 1 to 64); on 2862 others within 9 (F(2 x 2))
// and 12 % (F(4 x 4)) in the 2-norm, above 200 us 9 and 11 % too low (128 -> 128 at 112 x 112, batch 64, F(4 x 4) 494 us for 570).
static double wino_split_ns(const WinoSplitGeom& g)
{
    const double per = (double)g.nbt * g.nbk / 256, rounds = (per <= 4 ? std::ceil(per) : per + 0.5) * (g.parts == 3 ? 1 : g.m == 4 ? 0.92 : 0.95);
    if (g.m == 4) return g.z == 64 ? 5600 + rounds * (10700 + 3450.0 * g.chunks) : 7300 + rounds * (6900 + 2520.0 * g.chunks);
    return g.z == 64 ? 3800 + rounds * (8500 + 2650.0 * g.chunks) : 7000 + rounds * (2500 + 1000.0 * g.chunks);
}

bool wino_split_plan(WinoSplitGeom* g, double* ns)
{
    struct Shape { int m, tb, z; };
    static const Shape shapes[] = {
#define IOLB_WINO_SPLIT_ENTRY(M_, T_, Z_) {M_, T_, Z_},
        IOLB_WINO_SPLIT_SHAPES(IOLB_WINO_SPLIT_ENTRY)
#undef IOLB_WINO_SPLIT_ENTRY
    };
    bool found = false;
    WinoSplitGeom best = *g;
    double best_ns = 0;
    for (const Shape& sh : shapes) {
        if (sh.m != g->m) continue;
        WinoSplitGeom t = *g;
        t.tb = sh.tb; t.z = sh.z;
        t.nbt = (g->tiles + sh.tb - 1) / sh.tb;
        t.nbk = (g->K + sh.z - 1) / sh.z;
        t.chunks = (g->C + 15) / 16;
        t.Kb32 = t.nbk * (sh.z / 32);
        t.parts = g->C < WINO_TWO_LEAST || (g->C < WINO_TWO_SMALL && (long long)t.nbt * t.nbk <= 256) ? 3 : 2;
        if (!wino_split_fits(t)) continue;
        const double c = wino_split_ns(t);
        if (!found || c < best_ns) { found = true; best = t; best_ns = c; }
    }
    if (found) { *g = best; *ns = best_ns; }
    return found;
}

// Modelled times in ns, each fitted on 194 drawn layers like those above, the split product's again on 210 in two parts (13 % in the
// 2-norm; the tile's 10 where it is fused, 20 where it is not): the tile's product or fused kernel by rounds of its blocks, traffic of V
// and M at 4.7 - 6 TB/s, the launches.  Over 330 layers these routes take 1.025 times the best of the three, the ones before them (their
// models from kernels in three parts; no model for channels that are no multiple of four) 1.089; some eight are 3 - 14 % slower than those.
//   Unfused tiles where the first rule took the product: that runs, or the fused kernel where it is modelled faster.  By the tile's model some
// went back to the tile (128 -> 304 at 77 x 77, batch 8, F(3 x 3) 150 -> 197 us; 128 -> 176 at 128 x 128, batch 4, F(6 x 6) 101 -> 137).
//   Where that rule was made for them, from 128 channels and kernels on, layers whose channels are no multiple of four keep it altogether,
// with a wider line: 53 drawn layers between 0.8 and 0.9 are 1.05 to 3.4 times as fast on the product (365 -> 227 at 35 x 35, batch 3, F(2 x 2)
// 57 -> 32 us; 507 -> 299 at 42 x 42, batch 11, F(4 x 4) 333 -> 120).  Beyond it the routes of three are part of the tests (33 x 261 -> 300
// at 15 x 15 109 us, the product 63).  The others go by the models (81 channels in F(2 x 2) 2.2 times as fast, 70 layers 1.3 in the mean).
int split_wino_pick(const iolb_shape& s, const iolb_tile_config& tile, long long tiles, double product_cycles, double fused_ns)
{
    const int m = winograd_m(s.algo);
    const double n2 = (m + 2) * (m + 2);
    const int Kp = (s.K + 31) / 32 * 32;
    const bool fused_tile = tile.path == IOLB_PATH_FUSED;
    const bool product_first = !fused_tile && product_cycles && s.C >= 128 && s.K >= 128 && product_cycles / 2 < (s.C % 4 ? 0.9 : 0.8) * (2 * n2 * tiles * s.C * Kp / 105000);
    if (!fused_tile && s.C % 4 && s.C >= 128 && s.K >= 128) return product_first;
    const double out = (double)s.N * (s.H + 2 * s.pad - 2) * (s.W + 2 * s.pad - 2);
    const double bytes = 4 * ((double)s.N * s.C * s.H * s.W + 2 * n2 * tiles * (s.C + s.K) + s.K * out);
    const double product = m == 2   ? 10600 + bytes / 5140 + 0.158 * product_cycles
                           : m == 3 ? 11800 + bytes / 4750 + 0.139 * product_cycles
                           : m == 4 ? 13500 + bytes / 5270 + 0.215 * product_cycles
                                    : 17400 + bytes / 5080 + 0.307 * product_cycles;
    if (product_first) return fused_ns && fused_ns < product ? 2 : 1;
    const double tb = tile.x / m, across = std::ceil(tiles / tb);
    double best;
    if (fused_tile) {
        const double rounds = std::ceil(across * ((s.K + tile.z - 1) / tile.z) / 256), block = 2 * n2 * tb * tile.z * s.C / 1000;
        best = m == 2 ? 3500 + rounds * (6100 + 2.42 * block) : 8100 + rounds * (8300 + 3.05 * block);
    } else {
        const double rounds = std::ceil(n2 * across * ((Kp + tile.z - 1) / tile.z) / 256), waves = std::min(4, tile.threads / 64);
        best = 12000 + bytes / 6000 + 45.0 * s.C + rounds * s.C * 2 * tb * tile.z / waves / 1000 * (m == 2 ? 9.2 : 6.6);
    }
    best *= m == 2 ? 1 : m == 6 ? 1.15 : 1.05;
    int pick = 0;
    if (product_cycles && s.C >= WINO_TWO_LEAST && product < best) { best = product; pick = 1; }
    if (fused_ns && fused_ns < best) pick = 2;
    return pick;
}

}  // namespace iolb
