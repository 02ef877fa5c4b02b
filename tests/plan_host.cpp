// The library's host code on its own, for tests: what the planners choose and what the kernels are launched with.
#include "split_plan.h"

using namespace iolb;

extern "C" void divide(const int* n, int count, unsigned d, int* quotients)
{
    const Divisor by(d);
    for (int i = 0; i < count; ++i) quotients[i] = by.of(n[i]);
}

// Whether every n up to `most` is divided rightly; the ends and some 20000 multiples where there are too many.
static bool exact(const Divisor& by, long long most, long long d)
{
    const long long step = most / d / 20000 + 1;
    for (long long k = 0; k * d <= most; k += step)
        for (long long n : {k * d - 1, k * d, k * d + 1, most - k})
            if (n >= 0 && n <= most && by.of((int)n) != n / d) return false;
    return true;
}

// The fused Winograd kernel's block for a layer: {tb, z, chunks, grid, images of a block, channels}, false: does not run.
extern "C" int plan_wino_split(int N, int C, int H, int W, int K, int m, int pad, WinoSplitGeom* g)
{
    *g = WinoSplitGeom{};
    g->N = N; g->C = C; g->H = H; g->W = W; g->K = K; g->m = m; g->pad = pad; g->P = H + 2 * pad - 2; g->Q = W + 2 * pad - 2;
    g->th = (g->P + m - 1) / m; g->tw = (g->Q + m - 1) / m; g->tiles = N * g->th * g->tw;
    double ns = 0;
    return wino_split_plan(g, &ns);
}

// Of the input loads of such a layer: the greatest scalar offset less the buffer's range of one image.
extern "C" long long wino_split_beyond_range(int N, int C, int H, int W, int K, int m, int pad)
{
    WinoSplitGeom g;
    if (!plan_wino_split(N, C, H, W, K, m, pad, &g)) return -1;
    const bool single = wino_split_cols(g) == WINO_COLS_SINGLE;
    long long most = 0;
    for (int c0 = 0; c0 < 16 * (g.chunks + 2); c0 += 4)                   // (stages are loaded up to two ahead)
        for (int r = 0; r < m + 2; ++r) {
            const int at = single ? wino_split_offset<WINO_COLS_SINGLE>(g, c0, r) : wino_split_offset<WINO_COLS_WHOLE>(g, c0, r);
            if (at > most) most = at;
        }
    return most - (long long)wino_split_range(g, 1);
}

// The direct kernel's block for a layer (H x W padded by pad on both axes), and its workgroups.
extern "C" int plan_split(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, SplitGeom* g)
{
    *g = SplitGeom{};
    g->N = N; g->C = C; g->H = H; g->W = W; g->K = K; g->R = R; g->S = S; g->stride = stride; g->pad = g->pad_w = pad;
    g->P = (H + 2 * pad - R) / stride + 1; g->Q = (W + 2 * pad - S) / stride + 1;
    double cycles = 0;
    return split_plan(g, &cycles);
}
// {parts of an operand, images of a block, channel blocks of a wave, its pixel blocks, chunks, waves beside each other in kernels and pixels}
extern "C" int split_block(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int* block)
{
    SplitGeom g;
    if (!plan_split(N, C, H, W, K, R, S, stride, pad, &g)) return 0;
    const int of[7] = {g.parts, g.b, g.mb, g.nb, (int)split_chunks(g), g.wm, g.wn};
    for (int i = 0; i < 7; ++i) block[i] = of[i];
    return 1;
}
// {workgroups, whether they prepare their own kernels, whether ids are divided by multiplication, whether all divisions are exact}
extern "C" int split_facts(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int* facts)
{
    SplitGeom g;
    SplitDivisors dv;
    SplitOwn own;
    if (!plan_split(N, C, H, W, K, R, S, stride, pad, &g) || !split_divisors(g, false, &dv, &own)) return 0;
    const long long items = g.ch8 * g.halo - 1LL, units = 4LL * split_steps(g) - 1, slots = 16LL * g.nb * g.wn - 1, ids = (long long)g.nbk * g.nbx * g.nby * g.nbn - 1;
    bool good = exact(dv.halo, items, g.halo) && exact(dv.per, g.halo - 1, g.yh * g.rowp) && exact(dv.rowp, g.yh * g.rowp - 1, g.rowp) &&
                exact(dv.esx, g.rowp - 1, g.esx) && exact(dv.ch8, units, g.ch8) && exact(dv.S, units, g.S) && exact(dv.txy, slots, g.tx * g.ty) && exact(dv.tx, slots, g.tx);
    if (dv.small) good = good && exact(dv.pixel_blocks, ids, g.nbx * g.nby * g.nbn) && exact(dv.nbk, ids, g.nbk) && exact(dv.nbx, ids, g.nbx) && exact(dv.nby, ids, g.nby);
    const bool o = split_own(g);
    if (o)
        good = good && exact(own.row, 16LL * g.mb * g.wm * g.C * g.R * g.S - 1, g.C * g.R * g.S) && exact(own.steps, (long long)split_chunks(g) * split_steps(g) - 1, split_steps(g));
    facts[0] = (int)ids + 1; facts[1] = o; facts[2] = dv.small; facts[3] = good;
    return 1;
}
// The same of the fused Winograd kernel: {workgroups, whether divided by multiplication, whether exact}
extern "C" int wino_split_facts(int N, int C, int H, int W, int K, int m, int pad, int* facts)
{
    WinoSplitGeom g;
    if (!plan_wino_split(N, C, H, W, K, m, pad, &g)) return 0;
    const WinoSplitDivisors dv = wino_split_divisors(g);
    const int per = g.th * g.tw;
    facts[0] = g.nbt * g.nbk; facts[1] = dv.small;
    facts[2] = !dv.small || (exact(dv.nbt, facts[0] - 1LL, g.nbt) && exact(dv.per_image, g.nbt * (long long)g.tb - 1, per) && exact(dv.tw, per - 1, g.tw));
    return 1;
}
