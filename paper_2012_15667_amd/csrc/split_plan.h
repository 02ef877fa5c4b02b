// Which layers run on the 16-bit matrix cores with operands in parts, and on which workgroup shape.
#ifndef IOLB_SPLIT_PLAN_H
#define IOLB_SPLIT_PLAN_H

#include "kernels.h"

namespace iolb {

// Fills the derived fields of g (extents, pitches, block counts) from the layer, the block (b, tx, ty) and the
// workgroup shape (mb, nb, wm, wn, ch8).  False when the kernel cannot run it.
bool split_derive(SplitGeom* g);
// The block and workgroup shape of least modelled time for the layer in g; *cycles gets that time (clock cycles of
// the chip at full occupation).  False when no shape runs the layer.
bool split_plan(SplitGeom* g, double* cycles);
// Whether the workgroups of a planned layer prepare their own kernels (no launch before the convolution).
bool split_own(const SplitGeom& g);
// The same for 1 x 1 layers: groups, images, C, K, Ky, HW, HWy, HWin, Win, Q, stride, hwc and in describe the layer.
bool split_point_plan(SplitPointGeom* g, double* cycles);
// The block of the fused Winograd kernel for the layer in g (N, C, H, W, K, m, pad, P, Q, th, tw, tiles); *ns gets the
// modelled time of the call.  False when the kernel cannot run it.
bool wino_split_plan(WinoSplitGeom* g, double* ns);

// Whether a layer without a caller-supplied tile leaves the fp32 kernels (the reasons are in the definitions).
bool split_conv_faster(const iolb_shape& s);
bool split_point_faster(const iolb_shape& s, int P, int Q, bool hwc);
// 0: the tile, 1: the split product between transforms of their own, 2: the fused split kernel.  (A time of 0: does not run.)
int split_wino_pick(const iolb_shape& s, const iolb_tile_config& tile, long long tiles, double product_cycles, double fused_ns);

}  // namespace iolb

#endif
