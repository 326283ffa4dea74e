// Row-chunked Conv2d per-sample gradients (conv2d_rows.hip), for samples
// whose input planes do not fit one workgroup's LDS.
#pragma once

#include "common.hpp"

namespace dpg {

struct ConvRowsArgs {
    const void *X, *GY;
    i64 N, Cin, H, W, Cout, Ho, Wo, kh, kw, sh, sw, ph, pw;
};

// a chunk of at least one output row fits the LDS budget
bool conv_rows_ok(const ConvRowsArgs &a);
// ... and the automatic choice prefers it to the tiled kernel: tiles of at
// least four 32-column blocks (with fewer, most of the four waves' position
// work feeds no MFMA; measured on the CIFAR network's first layer)
bool conv_rows_preferred(const ConvRowsArgs &a);
// A grid's rounds over 256 CUs that hold `resident` workgroups each.  A last
// round that gives a CU one workgroup only takes `lone` of a full one.
inline double cu_rounds(double grid, int resident, double lone)
{
    const double full = 256.0 * resident, whole = (double)(i64)(grid / full), left = grid - whole * full;
    if (left == 0) return whole;
    return whole + (left <= 256 ? lone : left <= 256.0 * (resident - 1) ? 0.5 * (lone + 1) : 1.0);
}
// the kernel's time in us on aligned operands, within 12% rms (fitted with
// split_us of conv2d_split_plan.hpp); 0 where it does not take the shape
double conv_rows_us(const ConvRowsArgs &a);
// gradient tiles per sample (norm partials in the workspace when above one)
int conv_rows_tiles(const ConvRowsArgs &a);
// writes gW, gb (if not null) and sqnorm (if not null; partial: N * tiles
// floats of workspace when there are several tiles)
void conv_rows_launch(const ConvRowsArgs &a, bool bf16, float scale, float *gW, float *gb, float *sqnorm,
                      float *partial, hipStream_t stream);

}  // namespace dpg
