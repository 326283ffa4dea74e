// Conv2d per-sample gradients on bf16 matrix units (conv2d_split.hip): fp32
// inputs as three bf16 parts, bf16 inputs as they are.
#pragma once

#include "common.hpp"
#include "conv2d_rows.hpp"

namespace dpg {

// The kernel's time in us, 0 where it does not take the shape or has measured
// slower whatever the grid (the caller compares it with the kernel it would replace).
// slots: squared-norm partials per sample that the call's workspace holds
// (1: no workspace, one tile per sample).
double conv_split_us(const ConvRowsArgs &a, bool bf16, int slots);
void conv_split_launch(const ConvRowsArgs &a, bool bf16, int slots, float scale, float *gW, float *gb, float *sqnorm,
                       float *partial, hipStream_t stream);

}  // namespace dpg
