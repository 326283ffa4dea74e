// Per-sample gradients of Linear layers over a sequence (ps_split.hip): fp32
// layers of any shape, and the bf16 layers that the staged kernel does not take.
#pragma once

#include "common.hpp"

namespace dpg {

struct PsLayer {
    const void *A, *B;
    i64 T, din, dout;
    float scale;
    float *gW, *gb, *sqnorm;
    float *partial;   // N * ps_split_parts(din, dout) floats of scratch (unused when sqnorm is NULL)
};

// A and B rows of at least 16 bytes (a load that would pass a row's end is
// moved back inside it), features below 2^22 (32-bit offsets in a stage) and
// positions that 32 bits count.
bool ps_split_ok(dp_dtype dt, i64 T, i64 din, i64 dout);
// squared-norm partials per sample
int ps_split_parts(i64 din, i64 dout);
// one layer: the gradients and the squared norms
void ps_split_grad(const PsLayer &layer, dp_dtype dt, i64 N, hipStream_t stream);

// whether dp_grad_sample_many runs an fp32 layer in the grouped launch (T a
// multiple of 16, d_in and d_out multiples of 4, 16-byte aligned A, B, gW, and
// small enough that 16 of them fit one launch's grid)
bool fp32_staged_ok(const void *A, const void *B, const void *gW, i64 N, i64 T, i64 din, i64 dout);

// up to kPsGroupMax fp32 layers that share N, in one launch plus one that
// adds their squared-norm partials; bit for bit the single-layer results
constexpr int kPsGroupMax = 16;
void ps_split_group(const PsLayer *layers, int count, i64 N, hipStream_t stream);

}  // namespace dpg
