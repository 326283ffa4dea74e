// Conv2d per-sample gradients on v_mfma_f32_32x32x16_bf16 for layers with
// enough input channels to fill an MFMA block:
//   gW_n[co][ci][u][v] = s * sum_{oh,ow} GY_n[co][oh][ow] * X_n[ci][oh*sh+u-ph][ow*sw+v-pw]
// fp32 inputs are split into three bf16 parts (split_bf16.hpp: six products,
// fp32 sums), bf16 inputs are used as they are.
//
// For one tap (u, v) this is a GEMM of GY (channels x positions) and X
// (positions x channels).  MFMA rows are 32 input channels, columns 32 output
// channels, and the contraction runs over (output row, input column): K is
// cut into units of eight consecutive columns of one row, which is what a
// lane supplies to one MFMA.  With columns counted on the input side, X needs
// no shift along a row: tap column v pairs X[c] with GY[c - s], s = (v - pw)
// / sw, and X's columns of one phase c % sw are kept together.  So per unit a
// lane reads its X operand once per tap row u and its GY operand once, and
// makes the operand of a neighbouring shift, s - 1 or s + 1, from registers
// (one more word and an alignbit per word).
//
// A workgroup owns a tile of WI x WO such 32 x 32 channel blocks (WK waves
// share a block's units) for up to three tap rows and three tap columns of
// one phase (a group).  Two waves share a block's nine taps, so that each tap
// has two accumulators, for the large and the small products, in registers:
// one takes the center column and two taps of the column vc + sw, the other
// the column vc - sw and the third.  The workgroup walks the sample's output
// rows in chunks of RC.
//
// What bounds it: at 512 samples, 64 -> 128 channels @16^2 (252 MB, six times
// 19.3 GFLOP of bf16 MFMA, 62 us of it at the clock it runs at) a workgroup of
// 44 us spends 2 on its start, 31 on its chunks (staging and multiplying by
// turns, against the CU's other workgroup), 8 on its stores, which all
// workgroups of a round issue at about the same time.  160 us against 223 on
// fp32 MFMA (0.8e-7 against 1.9e-7 off 64 bits); 32 -> 64 @32^2 130 against
// 192.  Tried: nine taps per wave with one accumulator each (faster staging
// rounds, but 2.2e-7 off), six waves of one tap column (only one such
// workgroup fits a CU), 16-byte instead of 4-byte stores of the outputs,
// workgroups of a CU started apart or at different wave priorities (no change).
//
// LDS holds, per part, [ci][row][unit] of X and [co][row][guard, units] of GY
// (the zero guards are the neighbours past a row's ends), with channel
// strides of an odd number of 16-byte units, so that the 16 channels of a
// read's pass fall in different banks.
#include "common.hpp"
#include "split_bf16.hpp"
#include "conv2d_split.hpp"

namespace dpg {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
using split::finite_f32;

constexpr int kThreads = 256, kWaves = 4;
constexpr int kT = 3;                  // tap rows and columns per group, at most
constexpr int kBatch = 2;              // units per thread loaded at once
constexpr int kMaxGroups = 64;
constexpr size_t kLds = 76 * 1024;     // two workgroups per CU

struct ConvGroup {
    int8_t u0, ul;                     // tap rows u0 .. u0 + ul - 1
    int8_t vc, vl;                     // center tap column, 1: it, 2: and vc + sw, 3: and vc - sw
    int16_t sc, phase;                 // vc - pw = sw * sc + phase, 0 <= phase < sw
};

struct SplitShape {
    int Cin, H, W, Cout, Ho, Wo, kh, kw, sh, sw, ph, pw;
    int L, khw;
    int NU, inv_nu;                    // units per row, ceil(65536 / NU)
    int gl, inv_gl, gp;                // GY units loaded per row, ceil(65536 / gl), row pitch: NU and NU + 1 (a zero
                                       // guard before each row) where a row's neighbours past its ends are zero
                                       // for every group, else both NU + 2 (they are loaded)
    int RC, XR;                        // output rows per chunk, input rows they read
    int csx, csg;                      // channel strides in LDS (bytes)
    int px, pg;                        // plane strides (bytes)
    int nx, ng;                        // units per chunk of X and GY
    int inv_xrow, inv_grow;            // ceil(2^20 / (XR * NU)), ceil(2^20 / (RC * gl))
    int nci, nco, ngrp, gpw, tiles;    // channel tiles, groups, groups per workgroup, workgroups per sample
    int bias_at;                       // byte offset of the bias sums (one float per GY unit of a chunk), 0: none
    int full;                          // kh == kw == 3 in one group with stores by rows
    ConvGroup g[kMaxGroups];
};

// floor(i / d) from ceil(2^20 / d), exact while i * d < 2^20
__device__ __forceinline__ int div20(int i, int inv) { return (int)(((uint32_t)i * (uint32_t)inv) >> 20); }

template <typename T>
struct Unit {
    T v[8];
};

template <typename T>
__device__ __forceinline__ float as_f32(T v);
template <>
__device__ __forceinline__ float as_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float as_f32<uint16_t>(uint16_t v) { return bf16_to_f32(v); }

// Eight elements of a sample of `total` elements, at element offsets e + k *
// step; a dead unit is zeros.  fp32 elements in a row are two 16-byte loads;
// at the sample's ends these start inside it, and mend_unit then moves the
// elements to their places.  Single elements past the sample read zero.
template <typename T>
__device__ __forceinline__ void load_unit(__amdgpu_buffer_rsrc_t rs, int e, int step, int total, bool dead, Unit<T> &u)
{
    if constexpr (sizeof(T) == 4) {
        if (step == 1) {
            const int st = e < 0 ? 0 : e > total - 8 ? total - 8 : e;
            const uint32_t o = dead ? kOutside : (uint32_t)st * 4u;
            const u32x4_t a = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0));
            const u32x4_t b = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, o + 16, 0, 0));
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                u.v[k] = __uint_as_float(a[k]);
                u.v[4 + k] = __uint_as_float(b[k]);
            }
            return;
        }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t o = dead ? kOutside : (uint32_t)(e + k * step) * (uint32_t)sizeof(T);
        if constexpr (sizeof(T) == 4) u.v[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, 0));
        else u.v[k] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, o, 0, 0);
    }
}

// The same unit once loaded.  clip: elements k with c + k * step outside [0, n) become zero.
template <typename T>
__device__ __forceinline__ void mend_unit(int e, int step, int total, bool clip, int c, int n, Unit<T> &u)
{
    if constexpr (sizeof(T) == 4) {
        const int d = e < 0 ? e : e > total - 8 ? e - (total - 8) : 0;
        if (step == 1 && d != 0) {
            const Unit<T> w = u;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                u.v[k] = T(0);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (j == k + d) u.v[k] = w.v[j];
            }
        }
    }
    if (clip) {
#pragma unroll
        for (int k = 0; k < 8; ++k) u.v[k] = (uint32_t)(c + k * step) < (uint32_t)n ? u.v[k] : T(0);
    }
}

template <typename T, int NP>
__device__ __forceinline__ void store_unit(char *p, int plane, const Unit<T> &u)
{
    if constexpr (NP == 3) {
        uint32_t q[3][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) split::split2(u.v[2 * k], u.v[2 * k + 1], q[0][k], q[1][k], q[2][k]);
#pragma unroll
        for (int a = 0; a < 3; ++a)
            *reinterpret_cast<uint4 *>(p + a * plane) = make_uint4(q[a][0], q[a][1], q[a][2], q[a][3]);
    } else {
        uint4 w;
        w.x = u.v[0] | (uint32_t)u.v[1] << 16;
        w.y = u.v[2] | (uint32_t)u.v[3] << 16;
        w.z = u.v[4] | (uint32_t)u.v[5] << 16;
        w.w = u.v[6] | (uint32_t)u.v[7] << 16;
        *reinterpret_cast<uint4 *>(p) = w;
    }
}

// A value the compiler cannot see through: index arithmetic that starts from
// it stays where it is written, instead of being hoisted out of the loops into
// registers that the accumulators need.
__device__ __forceinline__ int here(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// FULL: three tap rows and columns in every group
template <typename T, int WI, int WO, int WK, bool FULL>
__global__ __launch_bounds__(kThreads, 2) void conv_split_kernel(const T *__restrict__ X, const T *__restrict__ GY,
                                                                 const SplitShape s, float scale,
                                                                 float *__restrict__ gW, float *__restrict__ gb,
                                                                 float *__restrict__ sqout)
{
    static_assert(2 * WI * WO * WK == kWaves, "two waves per block and part of its units");
    constexpr int NP = sizeof(T) == 4 ? 3 : 1;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    __shared__ float red[kWaves];
    const uint32_t b = xcd_swizzle32(blockIdx.x, gridDim.x);
    const uint32_t n = b / (uint32_t)s.tiles;
    uint32_t tile = b - n * (uint32_t)s.tiles;
    const uint32_t per = (uint32_t)(s.nco * s.nci);
    const int gpart = (int)(tile / per);
    tile -= gpart * per;
    const int cot = (int)(tile / (uint32_t)s.nci), cit = (int)(tile - (uint32_t)cot * s.nci);
    const int ci0 = cit * 32 * WI, co0 = cot * 32 * WO;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, kg = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave & 1, blk = wave / 2 % (WI * WO), wi = blk % WI, wo = blk / WI, wk = wave / (2 * WI * WO);
    const T *Xn = X + (i64)n * s.Cin * s.H * s.W;
    const T *Gn = GY + (i64)n * s.Cout * s.L;
    const __amdgpu_buffer_rsrc_t rx = sample_rsrc(Xn, (uint32_t)(s.Cin * s.H * s.W) * (uint32_t)sizeof(T));
    const __amdgpu_buffer_rsrc_t rg = sample_rsrc(Gn, (uint32_t)(s.Cout * s.L) * (uint32_t)sizeof(T));
    char *const LX = smem, *const LG = smem + NP * s.px;

    // guards, and units past a chunk's end, are zero
    for (int i = tid; i < (NP * (s.px + s.pg)) / 16; i += kThreads)
        *reinterpret_cast<uint4 *>(smem + 16 * i) = make_uint4(0u, 0u, 0u, 0u);

    float sq = 0.0f;
    for (int gi = gpart * s.gpw; gi < (gpart + 1) * s.gpw && gi < s.ngrp; ++gi) {
        const int u0 = s.g[gi].u0, ul = s.g[gi].ul, vc = s.g[gi].vc, vl = s.g[gi].vl;
        const int sc = s.g[gi].sc, phase = s.g[gi].phase;

        const bool clip_x = (s.W % (8 * s.sw)) != 0, clip_g = sc != 0 || s.NU * 8 != s.Wo;
        // One chunk into LDS: X unit i = (ci, row, unit), GY unit i = (co, row,
        // unit), kBatch of them per thread in flight.  Nothing of it stays in
        // registers while the chunk is multiplied (the accumulators leave room
        // for the operands only); the CU's other workgroup multiplies meanwhile.
        // the first input channel tile also adds GY's units up, each thread its own
        const bool bias_here = gb && s.bias_at && cit == 0 && gi == 0;
        float *const bias_sums = reinterpret_cast<float *>(smem + s.bias_at);
        auto stage_x = [&](int oh0) {
            const int t = here(tid);
            for (int base = 0; base < s.nx; base += kBatch * kThreads) {
                Unit<T> u[kBatch];
                int at[kBatch], col[kBatch], e[kBatch];
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    const int i = base + t + kThreads * q, c = div20(i, s.inv_xrow), w = i - c * (s.XR * s.NU);
                    const int r = (w * s.inv_nu) >> 16, cu = w - r * s.NU, ih = oh0 * s.sh + r + u0 - s.ph;
                    at[q] = i < s.nx ? c * s.csx + w * 16 : -1;
                    col[q] = 8 * cu * s.sw + phase;
                    e[q] = ((ci0 + c) * s.H + ih) * s.W + col[q];
                    load_unit<T>(rx, e[q], s.sw, s.Cin * s.H * s.W,
                                 (uint32_t)ih >= (uint32_t)s.H || ci0 + c >= s.Cin || i >= s.nx, u[q]);
                }
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    mend_unit<T>(e[q], s.sw, s.Cin * s.H * s.W, clip_x, col[q], s.W, u[q]);
                    if (at[q] >= 0) store_unit<T, NP>(LX + at[q], s.px, u[q]);
                }
            }
        };
        auto stage_g = [&](int oh0) {
            const int t = here(tid);
            for (int base = 0; base < s.ng; base += kBatch * kThreads) {
                Unit<T> u[kBatch];
                int at[kBatch], col[kBatch], e[kBatch];
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    const int i = base + t + kThreads * q, c = div20(i, s.inv_grow), w = i - c * (s.RC * s.gl);
                    const int r = (w * s.inv_gl) >> 16, cu = w - r * s.gl, oh = oh0 + r;
                    at[q] = i < s.ng ? c * s.csg + (r * s.gp + cu + s.gp - s.gl) * 16 : -1;
                    col[q] = 8 * (cu + s.gp - s.gl - 1) - sc;
                    e[q] = ((co0 + c) * s.Ho + oh) * s.Wo + col[q];
                    load_unit<T>(rg, e[q], 1, s.Cout * s.L, oh >= s.Ho || co0 + c >= s.Cout || i >= s.ng, u[q]);
                }
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    mend_unit<T>(e[q], 1, s.Cout * s.L, clip_g, col[q], s.Wo, u[q]);
                    if (bias_here && at[q] >= 0) {
                        float f[8];
#pragma unroll
                        for (int k = 0; k < 8; ++k) f[k] = as_f32<T>(u[q].v[k]);
                        const float t8 = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
                        float *sum = bias_sums + base + t + kThreads * q;
                        *sum = oh0 == 0 ? t8 : *sum + t8;
                    }
                    if (at[q] >= 0) store_unit<T, NP>(LG + at[q], s.pg, u[q]);
                }
            }
        };

        // Slots 0 .. 2: the tap rows of the wave's own column; 3 and 4: of the
        // column that the two waves share, the rows of slots 0 and 1.  The second
        // wave's slots start at row 2, so that its one shared tap is slot 3.
        // big: the h*h products; rest: the five smaller ones.
        const int ym = vl == 3 ? 2 * half : vl == 2 ? half : 0;
        const int own = vl == 1 ? (half ? 1 : 2) : 3, shared = vl == 3 ? (half ? 1 : 2) : 0;
        int row[kT];
        bool on[kT + 2];
#pragma unroll
        for (int x = 0; x < kT; ++x) {
            row[x] = half ? (x + 2) % 3 : x;
            on[x] = FULL || (x < own && row[x] < ul);
        }
        on[3] = FULL || (shared >= 1 && row[0] < ul);
        on[4] = shared == 2 && (FULL || row[1] < ul);
        f32x16_t big[kT + 2], rest[kT + 2];
#pragma unroll
        for (int x = 0; x < kT + 2; ++x)
#pragma unroll
            for (int r = 0; r < 16; ++r) big[x][r] = rest[x][r] = 0.0f;

        const char *ax = LX + (32 * wi + li) * s.csx, *bx = LG + (32 * wo + li) * s.csg;
        const int rowb = s.NU * 16;
        int arow[kT];
#pragma unroll
        for (int x = 0; x < kT; ++x) arow[x] = (FULL || row[x] < ul ? row[x] : 0) * rowb;
        auto multiply = [&](int rows) {
            const int steps = (rows * s.NU + 1) / 2;
            for (int ks = wk; ks < steps; ks += WK) {
                const int U = 2 * ks + kg, r = (U * s.inv_nu) >> 16, cu = U - r * s.NU;
                const char *pa = ax + (r * s.sh * s.NU + cu) * 16;
                const char *pb = bx + (r * s.gp + 1 + cu) * 16;
                bf16x8_t qm[NP], qs[NP];
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const u32x4_t w = *reinterpret_cast<const u32x4_t *>(pb + p * s.pg);
                    const uint32_t before = *reinterpret_cast<const uint32_t *>(pb + p * s.pg - 4);
                    // column vc + sw takes GY[c - s - 1], one column earlier; vc - sw one later
                    u32x4_t e;
#pragma unroll
                    for (int k = 3; k >= 1; --k) e[k] = __builtin_amdgcn_alignbit(w[k], w[k - 1], 16);
                    e[0] = __builtin_amdgcn_alignbit(w[0], before, 16);
                    qs[p] = __builtin_bit_cast(bf16x8_t, e);
                    u32x4_t m = w;
                    if (ym == 1) {
                        m = e;
                    } else if (ym == 2) {
                        const uint32_t after = *reinterpret_cast<const uint32_t *>(pb + p * s.pg + 16);
#pragma unroll
                        for (int k = 0; k < 3; ++k) m[k] = __builtin_amdgcn_alignbit(w[k + 1], w[k], 16);
                        m[3] = __builtin_amdgcn_alignbit(after, w[3], 16);
                    }
                    qm[p] = __builtin_bit_cast(bf16x8_t, m);
                }
                // by parts of X: only one part's operands are held at a time
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    bf16x8_t a[kT];
#pragma unroll
                    for (int x = 0; x < kT; ++x) a[x] = *reinterpret_cast<const bf16x8_t *>(pa + p * s.px + arow[x]);
#pragma unroll
                    for (int o = NP - 1 - p; o >= 0; --o) {
#pragma unroll
                        for (int x = 0; x < kT; ++x)
                            if (on[x]) {
                                f32x16_t &d = p + o ? rest[x] : big[x];
                                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[x], qm[o], d, 0, 0, 0);
                            }
                        if (on[3]) {
                            f32x16_t &d = p + o ? rest[3] : big[3];
                            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], qs[o], d, 0, 0, 0);
                        }
                    }
                    if (on[4]) {
#pragma unroll
                        for (int o = NP - 1 - p; o >= 0; --o) {
                            f32x16_t &d = p + o ? rest[4] : big[4];
                            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], qs[o], d, 0, 0, 0);
                        }
                    }
                }
            }
        };

        for (int oh0 = 0; oh0 < s.Ho; oh0 += s.RC) {
            lds_barrier();                               // the previous chunk (or the zeroing) is done
            stage_x(oh0);
            stage_g(oh0);
            lds_barrier();
            multiply(s.Ho - oh0 < s.RC ? s.Ho - oh0 : s.RC);
        }
        lds_barrier();

        if (bias_here && tid < 32 * WO && co0 + tid < s.Cout) {
            const int units = s.RC * s.gl;               // of one channel, added in unit order
            float t = 0.0f;
            for (int k = 0; k < units; ++k) t += bias_sums[tid * units + k];
            t *= scale;
            gb[(i64)n * s.Cout + co0 + tid] = t;
            sq += t * t;
        }
        if (s.bias_at) lds_barrier();                    // the output and hand-over staging may lie over the sums
        if constexpr (NP == 3) {
#pragma unroll
            for (int x = 0; x < kT + 2; ++x) big[x] += rest[x];
        }
        // waves that share a block: partial sums handed over through LDS, in wave order
        if constexpr (WK > 1) {
            float *hand = reinterpret_cast<float *>(smem) + lane;
            if (wk > 0) {
                float *h = hand + (wave - 2 * WI * WO) * (1024 * (kT + 2));
#pragma unroll
                for (int x = 0; x < kT + 2; ++x)
#pragma unroll
                    for (int r = 0; r < 16; ++r) h[1024 * x + 64 * r] = big[x][r];
            }
            lds_barrier();
            if (wk == 0) {
#pragma unroll
                for (int w = 1; w < WK; ++w) {
                    const float *h = hand + (wave + (w - 1) * 2 * WI * WO) * (1024 * (kT + 2));
#pragma unroll
                    for (int x = 0; x < kT + 2; ++x)
#pragma unroll
                        for (int r = 0; r < 16; ++r) big[x][r] += h[1024 * x + 64 * r];
                }
            }
            lds_barrier();
        }
        // big[x], register r of lane l: ci = ci0 + 32 wi + 8 (r / 4) + 4 (l / 32) + r % 4,
        // co = co0 + 32 wo + l % 32, tap row u0 + row[x % 3], tap column vm, or vs for x >= 3
        const int vm = vc + (ym == 0 ? 0 : ym == 1 ? s.sw : -s.sw), vs = vc + s.sw;
        const int ln = here(lane), el = ln & 31, eg = ln >> 5;
        const int co = co0 + 32 * wo + el, cib = ci0 + 32 * wi + 4 * eg;
        float *G = gW + (i64)n * s.Cout * s.Cin * s.khw;
        float gsq = 0.0f;
#pragma unroll
        for (int x = 0; x < kT + 2; ++x)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float g = scale * big[x][r];
                big[x][r] = g;
                // (slots that are not in use stayed zero)
                const float in = co < s.Cout && cib + 8 * (r >> 2) + (r & 3) < s.Cin ? g : 0.0f;
                gsq += in * in;
            }
        if (wk != 0) gsq = 0.0f;
        const bool bad = __any(!finite_f32(gsq));
        if (FULL && s.full) {
            // Through LDS, so that the waves of a block store whole rows of it:
            // 32 channels x 9 taps are 1152 consecutive bytes.
            // (an odd row length: the lanes' rows start in different banks)
            constexpr int LD = 289;
            float *buf = reinterpret_cast<float *>(smem) + blk * (32 * LD);
            if (wk == 0) {
                float *w = buf + el * LD + 36 * eg;
#pragma unroll
                for (int x = 0; x < kT + 2; ++x) {
                    if (x == 4 && !on[4]) break;
                    float *wx = w + 3 * row[x % kT] + (x < kT ? vm : vs);
#pragma unroll
                    for (int r = 0; r < 16; ++r) wx[9 * (8 * (r >> 2) + (r & 3))] = big[x][r];
                }
            }
            lds_barrier();
            if (wk == 0) {
                const int left = 9 * (s.Cin - ci0 - 32 * wi);    // outputs of a row inside the layer
                const int rows = s.Cout - co0 - 32 * wo;
                float *p = G + ((i64)(co0 + 32 * wo) * s.Cin + ci0 + 32 * wi) * 9;
                const int pitch = s.Cin * 9;
                // nine waves' worth of words for every two rows of 288
#pragma unroll
                for (int k0 = 0; k0 < 8; ++k0) {
#pragma unroll
                    for (int k1 = 0; k1 < 9; ++k1) {
                        const int i = ln + kWave * k1, odd = i >= 288, k = i - (odd ? 288 : 0), rw = 2 * (half + 2 * k0) + odd;
                        const float f = buf[rw * LD + k];
                        if (rw < rows && k < left) p[rw * pitch + k] = f;
                    }
                }
            }
        } else if (wk == 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int c = cib + 8 * (r >> 2) + (r & 3);
                if (co >= s.Cout || c >= s.Cin) continue;
                float *p = G + ((i64)co * s.Cin + c) * s.khw + u0 * s.kw;
#pragma unroll
                for (int x = 0; x < kT + 2; ++x)
                    if (on[x]) p[row[x % kT] * s.kw + (x < kT ? vm : vs)] = big[x][r];
            }
        }
        if (__syncthreads_or(bad)) [[unlikely]] {
            // An infinity, a NaN or a value past bf16's range among the inputs,
            // or outputs whose squares pass fp32's range: the wave's outputs
            // again (the stores above are done: the barrier waits for them),
            // as plain fp32 sums.
            if (bad) {
                gsq = 0.0f;
                for (int e = ln; e < 1024 * (kT + 2); e += kWave) {
                    const int x = e >> 10, c = ci0 + 32 * wi + (e & 31), o = co0 + 32 * wo + ((e >> 5) & 31);
                    const int u = u0 + (x % kT == 0 ? row[0] : x % kT == 1 ? row[1] : row[2]), v = x < kT ? vm : vs;
                    if (!(x == 0 ? on[0] : x == 1 ? on[1] : x == 2 ? on[2] : x == 3 ? on[3] : on[4])) continue;
                    if (c >= s.Cin || o >= s.Cout) continue;
                    float t = 0.0f;
                    for (int oh = 0; oh < s.Ho; ++oh) {
                        const int ih = oh * s.sh + u - s.ph;
                        if (ih < 0 || ih >= s.H) continue;
                        for (int ow = 0; ow < s.Wo; ++ow) {
                            const int iw = ow * s.sw + v - s.pw;
                            if (iw >= 0 && iw < s.W)
                                t = fmaf(as_f32<T>(Gn[(o * s.Ho + oh) * s.Wo + ow]),
                                         as_f32<T>(Xn[(c * s.H + ih) * s.W + iw]), t);
                        }
                    }
                    t *= scale;
                    G[((i64)o * s.Cin + c) * s.khw + u * s.kw + v] = t;
                    gsq += t * t;
                }
            }
        }
        sq += gsq;
        if (gi + 1 < s.ngrp && gi + 1 < (gpart + 1) * s.gpw) {
            // the output staging and hand-over wrote over the guards
            lds_barrier();
            for (int i = tid; i < (NP * (s.px + s.pg)) / 16; i += kThreads)
                *reinterpret_cast<uint4 *>(smem + 16 * i) = make_uint4(0u, 0u, 0u, 0u);
        }
    }

    // Bias: 16 lanes per output channel, over its positions; the workgroups of
    // a channel tile's input channel tiles share its channels.
    if (gb && gpart == 0 && !s.bias_at) {
        const int share = (32 * WO + s.nci - 1) / s.nci, l16 = lane & 15;
        const int last = co0 + (cit + 1) * share < s.Cout ? co0 + (cit + 1) * share : s.Cout;
        for (int c0 = co0 + cit * share; c0 < last; c0 += 4 * kWaves) {
            const int co = c0 + 4 * wave + (lane >> 4);
            const bool on = co < last && co < co0 + 32 * WO;
            float t = 0.0f;
            const T *g = Gn + (i64)(on ? co : co0) * s.L;
            const int whole = s.L & ~3;
            for (int p0 = 4 * l16; p0 < whole; p0 += 64 * 8) {
                struct __attribute__((packed, aligned(sizeof(T)))) G4 { T v[4]; };
                G4 v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    v[k] = *reinterpret_cast<const G4 *>(g + (p0 + 64 * k < whole ? p0 + 64 * k : 0));
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float f = (as_f32<T>(v[k].v[0]) + as_f32<T>(v[k].v[1])) + (as_f32<T>(v[k].v[2]) + as_f32<T>(v[k].v[3]));
                    t += p0 + 64 * k < whole ? f : 0.0f;
                }
            }
            if (whole + l16 < s.L) t += as_f32<T>(g[whole + l16]);
#pragma unroll
            for (int d = 8; d >= 1; d >>= 1) t += __shfl_xor(t, d, kWave);
            t *= scale;
            if (on && l16 == 0) {
                gb[(i64)n * s.Cout + co] = t;
                sq += t * t;
            }
        }
    }
    sq = wave_sum(sq);
    if (lane == 0) red[wave] = sq;
    lds_barrier();
    if (sqout && tid == 0) sqout[(i64)n * s.tiles + (b - n * (uint32_t)s.tiles)] =
            (red[0] + red[1]) + (red[2] + red[3]);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct Layout {
    int wi, wo, wk;
};
constexpr Layout kLayouts[] = {{1, 2, 1}, {2, 1, 1}, {1, 1, 2}};
// output staging of two blocks (the hand-over needs less)
constexpr size_t kLeastLds = 2 * 32 * 289 * 4;

int odd_units(int bytes) { return (((bytes + 15) / 16) | 1) * 16; }

bool plan(const ConvRowsArgs &a, bool bf16, int slots, const Layout &w, SplitShape &s)
{
    s.Cin = (int)a.Cin; s.H = (int)a.H; s.W = (int)a.W; s.Cout = (int)a.Cout; s.Ho = (int)a.Ho; s.Wo = (int)a.Wo;
    s.kh = (int)a.kh; s.kw = (int)a.kw; s.sh = (int)a.sh; s.sw = (int)a.sw; s.ph = (int)a.ph; s.pw = (int)a.pw;
    s.L = s.Ho * s.Wo;
    s.khw = s.kh * s.kw;
    const int np = bf16 ? 1 : 3;
    // columns of one phase, and room for the outputs that only reach padding
    const int cols = (s.W + s.sw - 1) / s.sw;
    s.NU = (cols + 7) / 8;
    s.inv_nu = (65536 + s.NU - 1) / s.NU;
    s.nci = (s.Cin + 32 * w.wi - 1) / (32 * w.wi);
    s.nco = (s.Cout + 32 * w.wo - 1) / (32 * w.wo);
    // tap groups: rows in balanced threes; columns of one phase in balanced threes
    s.ngrp = 0;
    bool all3 = true, zero_ends = true;
    const int nu = (s.kh + kT - 1) / kT;
    for (int i = 0; i < nu; ++i) {
        const int u0 = i * s.kh / nu, u1 = (i + 1) * s.kh / nu;
        for (int f = 0; f < s.sw && f < s.kw; ++f) {
            const int nv = (s.kw - f + s.sw - 1) / s.sw, parts = (nv + kT - 1) / kT;   // v = f, f + sw, ...
            for (int j = 0; j < parts; ++j) {
                const int v0 = j * nv / parts, v1 = (j + 1) * nv / parts, vl = v1 - v0;
                if (s.ngrp == kMaxGroups) return false;
                const int vc = f + s.sw * (v0 + (vl == 3 ? 1 : 0));
                const int dv = vc - s.pw, sc = dv >= 0 ? dv / s.sw : -((s.sw - 1 - dv) / s.sw);
                s.g[s.ngrp++] = {(int8_t)u0, (int8_t)(u1 - u0), (int8_t)vc, (int8_t)vl, (int16_t)sc, (int16_t)(dv - sc * s.sw)};
                all3 = all3 && vl == 3 && u1 - u0 == 3;
                // GY[-1 - sc] and GY[8 NU - sc] are outside the row
                zero_ends = zero_ends && (vl == 1 || (sc >= 0 && 8 * s.NU - sc >= s.Wo));
            }
        }
    }
    s.gl = zero_ends ? s.NU : s.NU + 2;
    s.gp = zero_ends ? s.NU + 1 : s.NU + 2;
    s.inv_gl = (65536 + s.gl - 1) / s.gl;
    s.full = all3 ? (s.kh == 3 && s.kw == 3 && s.sw == 1 ? 2 : 1) : 0;
    const int room = slots / (s.nci * s.nco);
    if (room < 1) return false;
    s.gpw = (s.ngrp + room - 1) / room;
    s.tiles = s.nci * s.nco * ((s.ngrp + s.gpw - 1) / s.gpw);
    // every column of GY is in exactly one unit of the first group
    const int first = -8 * (s.gp - s.gl - 1) + s.g[0].sc;
    const bool covers = first >= 0 && 8 * s.gl - first >= s.Wo;
    // the most output rows per chunk that fit
    s.RC = 0;
    for (int rc = s.Ho < 64 ? s.Ho : 64; rc >= 1; --rc) {
        const int xr = (rc - 1) * s.sh + (s.kh < kT ? s.kh : kT);
        const i64 nx = (i64)32 * w.wi * xr * s.NU, ng = (i64)32 * w.wo * rc * s.gl;
        if ((i64)xr * s.NU * nx >= (1 << 20) || (i64)rc * s.gl * ng >= (1 << 20)) continue;   // div20
        // an odd number of units leaves one step a unit past the chunk: it reads
        // X at row (rc - 1) * sh + 2 + sh (any finite value) and GY's two units
        // from rc * gp + 1 on (zeros)
        const int csx = odd_units(((xr + s.sh - 1) * s.NU + 1) * 16), csg = odd_units((rc * s.gp + 3) * 16);
        const int px = 32 * w.wi * csx, pg = 32 * w.wo * csg;
        const i64 total = (i64)np * (px + pg) + (covers ? 4 * ng : 0);
        if (total > (i64)kLds) continue;
        const int chunks = (s.Ho + rc - 1) / rc, even = (s.Ho + chunks - 1) / chunks;
        if (even < rc) {                                 // the same number of chunks, of equal size
            rc = even + 1;
            continue;
        }
        s.bias_at = covers ? np * (px + pg) : 0;
        s.RC = rc; s.XR = xr; s.csx = csx; s.csg = csg; s.px = px; s.pg = pg; s.nx = (int)nx; s.ng = (int)ng;
        break;
    }
    if (s.RC == 0) return false;
    s.inv_xrow = ((1 << 20) + s.XR * s.NU - 1) / (s.XR * s.NU);
    s.inv_grow = ((1 << 20) + s.RC * s.gl - 1) / (s.RC * s.gl);
    return true;
}

// A plan's time in cycles, from measured parts: a workgroup's start, output and
// end; per chunk the staging's round trip and its units (256 threads, the
// splitting of one unit each); per step the MFMAs of the wave with more taps.
// Two workgroups share a CU: one stages while the other multiplies.
double cost_of(const SplitShape &s, const Layout &w, i64 N, bool bf16)
{
    const int chunks = (s.Ho + s.RC - 1) / s.RC, steps = ((s.RC * s.NU + 1) / 2 + w.wk - 1) / w.wk;
    const double units = (s.nx + 255) / 256 + (s.ng + 255) / 256, np = bf16 ? 1 : 6;
    double c = 0;
    for (int i = 0; i < s.ngrp; ++i) {
        const int taps = s.g[i].vl == 3 ? (3 * s.g[i].ul + 1) / 2 : s.g[i].vl == 2 ? s.g[i].ul : (s.g[i].ul + 1) / 2;
        const double mult = steps * (taps * np * 32.0 + 120.0), stage = 3000.0 + units * (bf16 ? 400.0 : 600.0);
        c += chunks * (2 * mult > stage ? mult + (stage > mult ? stage : mult) : mult + stage) + 6000.0;
    }
    const double groups = (double)s.ngrp / s.gpw;
    const double rounds = (double)N * s.tiles / 512.0;
    return (c / groups + 8000.0) * (rounds > 1.0 ? rounds : 1.0);
}

bool choose(const ConvRowsArgs &a, bool bf16, int slots, SplitShape &best, int &which)
{
    // 32-bit offsets, taps in eight bits, and the quotients of inv_nu and div20
    if (a.kh > 100 || a.kw > 100 || a.W > 2048 || a.Cin * a.H * a.W >= (i64(1) << 28) ||
        a.Cout * a.Ho * a.Wo >= (i64(1) << 28) || a.Cin * a.kh * a.kw * a.Cout >= (i64(1) << 30) || a.ph > a.H + a.kh ||
        a.pw > 1024 || a.ph > 1024 || a.H > (1 << 20))
        return false;
    which = -1;
    double cost = 0;
    for (int k = 0; k < (int)(sizeof(kLayouts) / sizeof(kLayouts[0])); ++k) {
        SplitShape s;
        if (!plan(a, bf16, slots, kLayouts[k], s)) continue;
        const double c = cost_of(s, kLayouts[k], a.N, bf16);
        if (which < 0 || c < cost) {
            best = s;
            which = k;
            cost = c;
        }
    }
    return which >= 0;
}

template <typename T, int WI, int WO, int WK>
void launch(const ConvRowsArgs &a, const SplitShape &s, float scale, float *gW, float *gb, float *sqout,
            hipStream_t stream)
{
    const int np = sizeof(T) == 4 ? 3 : 1;
    size_t lds = (size_t)np * (s.px + s.pg) + (s.bias_at ? 4 * s.ng : 0);
    const size_t least = s.full ? kLeastLds : WK > 1 ? 2 * (kT + 2) * 4096 : 0;
    if (lds < least) lds = least;
    const unsigned grid = (unsigned)(a.N * s.tiles);
    if (s.full)
        conv_split_kernel<T, WI, WO, WK, true><<<grid, kThreads, lds, stream>>>((const T *)a.X, (const T *)a.GY, s,
                                                                              scale, gW, gb, sqout);
    else
        conv_split_kernel<T, WI, WO, WK, false><<<grid, kThreads, lds, stream>>>((const T *)a.X, (const T *)a.GY, s,
                                                                               scale, gW, gb, sqout);
}

template <typename T>
void dispatch(int which, const ConvRowsArgs &a, const SplitShape &s, float scale, float *gW, float *gb, float *sqout,
              hipStream_t stream)
{
    switch (which) {
    case 0: launch<T, 1, 2, 1>(a, s, scale, gW, gb, sqout, stream); break;
    case 1: launch<T, 2, 1, 1>(a, s, scale, gW, gb, sqout, stream); break;
    default: launch<T, 1, 1, 2>(a, s, scale, gW, gb, sqout, stream); break;
    }
}

}  // namespace

// Measured against the row-chunked fp32 MFMA kernel (us, that one / this one).
// What decides is the positions a workgroup contracts per output it stores,
// so the rule is on useful = positions x the filled part of the channel blocks.
// fp32, 3 x 3 at stride 1, useful >= 96: 512 samples 32 -> 64 @32^2 192 / 130,
// 64 -> 128 @16^2 223 / 160, 256 samples 64 -> 64 @12^2 41 / 37, 128 samples
// 24 -> 48 @30^2 173 / 79; below: 512 samples 128 -> 256 @8^2 (useful 64)
// 264 / 281, 300 samples 100 -> 24 @9^2 (47) 52 / 62.  fp32 at stride 2 splits
// a group's columns by phase: 100 samples 48 -> 96 @27^2 72 / 93, but where
// the other kernel's grid leaves CUs idle 64 samples 64 -> 64 @28^2 82 / 45.
// fp32 5 x 5 and 7 x 7 (partly filled groups, several per workgroup): 26 / 41,
// 65 / 106, 24 / 58, 53 / 86.
// bf16 (one product instead of six, against widened fp32 ones), useful >= 40, or 90
// with more than four groups: 100 samples 24 -> 40 @27^2 5 x 5 stride 2
// 59 / 35, 512 samples 64 -> 128 @16^2 221 / 120, 300 samples 100 -> 24 @9^2
// 53 / 35, 50 samples 40 -> 40 @13^2 5 x 5 41 / 32; below: 200 samples
// 64 -> 30 @6^2 17 / 19, 64 samples 24 -> 24 @20^2 7 x 7 stride 2 24 / 33.
bool conv_split_ok(const ConvRowsArgs &a, bool bf16, int slots)
{
    if (a.Cin < 24 || a.kh * a.kw < 2 || a.N * slots >= (i64(1) << 31)) return false;
    const double fill = (double)(a.Cin * a.Cout) / (double)(ceil_div(a.Cin, 32) * ceil_div(a.Cout, 32) * 1024);
    const double useful = (double)(a.Ho * a.Wo) * fill;
    SplitShape s;
    int which;
    if (useful < 40.0 || !choose(a, bf16, slots, s, which)) return false;
    if (bf16) return useful >= (s.ngrp > 4 ? 90.0 : 40.0);
    if (a.kh != 3 || a.kw != 3) return false;
    if (a.sh == 1 && a.sw == 1) return useful >= 96.0;
    return useful >= 64.0 && a.N * conv_rows_tiles(a) < 256;
}

void conv_split_launch(const ConvRowsArgs &a, bool bf16, int slots, float scale, float *gW, float *gb, float *sqnorm,
                       float *partial, hipStream_t stream)
{
    SplitShape s;
    int which;
    if (!choose(a, bf16, slots, s, which)) return;      // conv_split_ok said yes
    const bool direct = s.tiles == 1;
    s.full = s.full == 2 ? 1 : 0;
    float *sqout = sqnorm ? (direct ? sqnorm : partial) : nullptr;
    if (bf16) dispatch<uint16_t>(which, a, s, scale, gW, gb, sqout, stream);
    else dispatch<float>(which, a, s, scale, gW, gb, sqout, stream);
    if (sqnorm && !direct) sum_partials(partial, a.N, s.tiles, sqnorm, stream);
}

}  // namespace dpg
