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
// workgroups of a round issue at about the same time.  162 us against 223 on
// fp32 MFMA; off 64 bits by 0.68e-7 (weights) and 0.84e-7 (bias) against 1.92e-7
// and 1.51e-7; 32 -> 64 @32^2 130 against 192.  Tried: nine taps per wave with one accumulator each (faster staging
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
#include "conv2d_split_plan.hpp"

namespace dpg {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
using split::finite_f32;
using namespace csplit;

constexpr int kThreads = 256, kWaves = 4;
constexpr int kBatch = 2;              // units per thread loaded at once
// output staging of two blocks (the hand-over needs less)
constexpr size_t kLeastLds = 2 * 32 * 289 * 4;

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

// FULL: 3 x 3 taps in one group
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

        const bool clip_x = clips_x(s), clip_g = clips_g(s, sc);
        // One chunk into LDS, kBatch units per thread in flight.  Nothing of it stays in
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
                    const UnitAt a = x_unit(s, u0, phase, ci0, oh0, base + t + kThreads * q);
                    at[q] = a.at;
                    col[q] = a.col;
                    e[q] = a.e;
                    load_unit<T>(rx, a.e, s.sw, s.Cin * s.H * s.W, a.dead, u[q]);
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
                    const UnitAt a = g_unit(s, sc, co0, oh0, base + t + kThreads * q);
                    at[q] = a.at;
                    col[q] = a.col;
                    e[q] = a.e;
                    load_unit<T>(rg, a.e, 1, s.Cout * s.L, a.dead, u[q]);
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
            for (int x = 0; x < kT + 2; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) big[x][r] = split::kUnscale * (big[x][r] + rest[x][r]);
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
        // (s.full always holds with FULL; without that condition the compiler allots the registers of the loop above
        // differently: bf16, 512 samples 64 -> 128 @16^2, 120 us against 101)
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
            // An infinity, a NaN or a value too large to split among the inputs,
            // or outputs whose squares pass fp32's range: the wave's outputs
            // again (the stores above are done: the barrier waits for them),
            // on fp32 MFMA, positions 2q + l / 32 of a step straight from memory
            // (512 samples, 64 -> 128 @16^2, all with a NaN 1100 us; by one fma
            // per lane and position 17100).
            if (bad) {
                constexpr int U = 8;
                const int c = ci0 + 32 * wi + el;
                const T *xc = Xn + (c < s.Cin ? c : 0) * s.H * s.W, *yo = Gn + (co < s.Cout ? co : 0) * s.L;
                gsq = 0.0f;
#pragma unroll 1
                for (int x = 0; x < kT + 2; ++x) {
                    if (!(x == 0 ? on[0] : x == 1 ? on[1] : x == 2 ? on[2] : x == 3 ? on[3] : on[4])) continue;
                    const int u = u0 + (x % kT == 0 ? row[0] : x % kT == 1 ? row[1] : row[2]), v = x < kT ? vm : vs;
                    f32x16_t d;
#pragma unroll
                    for (int r = 0; r < 16; ++r) d[r] = 0.0f;
                    for (int p0 = 0; p0 < s.L; p0 += 2 * U) {
                        float a[U], b[U];
#pragma unroll
                        for (int q = 0; q < U; ++q) {
                            const int p = p0 + 2 * q + eg, oh = (int)((uint32_t)p / (uint32_t)s.Wo);
                            const int ih = oh * s.sh + u - s.ph, iw = (p - oh * s.Wo) * s.sw + v - s.pw;
                            // a position outside the input is no term of the sum
                            const bool in = p < s.L && (uint32_t)ih < (uint32_t)s.H && (uint32_t)iw < (uint32_t)s.W;
                            a[q] = in && c < s.Cin ? as_f32<T>(xc[ih * s.W + iw]) : 0.0f;
                            b[q] = in && co < s.Cout ? as_f32<T>(yo[p]) : 0.0f;
                        }
#pragma unroll
                        for (int q = 0; q < U; ++q) d = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], d, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int ch = cib + 8 * (r >> 2) + (r & 3);
                        if (co >= s.Cout || ch >= s.Cin) continue;
                        const float g = scale * d[r];
                        G[((i64)co * s.Cin + ch) * s.khw + u * s.kw + v] = g;
                        gsq += g * g;
                    }
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

ConvGeom geom(const ConvRowsArgs &a)
{
    return {a.N, a.Cin, a.H, a.W, a.Cout, a.Ho, a.Wo, a.kh, a.kw, a.sh, a.sw, a.ph, a.pw};
}

}  // namespace

// Measured against the row-chunked fp32 MFMA kernel (us, that one / this one).
// What decides for a full chip is the positions a workgroup contracts per output it stores,
// so the first rule is on useful = positions x the filled part of the channel blocks.
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
double conv_split_us(const ConvRowsArgs &a, bool bf16, int slots)
{
    if (a.Cin < 24 || a.kh * a.kw < 2 || a.N * slots >= (i64(1) << 31)) return 0.0;
    const double fill = (double)(a.Cin * a.Cout) / (double)(ceil_div(a.Cin, 32) * ceil_div(a.Cout, 32) * 1024);
    const double useful = (double)(a.Ho * a.Wo) * fill;
    if (useful < 40.0) return 0.0;
    if (!bf16) {
        if (a.kh != 3 || a.kw != 3) return 0.0;
        if (a.sh == 1 && a.sw == 1 ? useful < 96.0 : useful < 64.0 || a.N * conv_rows_tiles(a) >= 256) return 0.0;
    }
    SplitShape s;
    int which;
    if (!choose(geom(a), bf16, slots, s, which) || (bf16 && s.ngrp > 4 && useful < 90.0)) return 0.0;
    return split_us(s, kLayouts[which], bf16, cu_rounds((double)a.N * s.tiles, 2, 0.85),
                    (double)ceil_div(a.N * s.tiles, 256));
}

void conv_split_launch(const ConvRowsArgs &a, bool bf16, int slots, float scale, float *gW, float *gb, float *sqnorm,
                       float *partial, hipStream_t stream)
{
    SplitShape s;
    int which;
    if (!choose(geom(a), bf16, slots, s, which)) return;      // conv_split_us took it
    const bool direct = s.tiles == 1;
    float *sqout = sqnorm ? (direct ? sqnorm : partial) : nullptr;
    if (bf16) dispatch<uint16_t>(which, a, s, scale, gW, gb, sqout, stream);
    else dispatch<float>(which, a, s, scale, gW, gb, sqout, stream);
    if (sqnorm && !direct) sum_partials(partial, a.N, s.tiles, sqnorm, stream);
}

}  // namespace dpg
