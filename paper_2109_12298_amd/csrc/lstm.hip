// Backward through time of an LSTM layer: the gate backprop that the per-
// sample gradients of its two weight matrices take as B.
//
// The paper's recurrent modules (DPLSTM) are its costliest per-sample layers:
// an LSTM's weights act as one Linear layer on the input x_t and one on the
// previous hidden state h_{t-1}, both fed the gradient with respect to the gate
// pre-activations z_t, and that gradient comes from the recurrence run
// backwards.  With PyTorch's gate order (i, f, g, o), zero initial state and
// the loss gradient arriving at the hidden states (dh_out at every step
// and/or dh_last at the last), for t = T-1 down to 0:
//   dh      = dh_out_t (+ dh_last at T-1) + W_hh^T delta_{t+1}   (no term at T-1)
//   dc_t    = dh * o * (1 - tanh(c_t)^2) + dc_{t+1} * f_{t+1}
//   delta_i = dc_t * g * i (1 - i)          delta_f = dc_t * c_{t-1} * f (1 - f)
//   delta_g = dc_t * i * (1 - g^2)          delta_o = dh * tanh(c_t) * o (1 - o)
//
// The steps of one sample are a chain, so the kernel is built for the
// latency of one step.  One workgroup per sample.  A group of 16 lanes owns UP
// consecutive hidden units: lane k holds, in registers, their weights for gate
// rows 2k and 2k + 1 (mod 32), so W_hh is read once per workgroup and a value
// of delta_{t+1} read from LDS (8 bytes per lane, the groups of a wave the same
// ones) feeds UP multiply-adds.  The 16 lanes' partial sums are added in four
// steps of lane permutes, of which the first two also distribute four units
// (each lane passes half of them on and keeps the other half), so that a
// unit's sum ends in four lanes, one per gate.  What of the update does not
// depend on delta_{t+1} (all but two multiply-adds and a product) is computed
// while its reads are on their way.  delta is double-buffered in LDS, so one
// barrier per step.  The gate activations and cell states of a step are loaded
// kRing steps ahead into a register ring, so their latency is hidden behind
// the chain.
//
// What bounds it: VALU issue.  A wave issues an instruction about every five
// cycles, two waves of a SIMD overlap, so a step costs what one wave's
// instructions cost (about 150 at H = 100, 104 of them multiply-adds) as long
// as no SIMD has more than two; of the 0.6 us of a step at H = 100 another 0.25
// are its chain (LDS write, barrier, LDS read, the permutes), which is all that
// is left at H = 14.  64 samples, T = 256, H = 100: 160 us, against 184 with four lanes per
// unit, where every wave read all of delta for a quarter as many
// multiply-adds; 32 samples, T = 100, H = 120 73 / 93; 300 samples, T = 128,
// H = 80 88 / 198; 512 samples, T = 64, H = 100 89 / 109; 16 samples, T = 100,
// H = 32 34 / 36.  The weights are loaded UP at a time: one by one, that prologue was 9 us of
// the 168 it then took at H = 100.
#include "common.hpp"

#include <type_traits>

namespace dpg {
namespace {

// tanh(x) = 1 - 2 / (1 + e^{2x}), from the hardware base-2 exponential and
// reciprocal (about 1e-7 absolute error; e^{2x} overflowing to infinity gives
// 1, underflowing to 0 gives -1)
__device__ __forceinline__ float tanh_exp(float x)
{
    const float e = __builtin_amdgcn_exp2f(x * 2.8853900817779268f);   // 2 log2(e)
    return 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + e);
}

constexpr int kMaxH = 128;

// KM: pieces of 32 gate rows (4H <= 32 KM); UP: units per group of 16 lanes;
// DHO: a loss gradient at every hidden state is given
template <int KM, int UP, bool DHO>
__global__ __launch_bounds__(UP > 4 ? 256 : 512) void lstm_bptt_kernel(const float *__restrict__ gates, const float *__restrict__ c,
                                                        const float *__restrict__ W_hh,
                                                        const float *__restrict__ dh_out,
                                                        const float *__restrict__ dh_last, i64 T64, int H,
                                                        float *__restrict__ delta)
{
    constexpr int kRing = 6, NV = DHO ? 6 : 5;
    __shared__ __attribute__((aligned(16))) float dbuf[2][32 * KM];
    const i64 n = blockIdx.x;
    const int tid = threadIdx.x, grp = tid >> 4, k16 = tid & 15;
    const bool b0 = k16 & 1, b1 = k16 & 2, b2 = k16 & 4, b3 = k16 & 8;
    // the unit and the gate whose delta this lane ends with
    // (above four units: the two gates 2 q and 2 q + 1)
    const int slot = UP > 4 ? 4 * b2 + 2 * b1 + b0 : UP > 2 ? 2 * b2 + b0 : UP == 2 ? b2 : 0;
    const int q = UP > 4 ? b3 : UP > 2 ? 2 * b3 + b1 : 2 * b1 + b0;
    const int G = 4 * H, T = (int)T64, u = grp * UP + slot;
    const bool live = slot < UP && u < H && (UP > 2 || (!b3 && (UP == 2 || !b2)));
    const int uu = u < H ? u : 0;

    // weights of units grp * UP + j for gate rows 2 k16 + 32 m + r (zero past the layer)
    // a group's units of a row are consecutive: one load where it has all of them
    struct __attribute__((packed, aligned(4))) Units {
        float v[UP];
    };
    float w[KM][2][UP];
    const int v0 = grp * UP;
    const bool whole = v0 + UP <= H;
#pragma unroll
    for (int m = 0; m < KM; ++m)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int g = 2 * k16 + 32 * m + r;
            const float *row = W_hh + (i64)(g < G ? g : 0) * H + (whole ? v0 : 0);
            const Units x = *reinterpret_cast<const Units *>(row);      // UP <= H: inside the row
#pragma unroll
            for (int j = 0; j < UP; ++j) w[m][r][j] = whole && g < G ? x.v[j] : 0.0f;
        }
    if (!whole && v0 < H) {
#pragma unroll
        for (int m = 0; m < KM; ++m)
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int j = 0; j < UP; ++j) {
                    const int g = 2 * k16 + 32 * m + r;
                    if (g < G && v0 + j < H) w[m][r][j] = W_hh[(i64)g * H + v0 + j];
                }
    }
    for (int e = tid; e < 64 * KM; e += blockDim.x) (&dbuf[0][0])[e] = 0.0f;   // rows past 4H stay zero

    float *dn = delta + n * T64 * G;
    const float dlast = dh_last ? dh_last[n * H + uu] : 0.0f;
    const __amdgpu_buffer_rsrc_t rg = sample_rsrc(gates + n * T64 * G, (uint32_t)(T * G) * 4u);
    const __amdgpu_buffer_rsrc_t rc = sample_rsrc(c + n * T64 * H, (uint32_t)(T * H) * 4u);
    const __amdgpu_buffer_rsrc_t rh = sample_rsrc(DHO ? dh_out + n * T64 * H : c, (uint32_t)(T * H) * 4u);
    const int gb = 4 * H;           // bytes between gate blocks
    // {i, f, g, o, c_t(, dh_out_t)} of a step; a step before 0 reads zeros
    float ring[kRing][NV];
    auto load_step = [&](int t, float (&v)[NV]) {
        const uint32_t og = t < 0 ? kOutside : (uint32_t)(t * G + uu) * 4u;
        const uint32_t oc = t < 0 ? kOutside : (uint32_t)(t * H + uu) * 4u;
        v[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, og, 0, 0));
        v[1] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, og, gb, 0));
        v[2] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, og, 2 * gb, 0));
        v[3] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, og, 3 * gb, 0));
        v[4] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rc, oc, 0, 0));
        if constexpr (DHO) v[NV - 1] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rh, oc, 0, 0));
    };
    auto dpp = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, false));
    };
    typedef std::integral_constant<int, 0x141> HalfMirror;   // lane i of 8 <-> 7 - i
    typedef std::integral_constant<int, 0xB1> Xor1;
    typedef std::integral_constant<int, 0x4E> Xor2;
    typedef std::integral_constant<int, 0x128> Ror8;         // lane i of 16 <-> i + 8

    float dc_next = 0.0f, f_next = 0.0f;        // dc_{t+1} and f_{t+1}
    int cur = 0;
    auto step = [&](int t, const float (&v)[NV], float cp) {
        const float *d = dbuf[cur ^ 1] + 2 * k16;
        float2 x[KM];
#pragma unroll
        for (int m = 0; m < KM; ++m) x[m] = *reinterpret_cast<const float2 *>(d + 32 * m);
        const float gi = v[0], gf = v[1], gg = v[2], go = v[3];
        const float tc = tanh_exp(v[4]);
        float e = go * (1.0f - tc * tc);
        // lane q's gate: delta_q = (q == 3 ? dh : dc) * fac
        float fac, fac2 = 0.0f;
        if constexpr (UP > 4) {
            fac = q ? gi * (1.0f - gg * gg) : gg * (gi * (1.0f - gi));
            fac2 = q ? tc * (go * (1.0f - go)) : cp * (gf * (1.0f - gf));
        } else {
            const float gq = q == 0 ? gi : q == 1 ? gf : go;
            const float s2 = q == 0 ? gg : q == 1 ? cp : q == 2 ? gi : tc;
            fac = s2 * (q == 2 ? 1.0f - gg * gg : gq * (1.0f - gq));
        }
        float add = (DHO ? v[NV - 1] : 0.0f) + (t == T - 1 ? dlast : 0.0f);
        asm volatile("" : "+v"(fac), "+v"(fac2), "+v"(e), "+v"(add));    // here, not behind the sums
        // two chains per unit (rows 2k and 2k + 1), four for a single unit, so that no
        // multiply-add waits for the one before it
        constexpr int MC = UP == 1 ? 2 : 1;
        constexpr int NU = UP > 4 ? 8 : 4;
        float a[MC][2][NU];
#pragma unroll
        for (int k = 0; k < MC; ++k)
#pragma unroll
            for (int j = 0; j < NU; ++j) a[k][0][j] = a[k][1][j] = 0.0f;
#pragma unroll
        for (int m = 0; m < KM; ++m)
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int j = 0; j < UP; ++j)
                    a[m % MC][r][j] = __builtin_fmaf(w[m][r][j], r ? x[m].y : x[m].x, a[m % MC][r][j]);
        float p[NU];
#pragma unroll
        for (int j = 0; j < NU; ++j) p[j] = MC == 2 ? (a[0][0][j] + a[0][1][j]) + (a[MC - 1][0][j] + a[MC - 1][1][j]) : a[0][0][j] + a[0][1][j];
        float sum;
        if constexpr (UP > 4) {
            float h[4], r[2];
#pragma unroll
            for (int j = 0; j < 4; ++j) h[j] = (b2 ? p[j + 4] : p[j]) + dpp(b2 ? p[j] : p[j + 4], HalfMirror());
#pragma unroll
            for (int j = 0; j < 2; ++j) r[j] = (b0 ? h[2 * j + 1] : h[2 * j]) + dpp(b0 ? h[2 * j] : h[2 * j + 1], Xor1());
            sum = (b1 ? r[1] : r[0]) + dpp(b1 ? r[0] : r[1], Xor2());
        } else if constexpr (UP > 2) {
            const float r0 = (b2 ? p[2] : p[0]) + dpp(b2 ? p[0] : p[2], HalfMirror());
            const float r1 = (b2 ? p[3] : p[1]) + dpp(b2 ? p[1] : p[3], HalfMirror());
            sum = (b0 ? r1 : r0) + dpp(b0 ? r0 : r1, Xor1());
        } else if constexpr (UP == 2) {
            sum = (b2 ? p[1] : p[0]) + dpp(b2 ? p[0] : p[1], HalfMirror());
            sum += dpp(sum, Xor1());
        } else {
            sum = p[0] + dpp(p[0], HalfMirror());
            sum += dpp(sum, Xor1());
        }
        if constexpr (UP <= 4) sum += dpp(sum, Xor2());
        sum += dpp(sum, Ror8());
        // (of the two products the chain's, dc f, is the one that is not rounded)
        const float dh = sum + add, dc = __builtin_fmaf(dc_next, f_next, dh * e);
        if constexpr (UP > 4) {
            const float v0 = dc * fac, v1 = (q ? dh : dc) * fac2;
            if (live) {
                float *o = dbuf[cur] + 2 * q * H + u, *m = dn + (i64)t * G + 2 * q * H + u;
                o[0] = v0;
                o[H] = v1;
                m[0] = v0;
                m[H] = v1;
            }
        } else {
            const float val = (q == 3 ? dh : dc) * fac;
            if (live) {
                dbuf[cur][q * H + u] = val;
                dn[(i64)t * G + q * H + u] = val;
            }
        }
        dc_next = dc;
        f_next = gf;
        lds_barrier();
        cur ^= 1;
    };

#pragma unroll
    for (int k = 0; k < kRing; ++k) load_step(T - 1 - k, ring[k]);
    __builtin_amdgcn_s_waitcnt(0);
    lds_barrier();
    const int full = T / kRing * kRing;        // steps T-1 .. T-full
    for (int t0 = T - 1; t0 > T - 1 - full; t0 -= kRing) {
#pragma unroll
        for (int k = 0; k < kRing; ++k) {
            const int t = t0 - k;
            step(t, ring[k], ring[(k + 1) % kRing][4]);     // c_{-1} read zero
            load_step(t - kRing, ring[k]);
        }
    }
#pragma unroll
    for (int k = 0; k + 1 < kRing; ++k)
        if (k < T - full) step(T - 1 - full - k, ring[k], ring[k + 1][4]);
}

template <int KM, int UP>
void launch(const float *gates, const float *c, const float *W_hh, const float *dh_out, const float *dh_last, i64 N,
            i64 T, int H, float *delta, hipStream_t stream)
{
    const int threads = (int)ceil_div(16 * ceil_div(H, UP), kWave) * kWave;
    if (dh_out)
        lstm_bptt_kernel<KM, UP, true><<<(unsigned)N, threads, 0, stream>>>(gates, c, W_hh, dh_out, dh_last, T, H,
                                                                            delta);
    else
        lstm_bptt_kernel<KM, UP, false><<<(unsigned)N, threads, 0, stream>>>(gates, c, W_hh, dh_out, dh_last, T, H,
                                                                             delta);
}

// KM = ceil(H / 8).  At most a workgroup per CU: units spread over eight waves
// (UP = ceil(H / 32)).  More samples than CUs: the CUs' VALUs are shared, so
// the fewest instructions count: four waves (UP = ceil(H / 16), up to six, as
// far as the weights leave a wave its registers).  Measured (us, eight waves /
// four): 100 samples, T = 128, H = 48 50 / 54; 500 samples, T = 50, H = 64
// 42 / 40; 300 samples, T = 128, H = 80 140 / 101.
template <int KM>
void launch_rows(bool full, const float *gates, const float *c, const float *W_hh, const float *dh_out,
                 const float *dh_last, i64 N, i64 T, int H, float *delta, hipStream_t stream)
{
    constexpr int few = (KM + 3) / 4, most = (KM + 1) / 2;
    if (full && most <= 6) launch<KM, (most <= 6 ? most : few)>(gates, c, W_hh, dh_out, dh_last, N, T, H, delta, stream);
    else launch<KM, few>(gates, c, W_hh, dh_out, dh_last, N, T, H, delta, stream);
}

}  // namespace
}  // namespace dpg

using namespace dpg;

extern "C" dp_status dp_lstm_backward(const float *gates, const float *c, const float *W_hh, const float *dh_out,
                                      const float *dh_last, int64_t N, int64_t T, int64_t H, float *delta,
                                      int32_t *status, hipStream_t stream)
{
    (void)status;
    DPG_REQUIRE(N >= 0 && T >= 0 && H >= 1, DP_EINVAL);
    DPG_REQUIRE(H <= kMaxH, DP_EUNSUPPORTED);
    DPG_REQUIRE(N < (i64(1) << 31) && T < (i64(1) << 40), DP_EINVAL);
    DPG_REQUIRE(T * 4 * H * 4 < (i64(1) << 31), DP_EUNSUPPORTED);   // 32-bit offsets within a sample
    DPG_REQUIRE(N * T == 0 || (gates != nullptr && c != nullptr && W_hh != nullptr && delta != nullptr),
                DP_EINVAL);
    DPG_REQUIRE(aligned(gates, 4) && aligned(c, 4) && aligned(delta, 4), DP_EINVAL);
    if (N == 0 || T == 0) return DP_OK;
    const int h = (int)H;
    const bool full = N > 256;             // more samples than CUs
    switch ((h + 7) / 8) {
    case 1: launch_rows<1>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 2: launch_rows<2>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 3: launch_rows<3>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 4: launch_rows<4>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 5: launch_rows<5>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 6: launch_rows<6>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 7: launch_rows<7>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 8: launch_rows<8>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 9: launch_rows<9>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 10: launch_rows<10>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 11: launch_rows<11>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 12: launch_rows<12>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 13: launch_rows<13>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 14: launch_rows<14>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    case 15: launch_rows<15>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    default: launch_rows<16>(full, gates, c, W_hh, dh_out, dh_last, N, T, h, delta, stream); break;
    }
    return launch_status();
}
