// GroupNorm / InstanceNorm affine per-sample gradients.  Both normalize
// [N][C][spatial] inputs within each sample (over a group of channels, or
// over one channel) and then apply a per-channel affine y = gamma[c] * xhat
// + beta[c]; neither mixes samples, so their per-sample gradients exist
// (unlike BatchNorm's).  With the normalized input xhat given:
//   ggamma_n[c] = s * sum_p B[n][c][p] * xhat[n][c][p]
//   gbeta_n[c]  = s * sum_p B[n][c][p]
// over the channel's P spatial positions, which are contiguous in memory.
// A wave reduces one channel at a time (lanes over the positions, loads of four
// elements at any alignment, up to four of each operand in flight, then a fixed
// tree), or, for planes of at most 64
// positions, four channels at a time on 16 lanes each; the sums are
// deterministic.  A workgroup takes 16 channels of one sample, and the
// sample's squared norm is added over its channel blocks in block order.
// Bound by the reads: 512 x 64 x 1024 fp32 268 MB in 45 us with the launch that adds
// the norm's blocks (6.0 TB/s; 56 us with one pair of loads in flight), 100 x
// 30 x 777 fp32 11 us (20 with single elements).
#include "common.hpp"

namespace dpg {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kChanPerBlock = 16;

// Four consecutive elements at their natural alignment only; NT: past the caches.
template <typename T, bool NT>
__device__ __forceinline__ float4 ld4(const T *p)
{
    typedef T v4_t __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    const v4_t *q = reinterpret_cast<const v4_t *>(p);
    const v4_t v = NT ? __builtin_nontemporal_load(q) : *q;
    if constexpr (sizeof(T) == 4) return make_float4(v[0], v[1], v[2], v[3]);
    else return make_float4(bf16_to_f32(v[0]), bf16_to_f32(v[1]), bf16_to_f32(v[2]), bf16_to_f32(v[3]));
}

// sum over the LPC lanes of a segment (a fixed butterfly; every lane of the
// segment ends with the sum)
template <int LPC>
__device__ __forceinline__ float seg_sum(float v)
{
    if constexpr (LPC == 64) return wave_sum(v);
#pragma unroll
    for (int o = LPC / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// LPC: lanes per channel (64, or 16 for planes of at most 64 positions);
// kLoads: loads of four elements of each operand in flight per lane (0: single elements)
template <typename T, int LPC, int kLoads, bool NT>
__global__ __launch_bounds__(kThreads) void gn_affine_kernel(const T *__restrict__ xh, const T *__restrict__ B,
                                                             i64 C, i64 P, int cblocks, float scale,
                                                             float *__restrict__ gg, float *__restrict__ gbt,
                                                             float *__restrict__ sqout, int direct)
{
    __shared__ float red[kWaves];
    const i64 n = blockIdx.x / cblocks;
    const int cb = (int)(blockIdx.x % cblocks);
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    constexpr int SEGS = 64 / LPC;                 // channels a wave takes at once
    const int seg = lane / LPC, sl = lane % LPC;
    const i64 P4 = P & ~i64(3);
    float sq = 0.0f;
    for (int k = wave * SEGS; k < kChanPerBlock; k += kWaves * SEGS) {
        const i64 c = (i64)cb * kChanPerBlock + k + seg;
        const bool live = c < C;
        const T *x = xh + (n * C + (live ? c : 0)) * P;
        const T *b = B + (n * C + (live ? c : 0)) * P;
        float ag = 0.0f, ab = 0.0f;
        if (live && kLoads == 0) {
            for (i64 p = sl; p < P; p += LPC) {
                const float bv = load_elem<T>(b, p);
                ag += bv * load_elem<T>(x, p);
                ab += bv;
            }
        }
        if (live && kLoads > 0) {
            constexpr int L = kLoads > 0 ? kLoads : 1, kStep = 4 * LPC * L;
            const auto add = [&](const float4 &b4, const float4 &x4) {
                ag += (b4.x * x4.x + b4.y * x4.y) + (b4.z * x4.z + b4.w * x4.w);
                ab += (b4.x + b4.y) + (b4.z + b4.w);
            };
            float4 bv[L], xv[L];
            i64 p0 = 4 * sl;
            // (one load per step: each lane's own bound)
            for (; L == 1 ? p0 < P4 : p0 + kStep <= P4 + 4 * sl; p0 += kStep) {
#pragma unroll
                for (int j = 0; j < L; ++j) {
                    bv[j] = ld4<T, NT>(b + p0 + 4 * LPC * j);
                    xv[j] = ld4<T, NT>(x + p0 + 4 * LPC * j);
                }
#pragma unroll
                for (int j = 0; j < L; ++j) add(bv[j], xv[j]);
            }
            // what is left of a step: only the lanes and loads inside the plane (past the caches, a load
            // repeated to fill the step is read from memory again)
            if (L > 1 && p0 < P4) {
#pragma unroll
                for (int j = 0; j < L; ++j) {
                    bv[j] = xv[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if (p0 + 4 * LPC * j < P4) {
                        bv[j] = ld4<T, NT>(b + p0 + 4 * LPC * j);
                        xv[j] = ld4<T, NT>(x + p0 + 4 * LPC * j);
                    }
                }
#pragma unroll
                for (int j = 0; j < L; ++j) add(bv[j], xv[j]);
            }
            if (P4 + sl < P) {
                const float bv = load_elem<T>(b, P4 + sl);
                ag += bv * load_elem<T>(x, P4 + sl);
                ab += bv;
            }
        }
        ag = seg_sum<LPC>(ag);
        ab = seg_sum<LPC>(ab);
        if (live && sl == 0) {
            const float g = scale * ag, e = scale * ab;
            gg[n * C + c] = g;
            if (gbt) gbt[n * C + c] = e;
            sq += g * g + (gbt ? e * e : 0.0f);
        }
    }
    sq = wave_sum(sq);                             // the segments' shares (one lane each), in a fixed order
    if (lane == 0) red[wave] = sq;
    __syncthreads();
    if (threadIdx.x == 0 && sqout) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) t += red[w];
        if (direct) sqout[n] = t;
        else sqout[n * cblocks + cb] = t;
    }
}

template <typename T>
void launch_gn(dim3 grid, const void *xh, const void *B, i64 C, i64 P, int cblocks, float scale,
               float *gg, float *gbt, float *sqout, int direct, hipStream_t stream)
{
    const T *x = (const T *)xh, *b = (const T *)B;
    const auto go = [&](auto kernel) {
        kernel<<<grid, kThreads, 0, stream>>>(x, b, C, P, cblocks, scale, gg, gbt, sqout, direct);
    };
    // Inputs of whole cache lines per channel, too large to be still cached, go
    // past the caches.  us with / without, the same inputs again and four sets in turn:
    // 512 x 64 x 1024 fp32 (268 MB) 43.9 / 42.0 and 45.4 / 51.5, 384 x 64 x 1024 (201 MB)
    // 32.9 / 32.3 and 34.3 / 39.1, 108 x 67 x 3328 (193 MB) 36.8 / 33.2 and 38.9 / 43.2,
    // 256 x 64 x 1024 (134 MB) 24.0 / 23.1 and 24.6 / 28.0, 200 x 64 x 1056 (108 MB) 22.1 /
    // 20.1 and 23.3 / 25.9; smaller inputs stay cached either way: 128 x 64 x 1024
    // (67 MB) 14.1 / 13.5 and 14.1 / 13.9.  Channels that share lines never (300 x 59
    // x 989 bf16: 19 against 15).
    const bool lines = P * sizeof(T) % 128 == 0 && aligned(xh, 128) && aligned(B, 128);
    const double bytes = 2.0 * (double)(grid.x / cblocks) * (double)C * (double)P * sizeof(T);
    if (P <= 64 && P % 4 != 0) go(gn_affine_kernel<T, 16, 0, false>);
    else if (P <= 64) go(gn_affine_kernel<T, 16, 1, false>);
    else if (P <= 128 && P % 4 != 0) go(gn_affine_kernel<T, 64, 0, false>);   // 400 x 200 x 90 fp32 19.4 us against 20.1
    else if (P < 260) go(gn_affine_kernel<T, 64, 1, false>);
    else if (P < 516) go(gn_affine_kernel<T, 64, 2, false>);
    else if (lines && bytes >= 96e6) go(gn_affine_kernel<T, 64, 4, true>);
    else go(gn_affine_kernel<T, 64, 4, false>);
}

}  // namespace
}  // namespace dpg

using namespace dpg;

extern "C" size_t dp_grad_sample_groupnorm_workspace_bytes(int64_t N, int64_t C, int64_t P)
{
    if (N <= 0 || C <= 0 || P < 0) return 0;
    const i64 cblocks = ceil_div(C, (i64)kChanPerBlock);
    return cblocks > 1 ? (size_t)(N * cblocks) * sizeof(float) : 0;
}

extern "C" dp_status dp_grad_sample_groupnorm(const void *xhat, const void *B, dp_dtype dt, int64_t N, int64_t C,
                                              int64_t P, float scale, float *ggamma, float *gbeta, float *sqnorm,
                                              int32_t *status, void *ws, size_t ws_bytes, hipStream_t stream)
{
    (void)status;
    DPG_REQUIRE(dtype_ok(dt), DP_EDTYPE);
    DPG_REQUIRE(N >= 0 && C >= 1 && P >= 0, DP_EINVAL);
    DPG_REQUIRE(N * C < (i64(1) << 40) && C * P < (i64(1) << 40), DP_EINVAL);
    DPG_REQUIRE(N == 0 || ggamma != nullptr, DP_EINVAL);
    DPG_REQUIRE(N == 0 || P == 0 || (xhat != nullptr && B != nullptr), DP_EINVAL);
    const size_t need = dp_grad_sample_groupnorm_workspace_bytes(N, C, P);
    DPG_REQUIRE(ws_bytes >= need && (need == 0 || ws != nullptr), DP_EINVAL);
    if (N == 0) return DP_OK;
    const int cblocks = (int)ceil_div(C, (i64)kChanPerBlock);
    const int direct = cblocks == 1;
    float *sqout = sqnorm ? (direct ? sqnorm : (float *)ws) : nullptr;
    const dim3 grid((unsigned)(N * cblocks));
    const bool bf = dt == DP_BF16;
    if (bf) launch_gn<uint16_t>(grid, xhat, B, C, P, cblocks, scale, ggamma, gbeta, sqout, direct, stream);
    else launch_gn<float>(grid, xhat, B, C, P, cblocks, scale, ggamma, gbeta, sqout, direct, stream);
    if (sqnorm && !direct) sum_partials((const float *)ws, N, cblocks, sqnorm, stream);
    return launch_status();
}
