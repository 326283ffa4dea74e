// Linear layer: per-sample gradients and the fused clipped sum.
//
// Per-sample gradient of y_t = W x_t + b for sample n (appendix "Vectorized
// Computation"; extra dimensions summed):
//   gW_n = s * B_n^T A_n   (d_out x d_in, K = T positions),  gb_n = s * sum_t B_n,t
// T = 1 is a rank-one outer product (linear_outer.hpp).  T > 1 is a real per-sample GEMM on
// MFMA with the squared-norm partials taken from the accumulators in the
// epilogue.
//
// Fused clipped sum: sum_n c_n gW_n = s * B^T diag(c) A, one GEMM whose K runs
// over all N*T rows, split over workgroups; partial tiles go to the workspace
// and a second kernel adds them in split order (no atomics).
#include "common.hpp"
#include "mfma_tile.hpp"
#include "linear_bf16.hpp"
#include "grad_sample_bf16.hpp"
#include "linear_outer.hpp"
#include "ps_split.hpp"

namespace dpg {
namespace {

constexpr int kThreads = 256;
constexpr int kBM = 64, kBN = 64, kBK = 32;

// T = 1: the rank-one outer product (linear_outer.hpp), block = (sample, rows)
template <typename T, bool VEC>
__global__ __launch_bounds__(kThreads) void outer_kernel(const T *__restrict__ A, const T *__restrict__ B, i64 din,
                                                         i64 dout, int rows, int bps, float scale,
                                                         float *__restrict__ gW, float *__restrict__ gb,
                                                         float *__restrict__ sqnorm)
{
    louter::outer_block<T, VEC>(A, B, din, dout, rows, blockIdx.x / bps, (int)(blockIdx.x % bps), scale, gW, gb,
                                sqnorm);
}

// ---------------------------------------------------------------------------
// T > 1: per-sample GEMM on MFMA.  Block = (sample n, 64 x 64 tile of gW_n).
// The kernel of layers whose rows are shorter than the 16-byte loads of
// ps_split.hip (fewer than four fp32 or eight bf16 features on a side): element loads,
// fp32 MFMA.  MFMA rows run over j (d_in, the contiguous index of gW),
// columns over i (d_out).  Both operands are staged K-major exactly as they
// lie in memory ([t][feature]); the next chunk of positions is loaded into
// registers while the current one is multiplied.
// ---------------------------------------------------------------------------
constexpr int kPM = 64, kPN = 64, kPK = 32;

template <typename T>
__global__ __launch_bounds__(kThreads) void ps_gemm_kernel(
    const T *__restrict__ A, const T *__restrict__ B, i64 Tn, i64 din, i64 dout, int tiles_j,
    int tiles, float scale, float *__restrict__ gW, float *__restrict__ gb,
    float *__restrict__ partial)
{
    __shared__ float As[kPK * kPM];   // [t][j]
    __shared__ float Bs[kPK * kPN];   // [t][i]
    __shared__ float red[16];
    const i64 bsw = xcd_swizzle(blockIdx.x, gridDim.x);
    const i64 n = bsw / tiles;
    const int tile = (int)(bsw % tiles);
    const int ti = tile / tiles_j, tj = tile % tiles_j;
    const i64 j0 = (i64)tj * kPM, i0 = (i64)ti * kPN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
    const T *An = A + n * Tn * din;
    const T *Bn = B + n * Tn * dout;
    const bool do_bias = gb != nullptr && tj == 0;

    constexpr int NG = kPK * kPM / kThreads;
    static_assert(kPM == kPN && NG * kThreads == kPK * kPM, "staging map");
    float ra[NG], rb[NG];
    auto load = [&](i64 t0) {
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            const int g = tid + kThreads * q;
            const int r = g / kPM, c = g % kPM;
            const i64 t = t0 + r;
            const bool okA = t < Tn && j0 + c < din;
            const bool okB = t < Tn && i0 + c < dout;
            ra[q] = okA ? load_elem<T>(An, t * din + j0 + c) : 0.0f;
            rb[q] = okB ? load_elem<T>(Bn, t * dout + i0 + c) : 0.0f;
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            As[tid + kThreads * q] = ra[q];
            Bs[tid + kThreads * q] = rb[q];
        }
    };

    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    float bias_acc = 0.0f;
    load(0);
    for (i64 t0 = 0; t0 < Tn; t0 += kPK) {
        __syncthreads();   // previous chunk consumed
        store();
        __syncthreads();
        if (t0 + kPK < Tn) load(t0 + kPK);
        const int li = lane & 31, lk = lane >> 5;
#pragma unroll
        for (int kk = 0; kk < kPK; kk += 2) {
            const float a = As[(kk + lk) * kPM + wm + li];
            const float b = Bs[(kk + lk) * kPN + wn + li];
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
        }
        if (do_bias && tid < kPN) {
#pragma unroll 8
            for (int kk = 0; kk < kPK; ++kk) bias_acc += Bs[kk * kPN + tid];
        }
    }

    // acc[r] holds gW[i][j], j = j0 + wm + 8 (r / 4) + 4 (lane / 32) + r % 4, i = i0 + wn + lane % 32
    float sq = 0.0f;
    const i64 i = i0 + wn + (lane & 31);
    if (i < dout) {
        float *G = gW + n * dout * din + i * din;
#pragma unroll
        for (int rb4 = 0; rb4 < 4; ++rb4) {
            const i64 j = j0 + wm + 8 * rb4 + 4 * (lane >> 5);
            const float g0 = scale * acc[4 * rb4 + 0], g1 = scale * acc[4 * rb4 + 1];
            const float g2 = scale * acc[4 * rb4 + 2], g3 = scale * acc[4 * rb4 + 3];
            if (j + 0 < din) { G[j + 0] = g0; sq += g0 * g0; }
            if (j + 1 < din) { G[j + 1] = g1; sq += g1 * g1; }
            if (j + 2 < din) { G[j + 2] = g2; sq += g2 * g2; }
            if (j + 3 < din) { G[j + 3] = g3; sq += g3 * g3; }
        }
    }
    if (do_bias && tid < kPN && i0 + tid < dout) {
        const float g = scale * bias_acc;
        gb[n * dout + i0 + tid] = g;
        sq += g * g;
    }
    sq = block_sum(sq, red);
    if (partial && tid == 0) partial[n * tiles + tile] = sq;
}

// the fp32 layers that dp_grad_sample_many groups into one launch
bool grouped_shape_ok(const void *A, const void *B, const float *gW, i64 T, i64 din, i64 dout)
{
    return T >= 16 && T % 16 == 0 && din % 4 == 0 && dout % 4 == 0 && aligned(A, 16) && aligned(B, 16) &&
           aligned(gW, 16) && T * (din > dout ? din : dout) < (i64(1) << 31);
}

// ---------------------------------------------------------------------------
// Fused clipped sum: block = (split, tile).  Rows of the flattened [N*T]
// operands are scaled by s * c_n as they are staged.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kThreads) void clipsum_gemm_kernel(
    const T *__restrict__ A, const T *__restrict__ B, i64 Tn, i64 rows_total, i64 rows_per_split,
    i64 din, i64 dout, int tiles_n, int tiles, float scale, const float *__restrict__ norm,
    float C, float *__restrict__ outW, float *__restrict__ outb, i64 split_strideW,
    i64 split_strideb)
{
    __shared__ float As[kBK * kBM];
    __shared__ float Bs[kBK * kBN];
    __shared__ float rs[kBK];
    const i64 bsw = xcd_swizzle(blockIdx.x, gridDim.x);
    const int split = (int)(bsw / tiles);
    const int tile = (int)(bsw % tiles);
    const int tm = tile / tiles_n, tn = tile % tiles_n;
    const i64 m0 = (i64)tm * kBM, n0 = (i64)tn * kBN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * (kBM / 2), wn = (wave & 1) * (kBN / 2);
    const i64 r0 = (i64)split * rows_per_split;
    const i64 r1 = r0 + rows_per_split < rows_total ? r0 + rows_per_split : rows_total;
    const bool do_bias = outb != nullptr && tn == 0;

    MfmaTile<kBM, kBN> t;
    t.zero();
    float bias_acc = 0.0f;

    for (i64 k0 = r0; k0 < r1; k0 += kBK) {
        if (tid < kBK) {
            const i64 k = k0 + tid;
            rs[tid] = k < r1 ? scale * clip_factor(norm[k / Tn], C) : 0.0f;
        }
        __syncthreads();
        for (int e = tid; e < kBK * kBM; e += kThreads) {
            const int kk = e / kBM, ii = e % kBM;
            const i64 k = k0 + kk, i = m0 + ii;
            As[e] = (k < r1 && i < dout) ? rs[kk] * load_elem<T>(B, k * dout + i) : 0.0f;
        }
        for (int e = tid; e < kBK * kBN; e += kThreads) {
            const int kk = e / kBN, jj = e % kBN;
            const i64 k = k0 + kk, j = n0 + jj;
            Bs[e] = (k < r1 && j < din) ? load_elem<T>(A, k * din + j) : 0.0f;
        }
        __syncthreads();
        t.template mma<kBK>(As, kBM, Bs, kBN, wm, wn, lane);
        if (do_bias && tid < kBM) {
#pragma unroll 8
            for (int kk = 0; kk < kBK; ++kk) bias_acc += As[kk * kBM + tid];
        }
        __syncthreads();
    }

    float *O = outW + (i64)split * split_strideW;
    t.for_each(wm, wn, lane, [&](int r, int c, float v) {
        const i64 i = m0 + r, j = n0 + c;
        if (i < dout && j < din) O[i * din + j] = v;
    });
    if (do_bias && tid < kBM && m0 + tid < dout) outb[(i64)split * split_strideb + m0 + tid] = bias_acc;
}

// out[e] = sum_s part[s][e], s ascending.
__global__ void split_sum_kernel(const float *__restrict__ part, int splits, i64 count,
                                 float *__restrict__ out)
{
    const i64 e = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= count) return;
    float s = 0.0f;
    s = ordered_sum(part + e, count, splits);
    out[e] = s;
}

struct ClipSplit {
    int tiles_n, tiles, splits;
    i64 rows_per_split;
};

ClipSplit clip_split(i64 N, i64 T, i64 din, i64 dout)
{
    ClipSplit s;
    s.tiles_n = (int)ceil_div(din, kBN);
    s.tiles = (int)ceil_div(dout, kBM) * s.tiles_n;
    const i64 rows = N * T;
    const i64 chunks = ceil_div(rows, kBK);
    i64 want = ceil_div(1024, s.tiles);           // aim for ~1024 workgroups
    if (want > chunks) want = chunks;
    if (want > 256) want = 256;
    if (want < 1) want = 1;
    s.rows_per_split = ceil_div(chunks, want) * kBK;
    s.splits = (int)(rows > 0 ? ceil_div(rows, s.rows_per_split) : 1);
    return s;
}

}  // namespace

bool fp32_staged_ok(const void *A, const void *B, const void *gW, i64 N, i64 T, i64 din, i64 dout)
{
    return grouped_shape_ok(A, B, (const float *)gW, T, din, dout) && ps_split_ok(DP_F32, T, din, dout) &&
           N < (i64(1) << 40) && N * ceil_div(din, kPM) * ceil_div(dout, kPN) < (i64(1) << 26);
}

dp_status check_linear(const void *A, const void *B, dp_dtype dt, i64 N, i64 T, i64 din, i64 dout)
{
    DPG_REQUIRE(dtype_ok(dt), DP_EDTYPE);
    DPG_REQUIRE(N >= 0 && T >= 0 && din >= 1 && dout >= 1, DP_EINVAL);
    DPG_REQUIRE(N * T == 0 || (A != nullptr && B != nullptr), DP_EINVAL);
    DPG_REQUIRE(N < (i64(1) << 40) && T < (i64(1) << 40), DP_EINVAL);
    return DP_OK;
}

}  // namespace dpg

using namespace dpg;

extern "C" size_t dp_grad_sample_linear_workspace_bytes(int64_t N, int64_t T, int64_t d_in,
                                                        int64_t d_out, dp_dtype dt)
{
    if (N <= 0 || T <= 1 || d_in <= 0 || d_out <= 0) return 0;
    // squared-norm partials of whichever path runs: one per 64x64 tile (fp32
    // MFMA; more than the 128x128 tiles of the bf16 kernel), or one per wave
    // and 128x128 tile (staged bf16 kernel)
    i64 parts = ceil_div(d_in, kPM) * ceil_div(d_out, kPN);
    if (dt == DP_BF16 && bf16_staged_parts(d_in, d_out) > parts) parts = bf16_staged_parts(d_in, d_out);
    return (size_t)(N * parts) * sizeof(float);
}

extern "C" dp_status dp_grad_sample_linear(const void *A, const void *B, dp_dtype dt, int64_t N,
                                           int64_t T, int64_t d_in, int64_t d_out, float scale,
                                           float *gW, float *gb, float *sqnorm, int32_t *status,
                                           void *ws, size_t ws_bytes, hipStream_t stream)
{
    (void)status;
    dp_status st = check_linear(A, B, dt, N, T, d_in, d_out);
    if (st != DP_OK) return st;
    DPG_REQUIRE(N == 0 || gW != nullptr, DP_EINVAL);
    const size_t need = dp_grad_sample_linear_workspace_bytes(N, T, d_in, d_out, dt);
    DPG_REQUIRE(ws_bytes >= need && (need == 0 || ws != nullptr), DP_EINVAL);
    if (N == 0) return DP_OK;

    if (T == 0) {
        // empty sum over positions: every gradient and norm is zero
        zero_fill(gW, N * d_out * d_in, stream);
        zero_fill(gb, N * d_out, stream);
        zero_fill(sqnorm, N, stream);
        return launch_status();
    }
    if (T == 1) {
        const louter::OuterPlan op = louter::outer_plan(d_in, d_out);
        const int rows = op.rows, bps = op.bps;
        const dim3 grid((unsigned)(N * bps));
        const bool vec = (d_in % 4) == 0 && aligned(A, dt == DP_F32 ? 16 : 8) && aligned(gW, 16);
        if (dt == DP_F32) {
            if (vec)
                outer_kernel<float, true><<<grid, kThreads, 0, stream>>>(
                    (const float *)A, (const float *)B, d_in, d_out, rows, bps, scale, gW, gb, sqnorm);
            else
                outer_kernel<float, false><<<grid, kThreads, 0, stream>>>(
                    (const float *)A, (const float *)B, d_in, d_out, rows, bps, scale, gW, gb, sqnorm);
        } else {
            if (vec)
                outer_kernel<uint16_t, true><<<grid, kThreads, 0, stream>>>(
                    (const uint16_t *)A, (const uint16_t *)B, d_in, d_out, rows, bps, scale, gW, gb, sqnorm);
            else
                outer_kernel<uint16_t, false><<<grid, kThreads, 0, stream>>>(
                    (const uint16_t *)A, (const uint16_t *)B, d_in, d_out, rows, bps, scale, gW, gb, sqnorm);
        }
        return launch_status();
    }

    float *partial = sqnorm ? (float *)ws : nullptr;
    if (dt == DP_BF16 && bf16_staged_ok(A, B, gW, N, T, d_in, d_out)) {
        bf16_grad_sample_staged(A, B, N, T, d_in, d_out, scale, gW, gb, partial, stream);
        if (sqnorm)
            sum_partials(partial, N, bf16_staged_parts(d_in, d_out), sqnorm, stream);
        return launch_status();
    }
    if (dt == DP_BF16 && bf16_path_ok(A, B, gW, T, d_in, d_out)) {
        bf16_grad_sample(A, B, N, T, d_in, d_out, scale, gW, gb, partial, stream);
        if (sqnorm)
            sum_partials(partial, N, bf16_tiles(d_in, d_out), sqnorm, stream);
        return launch_status();
    }
    if (ps_split_ok(dt, T, d_in, d_out)) {
        ps_split_grad({A, B, T, d_in, d_out, scale, gW, gb, sqnorm, partial}, dt, N, stream);
        return launch_status();
    }
    // rows too short for 16-byte loads
    const int tiles_j = (int)ceil_div(d_in, kPM);
    const int tiles = (int)ceil_div(d_out, kPN) * tiles_j;
    const dim3 grid((unsigned)(N * tiles));
    if (dt == DP_F32)
        ps_gemm_kernel<float><<<grid, kThreads, 0, stream>>>(
            (const float *)A, (const float *)B, T, d_in, d_out, tiles_j, tiles, scale, gW, gb, partial);
    else
        ps_gemm_kernel<uint16_t><<<grid, kThreads, 0, stream>>>(
            (const uint16_t *)A, (const uint16_t *)B, T, d_in, d_out, tiles_j, tiles, scale, gW, gb, partial);
    if (sqnorm)
        sum_partials(partial, N, tiles, sqnorm, stream);
    return launch_status();
}

extern "C" size_t dp_clip_accumulate_linear_workspace_bytes(int64_t N, int64_t T, int64_t d_in,
                                                            int64_t d_out, dp_dtype dt)
{
    if (N <= 0 || T <= 0 || d_in <= 0 || d_out <= 0) return 0;
    const ClipSplit s = clip_split(N, T, d_in, d_out);
    size_t need = s.splits > 1 ? (size_t)s.splits * (size_t)(d_out * d_in + d_out) * sizeof(float) : 0;
    if (dt == DP_BF16) {
        const size_t b = bf16_clip_workspace(N, T, d_in, d_out);
        if (b > need) need = b;
    }
    return need;
}

extern "C" dp_status dp_clip_accumulate_linear(const void *A, const void *B, dp_dtype dt,
                                               int64_t N, int64_t T, int64_t d_in, int64_t d_out,
                                               float scale, const float *norm, float C,
                                               float *sumW, float *sumb, int32_t *status,
                                               void *ws, size_t ws_bytes, hipStream_t stream)
{
    (void)status;
    dp_status st = check_linear(A, B, dt, N, T, d_in, d_out);
    if (st != DP_OK) return st;
    DPG_REQUIRE(sumW != nullptr && (N == 0 || norm != nullptr), DP_EINVAL);
    DPG_REQUIRE(C > 0.0f, DP_EINVAL);
    const size_t need = dp_clip_accumulate_linear_workspace_bytes(N, T, d_in, d_out, dt);
    DPG_REQUIRE(ws_bytes >= need && (need == 0 || ws != nullptr), DP_EINVAL);
    if (N * T == 0) {
        zero_fill(sumW, d_out * d_in, stream);
        zero_fill(sumb, d_out, stream);
        return launch_status();
    }
    if (dt == DP_BF16 && bf16_path_ok(A, B, sumW, T, d_in, d_out) && (sumb == nullptr || aligned(sumb, 4))) {
        bf16_clip_accumulate(A, B, N, T, d_in, d_out, scale, norm, C, sumW, sumb, ws, stream);
        return launch_status();
    }
    const ClipSplit s = clip_split(N, T, d_in, d_out);
    const i64 cw = d_out * d_in;
    float *pw = s.splits > 1 ? (float *)ws : sumW;
    float *pb = sumb ? (s.splits > 1 ? (float *)ws + (i64)s.splits * cw : sumb) : nullptr;
    const dim3 grid((unsigned)(s.splits * s.tiles));
    if (dt == DP_F32)
        clipsum_gemm_kernel<float><<<grid, kThreads, 0, stream>>>(
            (const float *)A, (const float *)B, T, N * T, s.rows_per_split, d_in, d_out, s.tiles_n,
            s.tiles, scale, norm, C, pw, pb, cw, d_out);
    else
        clipsum_gemm_kernel<uint16_t><<<grid, kThreads, 0, stream>>>(
            (const uint16_t *)A, (const uint16_t *)B, T, N * T, s.rows_per_split, d_in, d_out,
            s.tiles_n, s.tiles, scale, norm, C, pw, pb, cw, d_out);
    if (s.splits > 1) {
        split_sum_kernel<<<(unsigned)ceil_div(cw, 256), 256, 0, stream>>>(pw, s.splits, cw, sumW);
        if (sumb)
            split_sum_kernel<<<(unsigned)ceil_div(d_out, 256), 256, 0, stream>>>(pb, s.splits, d_out, sumb);
    }
    return launch_status();
}
