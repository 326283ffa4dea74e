// Per-sample gradients of a Linear layer over a sequence (appendix
// "Vectorized Computation", extra dimension summed):
//   gW_n[i][j] = s * sum_t B_n[t][i] * A_n[t][j],   gb_n[i] = s * sum_t B_n[t][i]
// for any T and alignment, fp32 or bf16 inputs, on v_mfma_f32_32x32x16_bf16.
// fp32 operands are split into three bf16 parts (split_bf16.hpp: six products,
// fp32 results); bf16 operands go in as they are.
//
// Block = (sample, tile of gW_n).  Stages of consecutive positions are loaded
// into registers two stages ahead, R rows x 16 bytes per thread, then split
// and written to LDS with the positions contiguous ([feature][t], one plane
// per part; packing two positions of a feature into a word costs the same as
// packing two features), so that an MFMA operand (eight positions of one
// feature per lane) is one ds_read_b128.
//
// What bounds it: at the LSTM's layer (fp32, 64 samples, T = 256, 100 -> 400:
// 43 MB and, in six products, 7.9 GFLOP of bf16 MFMA) about half of the call
// is fixed (two launches, the first loads, the last stores) and a stage costs
// its MFMAs plus about half of its split (the conversions and LDS writes
// that the interleaving does not hide).  19.9-21.2 us against 24.3 with fp32
// MFMA, and half the error against 64 bits (1.1e-7 against 2.1e-7); a bf16
// layer of odd sizes (48 samples, T = 75, 300 -> 514, 36 MB) 20.2 us against
// 42.0 with element loads and fp32 MFMA; 768 x 768 over T = 512 (16 samples,
// fp32) 69.6 against 85.4; 38 samples, T = 23, 1419 -> 29 11.2 against 11.8.
// Outputs written straight from the accumulators instead of by whole rows
// through LDS took 21.4 and 25.1 us at the first two.
#include "common.hpp"
#include "bf16_stage.hpp"
#include "split_bf16.hpp"
#include "ps_split.hpp"

namespace dpg {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
using split::finite_f32;

constexpr int kThreads = 256;

// 16 bytes of elements at their natural alignment only
template <typename T, int V>
struct __attribute__((packed, aligned(sizeof(T)))) Pack {
    T v[V];
};

// One operand of a tile: W features of stages of BK positions
template <typename T, int W_>
struct Side {
    static constexpr int W = W_;
    static constexpr int VEC = 16 / (int)sizeof(T);            // features per 16-byte load
    static constexpr int BK = sizeof(T) == 4 ? 32 : 64;
    static constexpr int ROW = 2 * BK;                          // LDS bytes per feature and plane
    static constexpr int SPARE = W * ROW;                       // a slot that nothing reads
    static constexpr int PLANE = SPARE + 16;
    static constexpr int FC = W / VEC;                          // feature groups
    static constexpr int R = BK * FC / kThreads;                // rows per thread
    static constexpr int FL = FC < 16 ? FC : 16;                // feature groups across a wave's lanes
    static_assert(R == 2 || R == 4, "staging map");

    // Byte offset of feature f in a plane, position unit 0, and the XOR its
    // 16-byte position units take.  Both the reads (16 consecutive features,
    // one unit) and the writes (every VEC-th feature) then spread over all
    // banks: the 16-byte slot inside a 256-byte window is linear in the bits
    // of f, injective on f's low four bits and on those above log2(VEC).
    static __device__ __forceinline__ int row_base(int f)
    {
        if constexpr (ROW == 64) return (f >> 2) * 256 + 64 * ((f ^ (f >> 4)) & 3);
        else return (f >> 1) * 256 + 128 * ((f ^ (f >> 4)) & 1);
    }
    static __device__ __forceinline__ int row_xor(int f)
    {
        if constexpr (ROW == 64) return (f >> 2) & 3;
        else return (((f >> 1) ^ (f >> 5)) & 3) | ((f >> 1) & 4);
    }
    static __device__ __forceinline__ int at(int f, int t)      // t even
    {
        return row_base(f) + 16 * ((t >> 3) ^ row_xor(f)) + 2 * (t & 7);
    }

    typedef Pack<T, VEC> Rows;

    int d;               // row length
    int f;               // first feature this thread loads
    int t;               // first row of its R rows
    uint32_t w[VEC];     // LDS offset of its features' first position

    // Features f .. f + VEC - 1, moved back to end at d when they would pass
    // it (the neighbour then writes some of them too, with the same values).
    // The ones before the tile, and whole groups past d, go to the spare slot.
    __device__ __forceinline__ void init(i64 d_, int f0)
    {
        d = (int)d_;
        const int tid = threadIdx.x;
        const int fc = (tid % FL) + FL * ((tid / 64) % (FC / FL));
        const int rg = (tid % 64) / FL + (64 / FL) * (tid / 64 / (FC / FL));
        const int lf = fc * VEC;
        f = f0 + lf;
        const bool none = f >= d;
        f = f < d - VEC ? f : d - VEC;
        t = R * rg;
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            const int row = f + k - f0;
            w[k] = none || row < 0 ? (uint32_t)SPARE : (uint32_t)at(row, t);
        }
    }
    // The rows of the stage whose first row is at q; rows at or past `left`
    // are zeros for fp32 (a buffer load past its range reads zero; a group
    // never passes its row's end) and must be cleared by zero_rows for bf16,
    // whose 2-byte aligned loads are ordinary ones.
    __device__ __forceinline__ void load(const T *q, int left, Pack<T, VEC> (&g)[R]) const
    {
        if constexpr (sizeof(T) == 4) {
            const __amdgpu_buffer_rsrc_t rs = sample_rsrc(q, (uint32_t)(left * d) * 4u);
#pragma unroll
            for (int r = 0; r < R; ++r)
                g[r] = __builtin_bit_cast(
                    Rows, __builtin_amdgcn_raw_buffer_load_b128(rs, (uint32_t)((t + r) * d + f) * 4u, 0, 0));
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int row = t + r < left ? t + r : left - 1;
                const uint32_t at_byte = (uint32_t)(row * d + f) * (uint32_t)sizeof(T);
                g[r] = *reinterpret_cast<const Pack<T, VEC> *>(reinterpret_cast<const char *>(q) + at_byte);
            }
        }
    }
    __device__ __forceinline__ void zero_rows(int left, Pack<T, VEC> (&g)[R]) const
    {
        if constexpr (sizeof(T) == 2) {
            if (left < BK) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int k = 0; k < VEC; ++k) g[r].v[k] = t + r < left ? g[r].v[k] : T(0);
            }
        }
    }
};

// Tile of 64 FM (j) x 64 FN (i): four waves as 2 x 2, each FM x FN blocks of 32 x 32
template <typename T, int FM_, int FN_>
struct Cfg {
    typedef T elem;
    static constexpr int FM = FM_, FN = FN_;
    static constexpr int BM = 64 * FM, BN = 64 * FN;
    typedef Side<T, BM> SA;
    typedef Side<T, BN> SB;
    static constexpr int BK = SA::BK;
    static constexpr int NP = sizeof(T) == 4 ? 3 : 1;       // planes
    static constexpr int STAGE = NP * (SA::PLANE + SB::PLANE);
};

template <typename C>
struct Shared {
    __attribute__((aligned(1024))) char stage[2 * C::STAGE];
    float red[16];
};

template <typename T>
__device__ __forceinline__ float as_f32(T v);
template <>
__device__ __forceinline__ float as_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float as_f32<uint16_t>(uint16_t v) { return bf16_to_f32(v); }

// Writes a thread's R rows x VEC features: per feature, its R positions in every plane
template <typename S, typename T, int NP>
__device__ __forceinline__ void put(char *L, const S &s, const Pack<T, S::VEC> (&g)[S::R])
{
#pragma unroll
    for (int k = 0; k < S::VEC; ++k) {
        uint32_t q[NP][S::R / 2];
#pragma unroll
        for (int r = 0; r < S::R; r += 2) {
            if constexpr (NP == 3)
                split::split2(g[r].v[k], g[r + 1].v[k], q[0][r / 2], q[1][r / 2], q[2][r / 2]);
            else
                q[0][r / 2] = (uint32_t)g[r].v[k] | (uint32_t)g[r + 1].v[k] << 16;
        }
#pragma unroll
        for (int a = 0; a < NP; ++a) {
            char *o = L + s.w[k] + a * S::PLANE;
            if constexpr (S::R == 4) *reinterpret_cast<uint2 *>(o) = make_uint2(q[a][0], q[a][1]);
            else *reinterpret_cast<uint32_t *>(o) = q[a][0];
        }
    }
}

// Tile `tile` of sample n (the body of the single-layer and grouped launches)
template <typename C>
__device__ __forceinline__ void tile_body(const typename C::elem *__restrict__ A,
                                          const typename C::elem *__restrict__ B, i64 T, i64 din, i64 dout,
                                          int tiles_j, int tiles, i64 n, int tile, float scale,
                                          float *__restrict__ gW, float *__restrict__ gb,
                                          float *__restrict__ partial, Shared<C> &sh)
{
    typedef typename C::elem E;
    typedef typename C::SA SA;
    typedef typename C::SB SB;
    constexpr int FM = C::FM, FN = C::FN, NP = C::NP, VEC = SA::VEC, BK = C::BK;
    const int ti = (int)((uint32_t)tile / (uint32_t)tiles_j), tj = tile - ti * tiles_j;
    const int j0 = tj * C::BM, i0 = ti * C::BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wj = (wave >> 1) * 32 * FM, wi = (wave & 1) * 32 * FN;
    const int li = lane & 31, kg = lane >> 5;
    const bool do_bias = gb != nullptr && tj == 0;
    const int Ti = (int)T, nst = (Ti + BK - 1) / BK;
    const E *An = A + n * T * din, *Bn = B + n * T * dout;

    SA sa;
    SB sb;
    sa.init(din, j0);
    sb.init(dout, i0);
    Pack<E, VEC> ga[2][SA::R], gbk[2][SB::R];
    float bsum[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) bsum[k] = 0.0f;

    // big: h*h products; rest: the five smaller ones (their rounding is that of much smaller sums)
    f32x16_t big[FM][FN], rest[FM][FN];
#pragma unroll
    for (int x = 0; x < FM; ++x)
#pragma unroll
        for (int y = 0; y < FN; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                big[x][y][r] = 0.0f;
                rest[x][y][r] = 0.0f;
            }

    const int last = nst - 1;
    auto load_stage = [&](int c, Pack<E, VEC> (&xa)[SA::R], Pack<E, VEC> (&xb)[SB::R]) {
        const i64 t0 = (i64)c * BK;
        const int left = Ti - c * BK < BK ? Ti - c * BK : BK;
        sa.load(An + t0 * din, left, xa);
        sb.load(Bn + t0 * dout, left, xb);
    };
    auto store_stage = [&](int c, Pack<E, VEC> (&xa)[SA::R], Pack<E, VEC> (&xb)[SB::R]) {
        const int left = Ti - c * BK;
        sa.zero_rows(left, xa);
        sb.zero_rows(left, xb);
        char *L = sh.stage + (c & 1) * C::STAGE;
        put<SA, E, NP>(L, sa, xa);
        put<SB, E, NP>(L + NP * SA::PLANE, sb, xb);
        if (do_bias && c <= last) {
            // (a thread's rows are added up first: fewer roundings at the size of the whole sum)
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                float t = as_f32<E>(xb[0].v[k]) + as_f32<E>(xb[1].v[k]);
                if constexpr (SB::R == 4) t += as_f32<E>(xb[2].v[k]) + as_f32<E>(xb[3].v[k]);
                bsum[k] += t;
            }
        }
    };
    // operand addresses: features wj + 32x + li (A), wi + 32y + li (B), unit 2 ks + kg
    auto mma_stage = [&](int c) {
        const char *L = sh.stage + (c & 1) * C::STAGE;
        const char *LB = L + NP * SA::PLANE;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8_t a[FM][NP], b[FN][NP];
#pragma unroll
            for (int x = 0; x < FM; ++x)
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    a[x][p] = *reinterpret_cast<const bf16x8_t *>(L + p * SA::PLANE +
                                                                  SA::at(wj + 32 * x + li, 16 * ks + 8 * kg));
#pragma unroll
            for (int y = 0; y < FN; ++y)
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    b[y][p] = *reinterpret_cast<const bf16x8_t *>(LB + p * SB::PLANE +
                                                                  SB::at(wi + 32 * y + li, 16 * ks + 8 * kg));
            if constexpr (NP == 3) {
#pragma unroll
                for (int o = 2; o >= 1; --o)             // hl, mm, lh, then hm, mh
#pragma unroll
                    for (int p = 0; p <= o; ++p)
#pragma unroll
                        for (int x = 0; x < FM; ++x)
#pragma unroll
                            for (int y = 0; y < FN; ++y)
                                rest[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[x][p], b[y][o - p], rest[x][y],
                                                                                     0, 0, 0);
            }
#pragma unroll
            for (int x = 0; x < FM; ++x)
#pragma unroll
                for (int y = 0; y < FN; ++y)
                    big[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[x][0], b[y][0], big[x][y], 0, 0, 0);
        }
    };

    // Stage c is multiplied while stage c+2 is loaded into the registers that
    // stage c left, and stage c+1, loaded a stage ago, is then written to the
    // other LDS buffer.  Past the end the last stage is loaded and written
    // again, for nobody: a loop without branches around loads lets each
    // register set be waited for by itself.
    load_stage(0, ga[0], gbk[0]);
    if (nst > 1) {
        load_stage(1, ga[1], gbk[1]);
        __builtin_amdgcn_sched_barrier(0);
        store_stage(0, ga[0], gbk[0]);
    } else {
        store_stage(0, ga[0], gbk[0]);
    }
    // Between two MFMAs of a stage, its share of the operand reads and of the
    // next stage's split and LDS writes: they run while the matrix unit works.
    auto interleave = [&]() {
        if constexpr (NP == 3) {
            constexpr int M = 6 * FM * FN * BK / 16;
            constexpr int RD = 3 * (FM + FN) * BK / 16, WR = 2 * VEC * NP;
            __builtin_amdgcn_sched_group_barrier(0x100, RD / 2, 0);
#pragma unroll
            for (int i = 0; i < M; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
                if ((i + 1) * WR / M > i * WR / M) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                if (i < M / 2 && (i + 1) * RD / M > i * RD / M) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
        }
    };
    auto step = [&](int c, Pack<E, VEC> (&xa)[SA::R], Pack<E, VEC> (&xb)[SB::R], Pack<E, VEC> (&ya)[SA::R],
                    Pack<E, VEC> (&yb)[SB::R]) {
        lds_barrier();                                   // stage c written; stage c-1 read
        load_stage(c + 2 < last ? c + 2 : last, xa, xb);
        __builtin_amdgcn_sched_barrier(0);               // the loads go out before the MFMAs
        mma_stage(c);
        store_stage(c + 1, ya, yb);
        interleave();
    };
    for (int c = 0; c + 1 < nst; c += 2) {
        step(c, ga[0], gbk[0], ga[1], gbk[1]);
        step(c + 1, ga[1], gbk[1], ga[0], gbk[0]);
    }
    if (nst & 1) {
        lds_barrier();
        mma_stage(last);
    }

    // block (x, y), register r of lane l: j = j0 + wj + 32x + 8 (r / 4) + 4 (l / 32) + r % 4, i = i0 + wi + 32y + l % 32
    const int Di = (int)din, Do = (int)dout;
    float sq = 0.0f;
    auto finish = [&](float factor) {                    // the gradients, and their squares inside the layer
        sq = 0.0f;
#pragma unroll
        for (int x = 0; x < FM; ++x)
#pragma unroll
            for (int y = 0; y < FN; ++y)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = j0 + wj + 32 * x + 8 * (r >> 2) + 4 * kg + (r & 3), i = i0 + wi + 32 * y + li;
                    const float g = scale * (factor * big[x][y][r]);
                    big[x][y][r] = g;
                    const float v = i < Do && j < Di ? g : 0.0f;
                    sq += v * v;
                }
    };
    if constexpr (NP == 3) {
#pragma unroll
        for (int x = 0; x < FM; ++x)
#pragma unroll
            for (int y = 0; y < FN; ++y) big[x][y] += rest[x][y];
        finish(split::kUnscale);
        if (__any(!finite_f32(sq))) [[unlikely]] {
            // An infinity, a NaN or a value too large to split among the wave's
            // inputs, or outputs whose squares pass fp32's range: the wave's
            // block again on fp32 MFMA, positions 2p + l / 32 of a step
            // straight from memory (64 samples of 100 -> 400, T = 256, all
            // with a NaN 54 us; by one fma per lane and position 1360).
            constexpr int U = 8;
#pragma unroll
            for (int x = 0; x < FM; ++x)
#pragma unroll
                for (int y = 0; y < FN; ++y)
#pragma unroll
                    for (int r = 0; r < 16; ++r) big[x][y][r] = 0.0f;
            for (int t0 = 0; t0 < Ti; t0 += 2 * U) {
                float a[FM][U], b[FN][U];
#pragma unroll
                for (int p = 0; p < U; ++p) {
                    const int t = t0 + 2 * p + kg;
#pragma unroll
                    for (int x = 0; x < FM; ++x) {
                        const int j = j0 + wj + 32 * x + li;
                        a[x][p] = t < Ti && j < Di ? as_f32<E>(An[t * din + j]) : 0.0f;
                    }
#pragma unroll
                    for (int y = 0; y < FN; ++y) {
                        const int i = i0 + wi + 32 * y + li;
                        b[y][p] = t < Ti && i < Do ? as_f32<E>(Bn[t * dout + i]) : 0.0f;
                    }
                }
#pragma unroll
                for (int p = 0; p < U; ++p)
#pragma unroll
                    for (int x = 0; x < FM; ++x)
#pragma unroll
                        for (int y = 0; y < FN; ++y)
                            big[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[x][p], b[y][p], big[x][y], 0, 0, 0);
            }
            finish(1.0f);
        }
    } else {
        finish(1.0f);
    }
    float *G = gW + n * dout * din;
    lds_barrier();                                       // the stages' LDS is free
    {
        // Through LDS, so that a wave's stores cover whole rows of its block:
        // straight from the accumulators every store instruction would touch
        // 32 rows with 32 bytes each.
        constexpr int LD = 32 * FM + 4, CPR = 32 * FM / 4, RPI = kWave / CPR;
        static_assert(4 * 32 * FN * LD * 4 <= 2 * C::STAGE, "output staging");
        float *buf = reinterpret_cast<float *>(sh.stage) + wave * (32 * FN * LD);
#pragma unroll
        for (int x = 0; x < FM; ++x)
#pragma unroll
            for (int y = 0; y < FN; ++y)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4 *>(buf + (32 * y + li) * LD + 32 * x + 8 * q + 4 * kg) =
                        make_float4(big[x][y][4 * q], big[x][y][4 * q + 1], big[x][y][4 * q + 2], big[x][y][4 * q + 3]);
        const int j = j0 + wj + 4 * (lane % CPR);
#pragma unroll
        for (int r = 0; r < 32 * FN / RPI; ++r) {
            const int row = RPI * r + lane / CPR, i = i0 + wi + row;
            const float4 v = *reinterpret_cast<const float4 *>(buf + row * LD + 4 * (lane % CPR));
            float *p = G + i * din + j;
            if (i < Do && j + 4 <= Di) {
                *reinterpret_cast<Pack<float, 4> *>(p) = Pack<float, 4>{{v.x, v.y, v.z, v.w}};
            } else if (i < Do && j < Di) {
                p[0] = v.x;
                if (j + 1 < Di) p[1] = v.y;
                if (j + 2 < Di) p[2] = v.z;
            }
        }
    }
    if (do_bias) {
        // a feature's row groups, added in pairs
        float *bred = reinterpret_cast<float *>(sh.stage);    // [RG][BN]
        constexpr int RG = BK / SB::R;
        static_assert(RG * C::BN * 4 <= 2 * C::STAGE, "bias scratch");
        lds_barrier();
#pragma unroll
        for (int k = 0; k < VEC; ++k)
            if (sb.w[k] != SB::SPARE) bred[(sb.t / SB::R) * C::BN + sb.f + k - i0] = bsum[k];
        lds_barrier();
        if (tid < C::BN && i0 + tid < Do) {
            float p[RG];
#pragma unroll
            for (int r = 0; r < RG; ++r) p[r] = bred[r * C::BN + tid];
#pragma unroll
            for (int n = RG / 2; n >= 1; n /= 2)
#pragma unroll
                for (int r = 0; r < n; ++r) p[r] += p[r + n];
            const float s = scale * p[0];
            gb[n * dout + i0 + tid] = s;
            sq += s * s;
        }
    }
    sq = wave_sum(sq);
    if (lane == 0) sh.red[wave] = sq;
    lds_barrier();
    if (partial && tid == 0) partial[n * tiles + tile] = sh.red[0] + sh.red[1] + sh.red[2] + sh.red[3];
}

template <typename C>
__global__ __launch_bounds__(kThreads, 2) void ps_split_kernel(const typename C::elem *__restrict__ A,
                                                               const typename C::elem *__restrict__ B, i64 T,
                                                               i64 din, i64 dout, int tiles_j, int tiles, float scale,
                                                               float *__restrict__ gW, float *__restrict__ gb,
                                                               float *__restrict__ partial)
{
    __shared__ Shared<C> sh;
    const uint32_t b = xcd_swizzle32(blockIdx.x, gridDim.x), n = b / (uint32_t)tiles;
    tile_body<C>(A, B, T, din, dout, tiles_j, tiles, n, (int)(b - n * tiles), scale, gW, gb, partial, sh);
}

struct Item {
    const float *A, *B;
    i64 T, din, dout;
    int tiles_j, tiles, tile0, wide;
    float scale;
    float *gW, *gb, *sqnorm, *partial;
};
struct Group16 {
    int count, tiles_all;
    i64 N;
    Item it[kPsGroupMax];
};

// Tiles of 64 (j) x 128 (i) or 128 x 64, whichever covers the layer with less
// padding.  On 64 x 64 and 128 x 128 tiles the LSTM's layer (100 x 400, T =
// 256, 64 samples) took 22.3 and 22.0 us against 19.9 (the first split and
// read every operand more often, the second has one workgroup per CU).
template <typename T>
using Wide = Cfg<T, 2, 1>;       // along j
template <typename T>
using Tall = Cfg<T, 1, 2>;       // along i

i64 tiles_of(i64 din, i64 dout, bool wide)
{
    return wide ? ceil_div(din, 128) * ceil_div(dout, 64) : ceil_div(din, 64) * ceil_div(dout, 128);
}
bool is_wide(i64 din, i64 dout) { return tiles_of(din, dout, true) < tiles_of(din, dout, false); }

// Several fp32 layers sharing N: workgroup b takes sample b / tiles_all and,
// of that sample's tiles of all layers (layer after layer), tile b %
// tiles_all, so layers that read the same B (an LSTM's two weight matrices)
// read it while it is in L2.
__global__ __launch_bounds__(kThreads, 2) void ps_split_group_kernel(const Group16 g)
{
    __shared__ union {
        Shared<Wide<float>> w;
        Shared<Tall<float>> t;
    } sh;
    const uint32_t b = xcd_swizzle32(blockIdx.x, gridDim.x), n = b / (uint32_t)g.tiles_all;
    const int r = (int)(b - n * g.tiles_all);
    int k = 0;
    while (k + 1 < g.count && g.it[k + 1].tile0 <= r) ++k;
    const Item &L = g.it[k];
    if (L.wide)
        tile_body<Wide<float>>(L.A, L.B, L.T, L.din, L.dout, L.tiles_j, L.tiles, n, r - L.tile0, L.scale, L.gW, L.gb,
                               L.partial, sh.w);
    else
        tile_body<Tall<float>>(L.A, L.B, L.T, L.din, L.dout, L.tiles_j, L.tiles, n, r - L.tile0, L.scale, L.gW, L.gb,
                               L.partial, sh.t);
}

// One wave per (layer, sample): sqnorm[n] = the sample's tile partials added
// as sum_partials adds them.
__global__ __launch_bounds__(256) void ps_split_group_sqnorm_kernel(const Group16 g)
{
    const Item &L = g.it[blockIdx.y];
    const i64 n = (i64)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (L.sqnorm == nullptr || n >= g.N) return;
    const float *p = L.partial + n * L.tiles;
    float s = 0.0f;
    for (int t = lane; t < L.tiles; t += kWave) s += p[t];
    s = wave_sum(s);
    if (lane == 0) L.sqnorm[n] = s;
}

template <typename C>
void launch(const PsLayer &L, i64 N, hipStream_t stream)
{
    typedef typename C::elem E;
    const int tiles_j = (int)ceil_div(L.din, C::BM), tiles = ps_split_parts(L.din, L.dout);
    ps_split_kernel<C><<<(unsigned)(N * tiles), kThreads, 0, stream>>>((const E *)L.A, (const E *)L.B, L.T, L.din, L.dout,
                                                                       tiles_j, tiles, L.scale, L.gW, L.gb,
                                                                       L.sqnorm ? L.partial : nullptr);
    if (L.sqnorm) sum_partials(L.partial, N, tiles, L.sqnorm, stream);
}

}  // namespace

bool ps_split_ok(dp_dtype dt, i64 T, i64 din, i64 dout)
{
    const i64 least = dt == DP_F32 ? 4 : 8, most = i64(1) << 22;
    return T >= 2 && T < (i64(1) << 31) && din >= least && dout >= least && din < most && dout < most;
}

int ps_split_parts(i64 din, i64 dout) { return (int)tiles_of(din, dout, is_wide(din, dout)); }

void ps_split_grad(const PsLayer &layer, dp_dtype dt, i64 N, hipStream_t stream)
{
    const bool wide = is_wide(layer.din, layer.dout);
    if (dt == DP_F32)
        wide ? launch<Wide<float>>(layer, N, stream) : launch<Tall<float>>(layer, N, stream);
    else
        wide ? launch<Wide<uint16_t>>(layer, N, stream) : launch<Tall<uint16_t>>(layer, N, stream);
}

void ps_split_group(const PsLayer *layers, int count, i64 N, hipStream_t stream)
{
    if (count <= 0 || N <= 0) return;
    Group16 g;
    g.count = count;
    g.N = N;
    int tiles_all = 0;
    bool norms = false;
    for (int k = 0; k < count; ++k) {
        const PsLayer &L = layers[k];
        const int tiles = ps_split_parts(L.din, L.dout);
        const bool wide = is_wide(L.din, L.dout);
        g.it[k] = {(const float *)L.A, (const float *)L.B, L.T, L.din, L.dout, (int)ceil_div(L.din, wide ? 128 : 64),
                   tiles, tiles_all, wide, L.scale, L.gW, L.gb, L.sqnorm, L.sqnorm ? L.partial : nullptr};
        tiles_all += tiles;
        norms = norms || L.sqnorm != nullptr;
    }
    for (int k = count; k < kPsGroupMax; ++k) {
        g.it[k] = g.it[count - 1];
        g.it[k].tile0 = tiles_all;
    }
    g.tiles_all = tiles_all;
    ps_split_group_kernel<<<(unsigned)(N * tiles_all), kThreads, 0, stream>>>(g);
    if (norms)
        ps_split_group_sqnorm_kernel<<<dim3((unsigned)ceil_div(N, 4), (unsigned)count), 256, 0, stream>>>(g);
}

}  // namespace dpg
