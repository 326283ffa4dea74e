// Per-sample gradients of a Linear layer over a sequence (appendix
// "Vectorized Computation", extra dimension summed):
//   gW_n[i][j] = s * sum_t B_n[t][i] * A_n[t][j],   gb_n[i] = s * sum_t B_n[t][i]
// for any T and alignment, fp32 or bf16 inputs, on v_mfma_f32_32x32x16_bf16.
// fp32 operands are split into three bf16 parts (split_bf16.hpp: six products,
// fp32 results); bf16 operands go in as they are.
//
// Block = (sample, tile of gW_n).  Stages of consecutive positions are loaded
// into registers one or two stages ahead, R rows x 16 bytes per thread, then split
// and written to LDS with the positions contiguous ([feature][t], one plane
// per part; packing two positions of a feature into a word costs the same as
// packing two features), so that an MFMA operand (eight positions of one
// feature per lane) is one ds_read_b128.
//
// What bounds it: at the LSTM's layer (fp32, 64 samples, T = 256, 100 -> 400:
// 43 MB and, in six products, 7.9 GFLOP of bf16 MFMA) about half of the call
// is fixed (two launches, the first loads, the last stores) and a stage costs
// its MFMAs plus about half of its split (the conversions and LDS writes
// that the interleaving does not hide).  20.5-21.7 us against 24.3 with fp32
// MFMA; off 64 bits by 0.90e-7 (weights) and 0.88e-7 (bias) against 2.05e-7 and
// 1.00e-7.  A bf16 layer of odd sizes (48 samples, T = 75, 300 -> 514, 36 MB) 20.6 us
// against 42.0 with element loads and fp32 MFMA; 768 x 768 over T = 512 (32 samples,
// fp32) 131 against 164.  Outputs written straight from the accumulators
// instead of by whole rows through LDS took 21.4 and 25.1 us at the first two.
#include "common.hpp"
#include "bf16_stage.hpp"
#include "split_bf16.hpp"
#include "ps_split.hpp"

#include <type_traits>

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
    bool none;           // its features are all past d
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
        f = f0 + fc * VEC;
        none = f >= d;
        f = f < d - VEC ? f : d - VEC;
        t = R * rg;
    }
    __device__ __forceinline__ void init_lds(int f0)
    {
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

// Tile of 64 FM (j) x 64 FN (i): four waves as 2 x 2, each FM x FN blocks of 32 x 32; NB stages in LDS
template <typename T, int FM_, int FN_, int NB_>
struct Cfg {
    typedef T elem;
    static constexpr int FM = FM_, FN = FN_, NB = NB_;
    static constexpr int WGS = NB == 1 ? 4 : sizeof(T) == 2 ? 3 : 2;   // workgroups per CU, at least
    static constexpr int BM = 64 * FM, BN = 64 * FN;
    typedef Side<T, BM> SA;
    typedef Side<T, BN> SB;
    static constexpr int BK = SA::BK;
    static constexpr int NP = sizeof(T) == 4 ? 3 : 1;       // planes
    static constexpr int STAGE = NP * (SA::PLANE + SB::PLANE);
    static constexpr int LD = 32 * FM + 4, OUT = 4 * 32 * FN * LD * 4;   // output staging: row length, bytes
    static constexpr int LDS = NB * STAGE > OUT ? NB * STAGE : OUT;
};

// LDS of a workgroup
template <typename C>
struct Shared {
    __attribute__((aligned(1024))) char stage[C::LDS];
    float red[4][2], bred[2];
};

template <typename T>
__device__ __forceinline__ float as_f32(T v);
template <>
__device__ __forceinline__ float as_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float as_f32<uint16_t>(uint16_t v) { return bf16_to_f32(v); }

// v added over the lanes that differ in the bits of D (a power of two, to 32), by
// the VALU alone (LDS permutes would add their latency to the end of every workgroup)
template <int D>
__device__ __forceinline__ float add_across(float v)
{
    const uint32_t u = __float_as_uint(v);
    if constexpr (D == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else if constexpr (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
        // rotations by 8 and 4 of 16 lanes (after 8, lanes i and i + 4 of any eight are i and i ^ 4), swaps in fours
        constexpr int ctrl = D == 8 ? 0x128 : D == 4 ? 0x124 : D == 2 ? 0x4E : 0xB1;
        return v + __int_as_float(__builtin_amdgcn_update_dpp(0, (int)u, ctrl, 0xF, 0xF, false));
    }
}
// the sum over a wave, in every lane
__device__ __forceinline__ float add_lanes(float v)
{
    return add_across<1>(add_across<2>(add_across<4>(add_across<8>(add_across<16>(add_across<32>(v))))));
}

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
                                          int tiles_j, int parts, i64 n, int tile, float scale,
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
    if constexpr (C::NB > 1) {
        sa.init_lds(j0);
        sb.init_lds(i0);
    }
    Pack<E, VEC> ga[C::NB][SA::R], gbk[C::NB][SB::R];
    float bsum[SB::R / 2][VEC];
#pragma unroll
    for (int r = 0; r < SB::R / 2; ++r)
#pragma unroll
        for (int k = 0; k < VEC; ++k) bsum[r][k] = 0.0f;

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
        char *L = sh.stage + c % C::NB * C::STAGE;
        if constexpr (C::NB == 1) {
            // steps of 16 rows past the last position are neither written nor multiplied
            const int rows = (left + 15) & ~15;
            if (sa.t < rows) put<SA, E, NP>(L, sa, xa);
            if (sb.t < rows) put<SB, E, NP>(L + NP * SA::PLANE, sb, xb);
        } else {
            put<SA, E, NP>(L, sa, xa);
            put<SB, E, NP>(L + NP * SA::PLANE, sb, xb);
        }
        if (do_bias && c <= last) {
            // (pairs of rows first: fewer roundings at the size of the whole sum)
#pragma unroll
            for (int r = 0; r < SB::R / 2; ++r)
#pragma unroll
                for (int k = 0; k < VEC; ++k) bsum[r][k] += as_f32<E>(xb[2 * r].v[k]) + as_f32<E>(xb[2 * r + 1].v[k]);
        }
    };
    // operand addresses: features wj + 32x + li (A), wi + 32y + li (B), unit 2 ks + kg
    auto mma_stage = [&](int c) {
        const char *L = sh.stage + c % C::NB * C::STAGE;
        const char *LB = L + NP * SA::PLANE;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            if (C::NB == 1 && 16 * ks >= Ti - c * BK) break;
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

    if constexpr (C::NB == 1) {
        // one stage in LDS: the CU's other workgroups multiply while this one loads and splits
        load_stage(0, ga[0], gbk[0]);
        __builtin_amdgcn_sched_barrier(0);
        sa.init_lds(j0);
        sb.init_lds(i0);
        for (int c = 0; c < nst; ++c) {
            if (c > 0) lds_barrier();                    // stage c-1 read
            store_stage(c, ga[0], gbk[0]);
            if (c < last) load_stage(c + 1, ga[0], gbk[0]);
            lds_barrier();                               // stage c written
            mma_stage(c);
        }
    } else {
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
    }

    // block (x, y), register r of lane l: j = j0 + wj + 32x + 8 (r / 4) + 4 (l / 32) + r % 4, i = i0 + wi + 32y + l % 32
    const int Di = (int)din, Do = (int)dout;
    float sq[FM][FN];
    auto finish = [&](float factor) {                    // the gradients; per block, the lane's squares inside the layer
        float all = 0.0f;
#pragma unroll
        for (int x = 0; x < FM; ++x)
#pragma unroll
            for (int y = 0; y < FN; ++y) {
                float t = 0.0f;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = j0 + wj + 32 * x + 8 * (r >> 2) + 4 * kg + (r & 3), i = i0 + wi + 32 * y + li;
                    const float g = scale * (factor * big[x][y][r]);
                    big[x][y][r] = g;
                    const float v = i < Do && j < Di ? g : 0.0f;
                    t += v * v;
                }
                sq[x][y] = t;
                all += t;
            }
        return all;
    };
    if constexpr (NP == 3) {
#pragma unroll
        for (int x = 0; x < FM; ++x)
#pragma unroll
            for (int y = 0; y < FN; ++y) big[x][y] += rest[x][y];
        if (__any(!finite_f32(finish(split::kUnscale)))) [[unlikely]] {
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
        constexpr int LD = C::LD, CPR = 32 * FM / 4, RPI = kWave / CPR;
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
    float bsq = 0.0f;
    if (do_bias) {
        // a feature's pairs of rows: a thread's, its neighbours' in the wave, then the waves', always two by two
        // (so in one order whatever the tile is)
        float *bred = reinterpret_cast<float *>(sh.stage);    // [GW][BN]
        constexpr int GW = 4 * SB::FL / SB::FC;               // waves that share features
        float v[VEC];
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            v[k] = SB::R == 4 ? bsum[0][k] + bsum[SB::R / 2 - 1][k] : bsum[0][k];
            if constexpr (SB::FL == 8) v[k] = add_across<8>(v[k]);
            v[k] = add_across<32>(add_across<16>(v[k]));
        }
        lds_barrier();
#pragma unroll
        for (int k = 0; k < VEC; ++k)
            if (lane < SB::FL && sb.w[k] != SB::SPARE) bred[wave * GW / 4 * C::BN + sb.f + k - i0] = v[k];
        lds_barrier();
        if (tid < C::BN && i0 + tid < Do) {
            float p[GW];
#pragma unroll
            for (int r = 0; r < GW; ++r) p[r] = bred[r * C::BN + tid];
            p[0] += p[1];
            if constexpr (GW == 4) p[0] += p[2] + p[3];
            const float s = scale * p[0];
            gb[n * dout + i0 + tid] = s;
            bsq = s * s;
        }
    }
    // The squares of every 64 x 64 tile are added in one order, block by block,
    // whatever the workgroup's tile is: so are the sample's, and neither they
    // nor the gradients depend on the choice of tiles.
    if (partial == nullptr) return;
#pragma unroll
    for (int x = 0; x < FM; ++x)
#pragma unroll
        for (int y = 0; y < FN; ++y) {
            const float t = add_lanes(sq[x][y]);
            if (lane == 0) sh.red[wave][x * FN + y] = t;
        }
    if (do_bias && wave < FN) {
        const float t = add_lanes(bsq);
        if (lane == 0) sh.bred[wave] = t;
    }
    lds_barrier();
    if (tid < FM * FN) {
        const int pj = (Di + 63) / 64, at = (FN * ti + (FN > 1 ? tid : 0)) * pj + FM * tj + (FM > 1 ? tid : 0);
        // blocks (j half, i half) of the tile: 00, 01, 10, 11
        float t;
        if constexpr (FM > 1) t = ((sh.red[2 * tid][0] + sh.red[2 * tid + 1][0]) + sh.red[2 * tid][1]) + sh.red[2 * tid + 1][1];
        else if constexpr (FN > 1) t = ((sh.red[tid][0] + sh.red[tid][1]) + sh.red[2 + tid][0]) + sh.red[2 + tid][1];
        else t = ((sh.red[0][0] + sh.red[1][0]) + sh.red[2][0]) + sh.red[3][0];
        if (do_bias && (FM == 1 || tid == 0)) t += sh.bred[FN > 1 ? tid : 0];
        if (FM * tj + (FM > 1 ? tid : 0) < pj && FN * ti + (FN > 1 ? tid : 0) < (Do + 63) / 64) partial[n * parts + at] = t;
    }
}

template <typename C>
__global__ __launch_bounds__(kThreads, C::WGS) void ps_split_kernel(const typename C::elem *__restrict__ A,
                                                               const typename C::elem *__restrict__ B, i64 T,
                                                               i64 din, i64 dout, int tiles_j, int tiles, int parts,
                                                               float scale,
                                                               float *__restrict__ gW, float *__restrict__ gb,
                                                               float *__restrict__ partial)
{
    __shared__ Shared<C> sh;
    const uint32_t b = xcd_swizzle32(blockIdx.x, gridDim.x), n = b / (uint32_t)tiles;
    tile_body<C>(A, B, T, din, dout, tiles_j, parts, n, (int)(b - n * tiles), scale, gW, gb, partial, sh);
}

struct Item {
    const float *A, *B;
    i64 T, din, dout;
    int tiles_j, parts, tile0, kind;
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
using Wide = Cfg<T, 2, 1, 2>;       // along j
template <typename T>
using Tall = Cfg<T, 1, 2, 2>;       // along i
// Tiles of 64 x 64: with one stage in LDS and five workgroups per CU, whose
// loads, splits, products and stores overlap each other's; or with two
// stages, for grids that put one workgroup on a CU, which is bound by the chain of a
// stage and hides its loads behind its own products only.
template <typename T>
using Small = Cfg<T, 1, 1, 1>;
template <typename T>
using Lone = Cfg<T, 1, 1, 2>;
enum Kind { kWide, kTall, kSmall, kLone };

i64 tiles_of(Kind kind, i64 din, i64 dout)
{
    return ceil_div(din, kind == kWide ? 128 : 64) * ceil_div(dout, kind == kTall ? 128 : 64);
}

// Measured over 1500 drawn layers, us on 64 x 128 / Small / Lone tiles.  fp32:
// 64 samples of 100 -> 400, T = 128 15.3 / 15.3 / 16.8, T = 256 21.4 / 22.0 / 23.5;
// 32 of 768 -> 768, T = 32 30.3 / 24.3 / 29.5, T = 128 48.7 / 47.4 / 54.0, T = 256
// 76.4 / 78.3 / 85.2, T = 512 132 / 141 / 148 (few positions: the stores count, and more
// workgroups keep more of them in flight; many: the reads and splits, which
// larger tiles do less often); 2000 of 16 -> 16, T = 64 30.3 / 15.0 / 19.1,
// T = 512 99 / 57 / 60 (64 x 128 tiles are mostly padding); 256 of 64 -> 64,
// T = 512 22.2 / 19.8 / 17.1 and 4 of 512 -> 512 20.6 / 21.4 / 16.3 (one
// workgroup per CU).  bf16, whose stages have no split and 64 positions:
// 32 of 769 -> 771, T = 64 31.0 / 31.7 / 32.3, T = 512 76 / 82 / 83; 2000 of 17 -> 19,
// T = 64 20.1 / 14.9 / 15.2; 16 of 257 -> 515, T = 128 13.4 / 11.4 / 11.6.
// On fp32 MFMA (64 x 64 tiles copied straight into LDS) these fp32 layers took
// 16.1, 24.3, 28.3, 52.5, 91.8, 166, 17.0, 72, 17.1 and 17.5 us; it was ahead by up to
// 1.2 us at T = 16 alone (191 samples of 16 -> 996 15.0 against 16.2 on Small).
constexpr i64 kLoneGrid = 256, kLoneGridBf16 = 512;

Kind large_kind(i64 din, i64 dout)
{
    return tiles_of(kWide, din, dout) < tiles_of(kTall, din, dout) ? kWide : kTall;
}

// 64 x 128 tiles would be padding to a large part
bool padded(i64 din, i64 dout)
{
    return 10 * tiles_of(kSmall, din, dout) < 17 * tiles_of(large_kind(din, dout), din, dout);
}

// grid64: 64 x 64 tiles of the launch
Kind kind_of(dp_dtype dt, i64 grid64, i64 T, i64 din, i64 dout)
{
    if (grid64 <= (dt == DP_F32 ? kLoneGrid : kLoneGridBf16)) return kLone;
    return padded(din, dout) || (dt == DP_F32 && T <= 192) ? kSmall : large_kind(din, dout);
}

template <typename... C>
union SharedOf;
template <typename A>
union SharedOf<A> {
    Shared<A> a;
};
template <typename A, typename... B>
union SharedOf<A, B...> {
    Shared<A> a;
    SharedOf<B...> b;
};

// Several fp32 layers sharing N: workgroup b takes sample b / tiles_all and,
// of that sample's tiles of all layers (layer after layer), tile b %
// tiles_all, so layers that read the same B (an LSTM's two weight matrices)
// read it while it is in L2.
// SMALL: all layers on Small tiles.
template <bool SMALL>
__global__ __launch_bounds__(kThreads, SMALL ? Small<float>::WGS : 2) void ps_split_group_kernel(const Group16 g)
{
    __shared__ std::conditional_t<SMALL, SharedOf<Small<float>>, SharedOf<Small<float>, Lone<float>, Wide<float>,
                                                                              Tall<float>>> sh;
    const uint32_t b = xcd_swizzle32(blockIdx.x, gridDim.x), n = b / (uint32_t)g.tiles_all;
    const int r = (int)(b - n * g.tiles_all);
    int k = 0;
    while (k + 1 < g.count && g.it[k + 1].tile0 <= r) ++k;
    const Item &L = g.it[k];
    const auto run = [&](auto c) {
        typedef decltype(c) C;
        tile_body<C>(L.A, L.B, L.T, L.din, L.dout, L.tiles_j, L.parts, n, r - L.tile0, L.scale, L.gW, L.gb, L.partial,
                     *reinterpret_cast<Shared<C> *>(&sh));
    };
    if constexpr (SMALL) {
        run(Small<float>());
    } else {
        if (L.kind == kWide) run(Wide<float>());
        else if (L.kind == kTall) run(Tall<float>());
        else if (L.kind == kLone) run(Lone<float>());
        else run(Small<float>());
    }
}

// One wave per (layer, sample): sqnorm[n] = the sample's tile partials added
// as sum_partials adds them.
__global__ __launch_bounds__(256) void ps_split_group_sqnorm_kernel(const Group16 g)
{
    const Item &L = g.it[blockIdx.y];
    const i64 n = (i64)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (L.sqnorm == nullptr || n >= g.N) return;
    const float *p = L.partial + n * L.parts;
    const float s = wave_sum(lane_partials(p, L.parts));
    if (lane == 0) L.sqnorm[n] = s;
}

template <typename C>
void launch(const PsLayer &L, i64 N, int tiles, hipStream_t stream)
{
    typedef typename C::elem E;
    const int tiles_j = (int)ceil_div(L.din, C::BM), parts = ps_split_parts(L.din, L.dout);
    ps_split_kernel<C><<<(unsigned)(N * tiles), kThreads, 0, stream>>>((const E *)L.A, (const E *)L.B, L.T, L.din, L.dout,
                                                                       tiles_j, tiles, parts, L.scale, L.gW, L.gb,
                                                                       L.sqnorm ? L.partial : nullptr);
    if (L.sqnorm) sum_partials(L.partial, N, parts, L.sqnorm, stream);
}

template <typename E>
void launch_kind(Kind kind, const PsLayer &L, i64 N, hipStream_t stream)
{
    const int tiles = (int)tiles_of(kind, L.din, L.dout);
    if (kind == kWide) launch<Wide<E>>(L, N, tiles, stream);
    else if (kind == kTall) launch<Tall<E>>(L, N, tiles, stream);
    else if (kind == kSmall) launch<Small<E>>(L, N, tiles, stream);
    else launch<Lone<E>>(L, N, tiles, stream);
}

}  // namespace

bool ps_split_ok(dp_dtype dt, i64 T, i64 din, i64 dout)
{
    // (positions up to three stages past the last one are counted in 32 bits)
    const i64 least = dt == DP_F32 ? 4 : 8, most = i64(1) << 22;
    return T >= 2 && T < (i64(1) << 31) - 256 && din >= least && dout >= least && din < most && dout < most;
}

int ps_split_parts(i64 din, i64 dout) { return (int)tiles_of(kSmall, din, dout); }

void ps_split_grad(const PsLayer &L, dp_dtype dt, i64 N, hipStream_t stream)
{
    const Kind kind = kind_of(dt, N * tiles_of(kSmall, L.din, L.dout), L.T, L.din, L.dout);
    if (dt == DP_F32) launch_kind<float>(kind, L, N, stream);
    else launch_kind<uint16_t>(kind, L, N, stream);
}

void ps_split_group(const PsLayer *layers, int count, i64 N, hipStream_t stream)
{
    if (count <= 0 || N <= 0) return;
    Group16 g;
    g.count = count;
    g.N = N;
    // The rule of the single call over the group's grid.  Where layers of 64 x
    // 128 tiles are among them, all run at their occupancy, and the others take
    // two stages, or those tiles too where they are not padding.
    i64 grid64 = 0;
    bool norms = false, small = true;
    for (int k = 0; k < count; ++k) {
        grid64 += N * tiles_of(kSmall, layers[k].din, layers[k].dout);
        norms = norms || layers[k].sqnorm != nullptr;
    }
    for (int k = 0; k < count; ++k)
        small = small && kind_of(DP_F32, grid64, layers[k].T, layers[k].din, layers[k].dout) == kSmall;
    int tiles_all = 0;
    for (int k = 0; k < count; ++k) {
        const PsLayer &L = layers[k];
        Kind kind = kind_of(DP_F32, grid64, L.T, L.din, L.dout);
        if (kind == kSmall && !small) kind = padded(L.din, L.dout) ? kLone : large_kind(L.din, L.dout);
        g.it[k] = {(const float *)L.A, (const float *)L.B, L.T, L.din, L.dout,
                   (int)ceil_div(L.din, kind == kWide ? 128 : 64), ps_split_parts(L.din, L.dout), tiles_all, kind,
                   L.scale, L.gW, L.gb, L.sqnorm, L.sqnorm ? L.partial : nullptr};
        tiles_all += (int)tiles_of(kind, L.din, L.dout);
    }
    for (int k = count; k < kPsGroupMax; ++k) {
        g.it[k] = g.it[count - 1];
        g.it[k].tile0 = tiles_all;
    }
    g.tiles_all = tiles_all;
    const unsigned grid = (unsigned)(N * tiles_all);
    if (small) ps_split_group_kernel<true><<<grid, kThreads, 0, stream>>>(g);
    else ps_split_group_kernel<false><<<grid, kThreads, 0, stream>>>(g);
    if (norms)
        ps_split_group_sqnorm_kernel<<<dim3((unsigned)ceil_div(N, 4), (unsigned)count), 256, 0, stream>>>(g);
}

}  // namespace dpg
