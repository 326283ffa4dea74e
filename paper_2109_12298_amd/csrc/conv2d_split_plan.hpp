// What the bf16-matrix Conv2d kernel (conv2d_split.hip) does, and when: the
// plan of a shape, and where a staged unit comes from and goes to.  Plain C++
// (constexpr functions run on both sides), so that the staging can be checked
// against the definition of the gradient without a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace dpg {
namespace csplit {

constexpr int kT = 3;                  // tap rows and columns per group, at most
constexpr int kMaxGroups = 64;
constexpr size_t kLds = 76 * 1024;     // two workgroups per CU

struct ConvGeom {
    int64_t N, Cin, H, W, Cout, Ho, Wo, kh, kw, sh, sw, ph, pw;
};

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
    int full;                          // 3 x 3 taps in one group: stores by whole rows (a bool costs registers:
                                       // 100 samples 24 -> 40 @27^2 5 x 5 stride 2 bf16 36.1 us against 34.7)
    ConvGroup g[kMaxGroups];
};

// floor(i / d) from ceil(2^20 / d), exact while i * d < 2^20
constexpr int div20(int i, int inv) { return (int)(((uint32_t)i * (uint32_t)inv) >> 20); }

// One staged unit: its byte offset in a plane of LDS (-1: none), the column
// and the element offset in the sample of its first element; dead: zeros.
struct UnitAt {
    int at, col, e;
    bool dead;
};

// X unit i = (ci, row, unit) of the chunk that starts at output row oh0
constexpr UnitAt x_unit(const SplitShape &s, int u0, int phase, int ci0, int oh0, int i)
{
    const int c = div20(i, s.inv_xrow), w = i - c * (s.XR * s.NU), r = (w * s.inv_nu) >> 16, cu = w - r * s.NU;
    const int ih = oh0 * s.sh + r + u0 - s.ph, col = 8 * cu * s.sw + phase;
    return {i < s.nx ? c * s.csx + w * 16 : -1, col, ((ci0 + c) * s.H + ih) * s.W + col,
            (uint32_t)ih >= (uint32_t)s.H || ci0 + c >= s.Cin || i >= s.nx};
}

// GY unit i = (co, row, unit) of the chunk that starts at output row oh0
constexpr UnitAt g_unit(const SplitShape &s, int sc, int co0, int oh0, int i)
{
    const int c = div20(i, s.inv_grow), w = i - c * (s.RC * s.gl), r = (w * s.inv_gl) >> 16, cu = w - r * s.gl;
    const int oh = oh0 + r, col = 8 * (cu + s.gp - s.gl - 1) - sc;
    return {i < s.ng ? c * s.csg + (r * s.gp + cu + s.gp - s.gl) * 16 : -1, col, ((co0 + c) * s.Ho + oh) * s.Wo + col,
            oh >= s.Ho || co0 + c >= s.Cout || i >= s.ng};
}

// whether units hold columns outside their row, which must become zeros (where
// any group loads the guards of GY's rows, all do: those are outside)
constexpr bool clips_x(const SplitShape &s) { return s.W % (8 * s.sw) != 0; }
constexpr bool clips_g(const SplitShape &s, int sc) { return s.gl != s.NU || sc != 0 || s.NU * 8 != s.Wo; }

struct Layout {
    int wi, wo, wk;
};
constexpr Layout kLayouts[] = {{1, 2, 1}, {2, 1, 1}, {1, 1, 2}};
inline int odd_units(int bytes) { return (((bytes + 15) / 16) | 1) * 16; }

inline bool plan(const ConvGeom &a, bool bf16, int slots, const Layout &w, SplitShape &s)
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
    bool zero_ends = true;
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
                // GY[-1 - sc] and GY[8 NU - sc] are outside the row
                zero_ends = zero_ends && (vl == 1 || (sc >= 0 && 8 * s.NU - sc >= s.Wo));
            }
        }
    }
    s.gl = zero_ends ? s.NU : s.NU + 2;
    s.gp = zero_ends ? s.NU + 1 : s.NU + 2;
    s.inv_gl = (65536 + s.gl - 1) / s.gl;
    s.full = s.kh == 3 && s.kw == 3 && s.sw == 1;
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
        const int64_t nx = (int64_t)32 * w.wi * xr * s.NU, ng = (int64_t)32 * w.wo * rc * s.gl;
        if ((int64_t)xr * s.NU * nx >= (1 << 20) || (int64_t)rc * s.gl * ng >= (1 << 20)) continue;   // div20
        // an odd number of units leaves one step a unit past the chunk: it reads
        // X at row (rc - 1) * sh + 2 + sh (any finite value) and GY's two units
        // from rc * gp + 1 on (zeros)
        const int csx = odd_units(((xr + s.sh - 1) * s.NU + 1) * 16), csg = odd_units((rc * s.gp + 3) * 16);
        const int px = 32 * w.wi * csx, pg = 32 * w.wo * csg;
        const int64_t total = (int64_t)np * (px + pg) + (covers ? 4 * ng : 0);
        if (total > (int64_t)kLds) continue;
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
inline double cost_of(const SplitShape &s, const Layout &w, int64_t N, bool bf16)
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

// A plan's time in us, for comparison with the kernels it may replace; rounds:
// of its grid over the CUs (cu_rounds), per CU: workgroups one after the other.
// Fitted to 3300 drawn layers (8% rms for fp32, 14% for bf16): a fixed part,
// the stores (single words of every tap per lane, each its own cache line,
// unless whole rows of 3 x 3 taps go through LDS), and per chunk the round trips
// of its loads (two units per thread each), its units, and its steps with
// their MFMAs.
inline double split_us(const SplitShape &s, const Layout &w, bool bf16, double rounds, double per_cu)
{
    const int chunks = (s.Ho + s.RC - 1) / s.RC, steps = ((s.RC * s.NU + 1) / 2 + w.wk - 1) / w.wk;
    const int trips = (s.nx + 511) / 512 + (s.ng + 511) / 512, units = (s.nx + 255) / 256 + (s.ng + 255) / 256;
    const double taps = (double)s.khw / s.ngrp, blocks = w.wi * w.wo;
    const double store = s.full ? (bf16 ? 2.2 : 2.1) : (bf16 ? 0.51 : 0.49) * s.gpw * taps;
    const double chunk = bf16 ? 1.8 + 0.78 * trips + 0.076 * units + 0.0085 * steps * (taps + 8)
                              : 0.5 + 1.8 * trips + 0.16 * units + 0.012 * steps * (6 * taps + 8);
    return (bf16 ? 9.5 : 11.6) + per_cu * blocks * store + rounds * s.gpw * chunks * chunk;
}

inline bool choose(const ConvGeom &a, bool bf16, int slots, SplitShape &best, int &which)
{
    // 32-bit offsets, taps in eight bits, and the quotients of inv_nu and div20
    if (a.kh > 100 || a.kw > 100 || a.W > 2048 || a.Cin * a.H * a.W >= (int64_t(1) << 28) ||
        a.Cout * a.Ho * a.Wo >= (int64_t(1) << 28) || a.Cin * a.kh * a.kw * a.Cout >= (int64_t(1) << 30) || a.ph > a.H + a.kh ||
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

}  // namespace csplit
}  // namespace dpg
