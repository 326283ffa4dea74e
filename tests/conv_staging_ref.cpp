// The staging and the index arithmetic of the bf16-matrix Conv2d kernel
// (csrc/conv2d_split_plan.hpp) run on the CPU with whole numbers, against the
// definition of the per-sample gradient.  One line per geometry that differs;
// the last line counts them.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "conv2d_split_plan.hpp"

using namespace dpg::csplit;

static int value(int i) { return 1 + (int)(((uint32_t)i * 2654435761u) >> 16) % 97; }

struct Tensor {
    std::vector<int> v;
    explicit Tensor(size_t n, int seed) : v(n)
    {
        for (size_t i = 0; i < n; ++i) v[i] = value((int)i + seed);
    }
    int at(int64_t o) const { return o >= 0 && o < (int64_t)v.size() ? v[o] : 0; }   // a buffer load
};

// a plane of LDS (element pairs of 16-byte units as eight whole numbers); every access in bounds
struct Plane {
    std::vector<int> v;
    bool ok = true;
    explicit Plane(int bytes) : v(bytes / 2, 0) {}
    int get(int byte, int k)
    {
        const int i = byte / 2 + k;
        if (i < 0 || i >= (int)v.size()) {
            ok = false;
            return 0;
        }
        return v[i];
    }
    void put(int byte, const int *u)
    {
        for (int k = 0; k < 8; ++k) {
            if (byte % 16 || byte / 2 + k >= (int)v.size()) ok = false;
            else v[byte / 2 + k] = u[k];
        }
    }
};

static void stage(Plane &L, const Tensor &src, const UnitAt &a, int step, bool clip, int n, long long *bias)
{
    int u[8];
    for (int k = 0; k < 8; ++k) {
        u[k] = a.dead ? 0 : src.at((int64_t)a.e + k * step);
        if (clip && !(a.col + k * step >= 0 && a.col + k * step < n)) u[k] = 0;
        if (bias && a.at >= 0) *bias += u[k];
    }
    if (a.at >= 0) L.put(a.at, u);
}

// whether the plan's gradients and bias sums are those of the definition
static bool check(const ConvGeom &g, const SplitShape &s, const Layout &w)
{
    const int ci_n = (int)g.Cin, co_n = (int)g.Cout, kh = (int)g.kh, kw = (int)g.kw;
    const Tensor X(g.Cin * g.H * g.W, 1), GY(g.Cout * g.Ho * g.Wo, 12345);
    std::vector<long long> got((size_t)co_n * ci_n * kh * kw, 0), bias(co_n, 0);
    std::vector<int> seen(kh * kw, 0);
    Plane LX(s.px), LG(s.pg);
    for (int gi = 0; gi < s.ngrp; ++gi) {
        const ConvGroup &q = s.g[gi];
        std::fill(LX.v.begin(), LX.v.end(), 0);
        std::fill(LG.v.begin(), LG.v.end(), 0);
        for (int oh0 = 0; oh0 < s.Ho; oh0 += s.RC) {
            for (int i = 0; i < s.nx; ++i)
                stage(LX, X, x_unit(s, q.u0, q.phase, 0, oh0, i), s.sw, clips_x(s), s.W, nullptr);
            for (int i = 0; i < s.ng; ++i) {
                const int c = i / (s.RC * s.gl);
                stage(LG, GY, g_unit(s, q.sc, 0, oh0, i), 1, clips_g(s, q.sc), s.Wo,
                      s.bias_at && gi == 0 && c < co_n ? &bias[c] : nullptr);
            }
            const int rows = s.Ho - oh0 < s.RC ? s.Ho - oh0 : s.RC, steps = (rows * s.NU + 1) / 2;
            for (int U = 0; U < 2 * steps; ++U) {
                const int r = (U * s.inv_nu) >> 16, cu = U - r * s.NU;
                for (int co = 0; co < co_n; ++co)
                    for (int ci = 0; ci < ci_n; ++ci)
                        for (int u = 0; u < q.ul; ++u)
                            for (int v = 0; v < q.vl; ++v) {       // columns vc, vc + sw, vc - sw
                                const int col = q.vc + (v == 0 ? 0 : v == 1 ? s.sw : -s.sw), shift = v == 0 ? 0 : v == 1 ? -1 : 1;
                                long long t = 0;
                                for (int k = 0; k < 8; ++k)
                                    t += (long long)LX.get(ci * s.csx + ((r * s.sh + u) * s.NU + cu) * 16, k) *
                                         LG.get(co * s.csg + (r * s.gp + 1 + cu) * 16, k + shift);
                                got[(((size_t)co * ci_n + ci) * kh + q.u0 + u) * kw + col] += t;
                            }
            }
        }
        for (int u = 0; u < q.ul; ++u)
            for (int v = 0; v < q.vl; ++v) ++seen[(q.u0 + u) * kw + q.vc + (v == 0 ? 0 : v == 1 ? s.sw : -s.sw)];
    }
    bool ok = LX.ok && LG.ok;
    for (int t : seen) ok = ok && t == 1;
    for (int co = 0; co < co_n; ++co) {
        long long sum = 0;
        for (int p = 0; p < s.Ho * s.Wo; ++p) sum += GY.v[co * s.Ho * s.Wo + p];
        ok = ok && (!s.bias_at || bias[co] == sum);
        for (int ci = 0; ci < ci_n; ++ci)
            for (int u = 0; u < kh; ++u)
                for (int v = 0; v < kw; ++v) {
                    long long t = 0;
                    for (int oh = 0; oh < s.Ho; ++oh) {
                        const int ih = oh * s.sh + u - s.ph;
                        if (ih < 0 || ih >= s.H) continue;
                        for (int ow = 0; ow < s.Wo; ++ow) {
                            const int iw = ow * s.sw + v - s.pw;
                            if (iw >= 0 && iw < s.W)
                                t += (long long)GY.v[(co * s.Ho + oh) * s.Wo + ow] * X.v[(ci * s.H + ih) * s.W + iw];
                        }
                    }
                    ok = ok && t == got[(((size_t)co * ci_n + ci) * kh + u) * kw + v];
                }
    }
    // the addresses that channels past the layer use lie in the planes too
    ok = ok && (32 * w.wi - 1) * s.csx + (((s.RC * s.NU - 1) / s.NU * s.sh + s.XR - (s.RC - 1) * s.sh) * s.NU) * 16 <= s.px;
    return ok;
}

int main()
{
    int plans = 0, bad = 0;
    for (int kh = 1; kh <= 9; ++kh)
        for (int kw = kh == 1 ? 2 : kh; kw <= (kh == 3 ? 6 : kh == 1 ? 2 : kh); ++kw)
            for (int st = 1; st <= 3; ++st)
                for (int p = 0; p < kw; ++p)
                    for (int W = 6; W <= 40; ++W) {
                        const int H = 6 + (W * 7 + kw) % 13, sh = (W + st) % 5 == 0 ? 1 : st;
                        if (H + 2 * p < kh || W + 2 * p < kw) continue;
                        const ConvGeom g = {4, 2, H, W, 2, (H + 2 * p - kh) / sh + 1, (W + 2 * p - kw) / st + 1, kh, kw, sh, st,
                                            p, p};
                        for (int t = 0; t < 2; ++t) {              // fp32 and bf16, the layouts in turn
                            const int at = (W + p + t) % 3, slots = 1 + (W + st) % 4;
                            SplitShape s;
                            if (!plan(g, t == 1, slots, kLayouts[at], s)) continue;
                            ++plans;
                            if (!check(g, s, kLayouts[at])) {
                                ++bad;
                                std::printf("%s kernel %dx%d stride %d,%d pad %d input %dx%d layout %d\n", t ? "bf16" : "f32",
                                            kh, kw, sh, st, p, H, W, at);
                            }
                        }
                    }
    std::printf("%d of %d plans differ\n", bad, plans);
    return bad != 0;
}
