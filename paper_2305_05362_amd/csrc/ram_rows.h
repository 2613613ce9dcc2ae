// ram_rows.h -- a wave's tile of a row that has its own mesh: its source
// window, every shifted node's source cell in it, and their Lagrange weights
// (the per-row step kernel and the per-row streaming plan).
#pragma once

#include "ram_wave.h"

namespace ram {
namespace dev {

// A tile's source window: extended index of its first cell, the period it lies
// in, the length its end nodes give it, its length here, first cell within the
// row, window index of the first node of the next period and of the one after (a
// window as long as its row crosses the row's end twice).
struct RowsWindow {
    int64_t wlo, k0, wide;
    int w, base, seam, seam2;
    __device__ __forceinline__ int period(int j) const { return (j >= seam ? 1 : 0) + (j >= seam2 ? 1 : 0); }
    // row index of window cell or node j (a node past the last period's end: n)
    __device__ __forceinline__ int at(int j, int n) const
    {
        const int m = base + j;
        return m >= 2 * n ? m - 2 * n : (m >= n ? m - n : m);
    }
};

// Brackets of the cells that hold two coordinates at once (lanes 0 to 31 search
// for xa, the others for xb): x[lo] <= xh, or lo 0, and x[hi] > xh, or hi n, at
// most kBracket apart.  32 nodes a side a load, so two loads deep on rows of
// 8192 cells where a binary search is thirteen.  (At least one load: on a row of a
// few cells the brackets would be all of it, and the window too long for it.)
constexpr int kBracket = 8;
__device__ __forceinline__ void find_two(const double *x, int n, double xa, double xb, int t, int &la,
                                         int &hb)
{
    const bool hi_half = t >= 32;
    const double target = hi_half ? xb : xa;
    const double inf = __builtin_huge_val();
    int lo = 0, hi = n;
    do {
        const int step = max((hi - lo + 31) / 32, 1);
        const int at = lo + (t & 31) * step;
        const uint64_t m = __ballot((at < hi ? x[at] : inf) <= target);
        const int k = __popc((uint32_t)(hi_half ? m >> 32 : m));
        lo = min(lo + max(k - 1, 0) * step, n - 1);
        hi = min(hi, lo + step);
    } while (__any(hi - lo > kBracket ? 1 : 0));
    la = __shfl(lo, 0);
    hb = __shfl(max(hi, lo + 1), 32);
}

// The row's shift v0 dt, rounded as the definition has it (a multiply-add of
// x - v0 dt would round a shift of many periods differently, by more than the
// FP64 error bound of a small cell).
__device__ __forceinline__ double rows_shift(double v0, double dt)
{
#pragma clang fp contract(off)
    return v0 * dt;
}

// Node x - s wrapped into the period: coordinate in [x0, xN) and the period it
// came from, as shifted_node_inv forms them.
__device__ __forceinline__ void wrap_node(double xe, double s, double x0, double xN, double len,
                                          double invlen, double &xh, int64_t &k)
{
    const double xt = xe - s;
    const double kf = floor((xt - x0) * invlen);
    xh = xt - kf * len;
    k = (int64_t)kf;
    if (xh >= xN) { xh -= len; k += 1; }
    else if (xh < x0) { xh += len; k -= 1; }
}

// The last node at or below each xh among window nodes xs[0 .. W], within period
// dk of the window (0, 1 or 2).
template <int NS>
__device__ __forceinline__ void rows_search(const double *xs, const RowsWindow &win, int W,
                                            const double (&xh)[NS], const int (&dk)[NS], int (&j)[NS])
{
    int end[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        j[u] = dk[u] == 0 ? 0 : min(dk[u] == 1 ? win.seam : win.seam2, W);
        end[u] = min(dk[u] == 0 ? win.seam : (dk[u] == 1 ? win.seam2 : W + 1), W + 1);
    }
    int top = 1;
    while (2 * top <= W) top *= 2;
    for (int step = top; step > 0; step >>= 1) {
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int at = j[u] + step;
            if (at < end[u] && xs[min(at, W)] <= xh[u]) j[u] = at;
        }
    }
}

// The tile's window and its nodes' cells.  Nodes e0 .. e0 + NE - 1 of the row
// (e0 may be a few below 0, the last a few past n), node m = t + 64 u in slot u
// of lane t (slots past the last repeat it), given as their unshifted
// coordinates xe and the periods kx they were wrapped by.  The window runs from
// the first node's stencil (or a few cells before) to the last one's (or a few
// after); its nodes (coordinates as stored,
// the row's first again past its end) go to xs[0 .. w].  Returns whether the
// window holds at most `cap` cells, crosses the row's end at most twice and
// holds every node's stencil; then j is each node's window cell and xh its
// wrapped coordinate.  The wave locates the two end nodes in the row, then
// every node among the window's in LDS: the row is read once, in whole lines,
// where a binary search a node reads thirteen lines a lane.
// `issue` is called once the window is known (its loads are on their way during
// the search).
template <int P, int NS, class Issue>
__device__ __forceinline__ bool rows_locate(const double *x, int n, double s, double x0, double xN,
                                            double len, double invlen, int NE, int t, int cap,
                                            const double (&xe)[NS], const int (&kx)[NS], double *xs,
                                            RowsWindow &win, double (&xh)[NS], int (&j)[NS],
                                            Issue issue)
{
    constexpr int LO = (P - 1) / 2;
    int64_t k[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        wrap_node(xe[u], s, x0, xN, len, invlen, xh[u], k[u]);
        k[u] += kx[u];
    }
    // the end nodes: node 0 in lane 0's first slot, node NE - 1 where it falls
    double xl = xh[0];
    int64_t kl = k[0];
#pragma unroll
    for (int u = 0; u < NS; ++u)
        if (u == (NE - 1) / kLanes) {
            xl = xh[u];
            kl = k[u];
        }
    const int last = (NE - 1) % kLanes;
    const double xa = __shfl(xh[0], 0), xb = __shfl(xl, last);
    int la, hb;
    find_two(x, n, xa, xb, t, la, hb);
    const int64_t ka = __shfl(k[0], 0);
    const int64_t ga = (int64_t)la + ka * (int64_t)n;
    const int64_t gb = (int64_t)(hb - 1) + __shfl(kl, last) * (int64_t)n;
    const int64_t wide = gb - ga + P;
    win.wide = wide;
    win.wlo = ga - LO;
    // (rows have more than LO cells)
    win.k0 = ka - (la < LO ? 1 : 0);
    win.base = la < LO ? la - LO + n : la - LO;
    win.seam = n - win.base;
    win.seam2 = win.seam + n;
    win.w = 0;
    if (wide < P || wide > cap || win.base + wide > 3 * (int64_t)n) return false;
    const int W = (int)wide;
    win.w = W;
    constexpr int NX = 4;                            // nodes a lane has in flight
    for (int i0 = t; i0 - t <= W; i0 += NX * kLanes) {
        double v[NX];
#pragma unroll
        for (int u = 0; u < NX; ++u) v[u] = x[win.at(min(i0 + u * kLanes, W), n)];
#pragma unroll
        for (int u = 0; u < NX; ++u) xs[min(i0 + u * kLanes, W)] = v[u];
    }
    issue();
    wave_sync();
    bool ok = true;
    int dk[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int64_t d = k[u] - win.k0;
        ok = ok && d >= 0 && d <= 2;
        dk[u] = (int)d;
    }
    rows_search<NS>(xs, win, W, xh, dk, j);
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        ok = ok && j[u] >= LO && j[u] + P - LO <= W && xs[j[u]] <= xh[u];
    }
    return __all(ok ? 1 : 0) != 0;
}

// Lagrange weights of the node at xh in window cell j, in WT: of every stencil
// node but the cell's own left one (w[LO] is not formed: no partial integral
// uses it), from the nodes' positions in units of the cell's size, the cell's
// own edges at 0 and 1.  The products of the node's distances from the front
// and from the back, each weight's denominator from the pairwise distances; a
// denominator past the type's largest number (in FP32 at order 5 from neighbours
// 2e7 times the cell) leaves a weight of 0.
// SEAM: the window crosses the row's end.
template <typename WT, int P, bool SEAM>
__device__ __forceinline__ void rows_weights(const double *xs, const RowsWindow &win, double len,
                                             double xh, int j, WT *w)
{
    constexpr int LO = (P - 1) / 2;
    const double xc = xs[j];
    const int kc = SEAM ? win.period(j) : 0;
    auto dist = [&](int b) {
        const int jb = j - LO + b;
        const double d = xs[jb] - xc;
        return SEAM ? d + (double)(win.period(jb) - kc) * len : d;
    };
    WT th[P + 1], tt;
    const double inv = 1.0 / dist(LO + 1);
#pragma unroll
    for (int b = 0; b <= P; ++b)
        if (b != LO && b != LO + 1) th[b] = (WT)(dist(b) * inv);
    tt = (WT)((xh - xc) * inv);
    th[LO] = (WT)0;
    th[LO + 1] = (WT)1;
    WT d[P + 1], pre[P + 1], suf[P + 1];
#pragma unroll
    for (int b = 0; b <= P; ++b) d[b] = tt - th[b];
    pre[0] = (WT)1;
#pragma unroll
    for (int b = 1; b <= P; ++b) pre[b] = pre[b - 1] * d[b - 1];
    suf[P] = (WT)1;
#pragma unroll
    for (int b = P - 1; b >= 0; --b) suf[b] = suf[b + 1] * d[b + 1];
    // th increases, so a < b gives th[b] - th[a] > 0; the denominator of a has
    // one sign change for every node above it
    WT den[P + 1];
#pragma unroll
    for (int b = 0; b <= P; ++b) den[b] = (WT)1;
#pragma unroll
    for (int x = 0; x <= P; ++x)
#pragma unroll
        for (int y = x + 1; y <= P; ++y) {
            const WT g = th[y] - th[x];
            if (x != LO) den[x] *= g;
            if (y != LO) den[y] *= g;
        }
#pragma unroll
    for (int b = 0; b <= P; ++b) {
        if (b == LO) continue;
        const WT num = (P - b) % 2 ? -(pre[b] * suf[b]) : pre[b] * suf[b];
        w[b] = num / den[b];
    }
    w[LO] = (WT)0;
}

// The exclusive cumulative (sp[0 .. W]) of a window's masses (sm[0 .. W), in
// LDS): W / 64 consecutive cells a lane, the lanes' sums scanned across the
// wave in DPP steps
// once.
template <int S>
__device__ __forceinline__ void rows_prefix(typename Acc<S>::A *sp, const typename Acc<S>::M *sm, int W,
                                            int t)
{
    using AC = Acc<S>;
    using A = typename AC::A;
    const int per = (W + kLanes - 1) / kLanes;
    const int j0 = t * per;
    A tot = AC::zero();
    for (int k = 0; k < per; ++k)
        if (j0 + k < W) tot = AC::add(tot, sm[j0 + k]);
    const A inc = wave_inclusive<AC>(tot);
    A e = AC::template dpp<kDppWaveShr1, 0xf, 0xf>(inc);
    if (t == 0) e = AC::zero();
    for (int k = 0; k < per; ++k) {
        if (j0 + k >= W) break;
        sp[j0 + k] = e;
        e = AC::add(e, sm[j0 + k]);
        if (j0 + k == W - 1) sp[W] = e;
    }
}

// Size of window cell j.
__device__ __forceinline__ double rows_size(const double *xs, const RowsWindow &win, double xN, int j)
{
    return (j + 1 == win.seam || j + 1 == win.seam2 ? xN : xs[j + 1]) - xs[j];
}

} // namespace dev
} // namespace ram
