// ram_node64.h -- a planned node: its wrapped coordinate, its FP64 position in
// its source cell and the cell's Lagrange stencil (the FP64 streaming step and
// the tile adjoint).
#pragma once

#include "ram_device.h"
#include "ram_wave.h"

namespace ram {
namespace dev {

// Offsets th_b (units of dx_c) and reciprocal denominators rd_b of source cell
// c's P + 1 nodes, from the mesh's FP64 stencil planes (pairs 1 .. P of stpd:
// the offsets other than the cell's own edges, 0 and 1, then the denominators
// other than the own node's, whose weight no partial integral uses).
// Neighbouring lanes read neighbouring cells' pairs: 16 bytes a lane a load.
template <int P>
__device__ __forceinline__ void node_stencil(const double2 *stpd, int n, int c,
                                             double (&rth)[P + 1], double (&rrd)[P + 1])
{
    constexpr int LO = (P - 1) / 2;
    double v[2 * P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const double2 pr = stpd[(k + 1) * n + c];
        v[2 * k] = pr.x;
        v[2 * k + 1] = pr.y;
    }
    int k = 0;
#pragma unroll
    for (int b = 0; b <= P; ++b) rth[b] = b == LO ? 0.0 : (b == LO + 1 ? 1.0 : v[k++]);
#pragma unroll
    for (int b = 0; b <= P; ++b) rrd[b] = b == LO ? 0.0 : v[k++];
}

// Reciprocal Lagrange denominator of node a among P+1 equally spaced nodes.
template <int P>
__host__ __device__ constexpr double eq_denominator_inv(int a)
{
    double d = 1.0;
    for (int b = 0; b <= P; ++b)
        if (b != a) d *= (double)(a - b);
    return 1.0 / d;
}

// The same for a cell of a uniform run, from the FP32 deviations of its
// offsets and denominators from those of equally spaced nodes (stdv: float4,
// float4, float planes): 36 bytes a node instead of 80.
template <int P>
__device__ __forceinline__ void node_stencil_uni(const float *stdv, int n, int c,
                                                 double (&rth)[P + 1], double (&rrd)[P + 1])
{
    constexpr int LO = (P - 1) / 2;
    float v[12];
    const float4 A = ((const float4 *)stdv)[c];
    v[0] = A.x; v[1] = A.y; v[2] = A.z; v[3] = A.w;
    if constexpr (2 * P - 1 > 4) {
        const float4 B = ((const float4 *)stdv)[n + c];
        v[4] = B.x; v[5] = B.y; v[6] = B.z; v[7] = B.w;
    }
    if constexpr (2 * P - 1 > 8) v[8] = stdv[8 * n + c];
    int k = 0;
#pragma unroll
    for (int b = 0; b <= P; ++b)
        rth[b] = b == LO ? 0.0 : (b == LO + 1 ? 1.0 : (double)(b - LO) + (double)v[k++]);
#pragma unroll
    for (int b = 0; b <= P; ++b)
        rrd[b] = b == LO ? 0.0 : eq_denominator_inv<P>(b) * (1.0 + (double)v[k++]);
}

// The FP32 stencil of cell c (stp: float4, float4, float planes).
template <int P>
__device__ __forceinline__ void node_stencil(const float *stp, int n, int c, float (&rth)[P + 1],
                                             float (&rrd)[P + 1])
{
    constexpr int LO = (P - 1) / 2;
    float v[12];
    const float4 A = ((const float4 *)stp)[c];
    v[0] = A.x; v[1] = A.y; v[2] = A.z; v[3] = A.w;
    if constexpr (2 * P - 1 > 4) {
        const float4 B = ((const float4 *)stp)[n + c];
        v[4] = B.x; v[5] = B.y; v[6] = B.z; v[7] = B.w;
    }
    if constexpr (2 * P - 1 > 8) v[8] = stp[8 * n + c];
    int k = 0;
#pragma unroll
    for (int b = 0; b <= P; ++b) rth[b] = b == LO ? 0.0f : (b == LO + 1 ? 1.0f : v[k++]);
#pragma unroll
    for (int b = 0; b <= P; ++b) rrd[b] = b == LO ? 0.0f : v[k++];
}

// Lagrange weights of the cumulative at theta, as prefix and suffix products
// of (theta - th_b).
template <int P, typename WT>
__device__ __forceinline__ void node_weights(const WT (&rth)[P + 1], const WT (&rrd)[P + 1], WT th,
                                             WT (&wk)[P + 1])
{
    WT tt[P + 1], pre[P + 1], suf[P + 1];
#pragma unroll
    for (int b = 0; b <= P; ++b) tt[b] = th - rth[b];
    pre[0] = (WT)1;
#pragma unroll
    for (int b = 1; b <= P; ++b) pre[b] = pre[b - 1] * tt[b - 1];
    suf[P] = (WT)1;
#pragma unroll
    for (int b = P - 1; b >= 0; --b) suf[b] = suf[b + 1] * tt[b + 1];
#pragma unroll
    for (int b = 0; b <= P; ++b) wk[b] = rrd[b] * (pre[b] * suf[b]);
}

// The weights' derivatives with respect to theta (the product rule carried
// through the prefix and suffix products).
template <int P, typename WT>
__device__ __forceinline__ void node_dweights(const WT (&rth)[P + 1], const WT (&rrd)[P + 1], WT th,
                                              WT (&dw)[P + 1])
{
    WT tt[P + 1], pre[P + 1], suf[P + 1], dpre[P + 1], dsuf[P + 1];
#pragma unroll
    for (int b = 0; b <= P; ++b) tt[b] = th - rth[b];
    pre[0] = (WT)1;
    dpre[0] = (WT)0;
#pragma unroll
    for (int b = 1; b <= P; ++b) {
        pre[b] = pre[b - 1] * tt[b - 1];
        dpre[b] = dpre[b - 1] * tt[b - 1] + pre[b - 1];
    }
    suf[P] = (WT)1;
    dsuf[P] = (WT)0;
#pragma unroll
    for (int b = P - 1; b >= 0; --b) {
        suf[b] = suf[b + 1] * tt[b + 1];
        dsuf[b] = dsuf[b + 1] * tt[b + 1] + suf[b + 1];
    }
#pragma unroll
    for (int b = 0; b <= P; ++b) dw[b] = rrd[b] * (dpre[b] * suf[b] + pre[b] * dsuf[b]);
}

// The source cells of nodes e0 + min(t + 64 s, NE - 1) (s = 0 .. NS - 1, lane t)
// of a row: the wrapped coordinate xt, the cell ce that holds it (bucket index,
// Eq. condition_p) and the cells to add for the periods between them, kx, beside
// rs.kf0 periods.  Each load of all the lane's nodes before the next one's.
template <int NS>
__device__ __forceinline__ void locate_nodes(const double *x, int n, const MeshTab &tb,
                                             const RowShift &rs, double x0, double xN, int e0, int NE,
                                             int t, int (&ce)[NS], int (&kx)[NS], double (&xt)[NS])
{
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int en = e0 + min(t + s * 64, NE - 1);
        kx[s] = en < 0 ? -n : (en >= n ? n : 0);
        xt[s] = x[en - kx[s]];
    }
    double2 nx[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const NodePos np = node_pos_same(xt[s], rs, x0, xN, tb.scal[0], tb.scal[2], tb.nb);
        ce[s] = tb.bucket[np.b];
        nx[s] = tb.bnext[np.b];
        xt[s] = np.xt;
        kx[s] += np.dk * n;
    }
    bool walk = false;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        ce[s] = cell_from_bucket(ce[s], nx[s], xt[s]);
        walk = walk || xt[s] >= nx[s].y;
    }
    if (__any(walk ? 1 : 0)) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (xt[s] >= nx[s].y) ce[s] = cell_walk(x, n, ce[s], xt[s]);
    }
}

// The window indices of a tile's nodes (extended cells ce + kx) in its window, and
// whether they hold every node's stencil (not expected otherwise: the record sized
// the window from the end nodes, and on increasing nodes the ones between lie
// between; a tile whose nodes do not goes the way of a window beyond the LDS, as
// the plan sends it).
template <int P, int NS>
__device__ __forceinline__ bool window_indices(const int (&ce)[NS], const int (&kx)[NS], const RowShift &rs,
                                               int n, const FastTile &ft, int (&j)[NS])
{
    constexpr int LO = (P - 1) / 2;
    const int64_t wlo = (int64_t)(((uint64_t)(uint32_t)ft.wlo_hi << 32) | (uint32_t)ft.wlo_lo);
    const int jbase = (int)(rs.kf0 * (int64_t)n - wlo);
    bool ok = true;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        j[u] = ce[u] + kx[u] + jbase;
        ok = ok && j[u] >= LO && j[u] + P - LO <= ft.w;
    }
    return __all(ok ? 1 : 0) != 0;
}

// Position in cell c (pair 0 of stpd: its left edge and 1/dx) of a node at
// xt.  A uniform tile's node may lie in its window by counting and beside c by
// the mesh's rounding, also across the period's seam (near: taken there; its
// cells are far smaller than half the period).  A planned node's cell holds xt,
// whatever the cell's size.  Not contracted, as node_wrap: theta is the same in
// every kernel, whatever it goes on to.
__device__ __forceinline__ double cell_theta(const double2 *stpd, int c, double xt, double len,
                                             bool near)
{
#pragma clang fp contract(off)
    const double2 g = stpd[c];
    double d = xt - g.x;
    if (near) d = d > 0.5 * len ? d - len : (d < -0.5 * len ? d + len : d);
    return d * g.y;
}

// The record of a tile (H halo cells a side): which path, its window, and for a
// tile in a uniform run the stencil and the run's geometry.  Two neighbouring
// lanes a tile, one for either end node (bucket index, Eq. condition_p), which
// then look the tile's cells and its window up in one run count each (coarse
// and fine); the even lane's record counts.
//
// uniform: the cells on both sides of the tile's nodes and its whole source
// window lie in one uniform run of the mesh, and the window holds one source
// cell per node plus the stencil, so node i0 - H + k sits in window cell LO + k
// at the first node's theta (rows shorter than a full tile's window stay with
// the other kernel, whose windows may wrap many times).
template <int P>
__device__ __forceinline__ FastTile plan_tile(const StepArgs &a, int tile, int H, int t)
{
    constexpr int LO = (P - 1) / 2;
    const Rows &R = a.rows;
    const MeshTab &tb = R.tab;
    const int n = (int)R.n_cols;
    const double *x = R.edges;
    const TilePos p = tile_pos(tile, n, H);
    const int i0 = p.i0, nd = p.nd;
    const RowShift rs = row_shift(a.v0[p.row] * a.dt, x[n] - x[0], tb.scal[1]);
    double xt;
    int c;
    const int64_t g = node_locate<true>(x, n, tb, rs, (t & 1) ? i0 + nd + H : i0 - H, xt, c);
    const int64_t g0 = __shfl(g, t & ~1), g1 = __shfl(g, t | 1);
    const int c0 = __shfl(c, t & ~1);
    const int64_t wide = g1 - g0 + P;
    const int64_t wlo = g0 - LO;
    const bool fits = wide >= P && wide <= kFastWin;
    int base = c0 - LO;
    while (base < 0) base += n;
    bool run = false;
    if (fits && tb.nonu && wide == nd + 2 * H + P && n >= kFastTile + 2 * H + P) {
        const int32_t *pre = (t & 1) ? tb.nonu_min : tb.nonu;
        const int all = pre[n];
        // cells of no run before cell i of the row and its neighbouring periods
        auto upto = [&](int i) {
            int k = 0;
            if (i < 0) { i += n; k = -all; }
            while (i >= n) { i -= n; k += all; }
            return k + pre[i];
        };
        run = upto(i0 + nd + H + 1) == upto(i0 - H - 1) && upto(base + (int)wide) == upto(base);
    }
    const int other = __shfl_xor(run ? 1 : 0, 1);
    const bool uni = run || other != 0;
    FastTile ft;
    ft.kind = uni ? kFastUniform : (fits ? kFastWindow : kFastDirect);
    ft.w = fits ? (int)wide : -1;
    ft.base = base;
    ft.wlo_lo = (int32_t)(uint32_t)((uint64_t)wlo & 0xffffffffull);
    ft.wlo_hi = (int32_t)((uint64_t)wlo >> 32);
    for (int d = 0; d < 6; ++d) ft.cc[d] = 0.0f;
    ft.dx = ft.hinv = ft.dxinv = 0.0f;
    ft.pad[0] = ft.pad[1] = tile;
    if (uni) {
        double th;
        {
#pragma clang fp contract(off)
            th = (xt - x[c]) * tb.dxinv[c];
        }
        double cc[P + 1];
        uniform_stencil<double, P>(th, cc);
        for (int d = 0; d <= P; ++d) ft.cc[d] = (float)cc[d];
        ft.pad[1] = __float_as_int((float)th);
        const float2 rr = tb.rrf[i0];
        ft.dx = rr.x;
        ft.hinv = rr.y;
        ft.dxinv = tb.dxinvf[i0];
    }
    return ft;
}

// The same by a wave for its own tile, every field in scalar registers.
template <int P>
__device__ __forceinline__ FastTile plan_wave(const StepArgs &a, int tile, int H, int t)
{
    FastTile ft = plan_tile<P>(a, tile, H, t);
    int32_t *w = (int32_t *)&ft;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(FastTile) / 4); ++k) w[k] = __builtin_amdgcn_readfirstlane(w[k]);
    return ft;
}

// Each node's window index and FP64 position in its cell, for a tile whose
// window fits: a uniform tile's by counting, another's from the call's node
// plan, or located here where the call has none (one step: the plan's launch
// costs more than the search: one FP64 step of a row of 256 cells 17 us
// against 20, an FP32 step back over 24,000 searching tiles 131 against 157).  wcell: window
// index -> cell of the row.  False: a node located here is not in the window.
template <int P, int NS, bool PLAN, class Cell>
__device__ __forceinline__ bool tile_nodes(const FastPlan &pl, const FastTile &ft, const double *x,
                                           int n, const MeshTab &tb, const RowShift &rs, double x0,
                                           double xN, int e0, int NE, Cell wcell, int t,
                                           int (&jv)[NS], double (&thv)[NS])
{
    constexpr int LO = (P - 1) / 2;
    const bool uniform = ft.kind == kFastUniform;
    const double len = xN - x0;
    if (!PLAN && !uniform) {
        int ce[NS], kx[NS];
        double xt[NS];
        locate_nodes<NS>(x, n, tb, rs, x0, xN, e0, NE, t, ce, kx, xt);
#pragma unroll
        for (int u = 0; u < NS; ++u) thv[u] = cell_theta(tb.stpd, ce[u], xt[u], len, false);
        return window_indices<P, NS>(ce, kx, rs, n, ft, jv);
    }
    const int16_t *jcp = uniform ? nullptr : pl.jc + (int64_t)ft.pad[1] * kFastNodes;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int m = min(t + u * 64, NE - 1);
        int e = e0 + m;
        e = e < 0 ? e + n : (e >= n ? e - n : e);
        int dk;
        const double xt = node_wrap(x[e], rs, x0, xN, dk);
        int j = jcp ? (int)jcp[m] : LO + m;
        int c = wcell(j);
        double th = cell_theta(tb.stpd, c, xt, len, uniform);
        // a uniform tile's inner node that the mesh's rounding puts in a
        // neighbouring cell (the end nodes' cells came from the search)
        if (!jcp && m > 0 && m < NE - 1 && (th < 0.0 || th >= 1.0)) {
            j += th < 0.0 ? -1 : 1;
            c = wcell(j);
            th = cell_theta(tb.stpd, c, xt, len, uniform);
        }
        jv[u] = j;
        thv[u] = th;
    }
    return true;
}

} // namespace dev
} // namespace ram
