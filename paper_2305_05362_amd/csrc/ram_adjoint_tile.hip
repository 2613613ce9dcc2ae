// ram_adjoint_tile.hip -- one RAM step backwards on rows that share a mesh, one
// tile of kFastTile destination cells a wave, for the states the FP32
// streaming adjoint does not take: FP64, and FP32 rows whose length is not a
// multiple of four cells or whose arrays are not 16-byte aligned.
//
// The algebra is that of the streaming adjoint, on the same tile plan
// (k_plan_fast, no halo); what differs:
//   * every array is read and written one cell a lane, so nothing depends on
//     alignment;
//   * the residual's transpose runs in the state's type on four consecutive
//     cells a lane, its six arrays passed through the wave's LDS in two turns
//     of three;
//   * no stencil shortcut on uniform runs in FP64 (a run counts as uniform far
//     above FP64 rounding): every node's weights are formed in the state's type from
//     its FP64 position and its source cell's stencil, and a uniform tile only
//     saves the node plan;
//   * the shift's transpose follows the forward sum term by term.  Cell i's
//     mass is its whole source cells plus ell_{i+1} - ell_i, ell_e a fixed
//     combination of the p source cells around node e; so each whole cell
//     gets Mbar'_i, and each node adds Vbar_e = Mbar'_{e-1} - Mbar'_e times
//     its p coefficients to the window cells around it.  No scan, and no
//     weight of a node's own cumulative to cancel.  The nodes of one LDS
//     instruction add to different cells: nodes that share a source cell go in
//     turns, by their rank among them, so the sum is the same in every run.
//     v0bar's pass over the nodes comes after it, in the same LDS.
//
// VALU issue bounds it.  512 rows of 2048 cells, FP64, order 5, with every
// gradient: 27 us, 70 with 1019-cell tiles a workgroup (58 KB of LDS, two
// workgroups a CU, a barrier after each of the p + 1 ordered scatter passes,
// three tiles for a row of two).  FP32, 1000 rows of 6001 cells, without v0bar:
// 93 us a step of eight, 120.
#include "ram_adjoint_wave.h"
#include "ram_node64.h"

namespace ram {
namespace {

using namespace dev;

constexpr int kFT = kFastTile;
constexpr int kSt = kFT + 8;             // staged cells of one array (cell i0 - 2 + k at k)
constexpr int kWin = kFastWin + 8;
constexpr int kU = 3 * kSt > kWin ? 3 * kSt : kWin;   // doubles: staging, window or node data

// The residual step's transpose on four consecutive cells of a lane, from
// cells a-2 .. a+5 (index w): the state the residual read q, the gradient of
// its result qb, 1/dx di, dx, the inverse centre gaps hv (cell w to w+1), and
// the velocities v8 of their left faces.  The upwind flux with the van Leer
// slope and the swept-interval average of Section 3.1; the limiter's derivative
// is 0 where the one-sided slopes differ in sign, the dv >= 0 branch is taken
// at dv = 0.  gs: the gradient of the shifted state on the four cells; fb: the
// dv gradient terms of their left faces.
template <typename T>
__device__ __forceinline__ void residual_adj(const T (&q)[8], const T (&qb)[8], const T (&di)[8],
                                             const T (&dx)[8], const T (&hv)[8], const T (&v8)[8],
                                             T dt, T (&gs)[4], T (&fb)[4])
{
    // faces a-1+f, between cells f and f+1
    T fbar[7], qsb[7], scs[7], half[7];
    bool up[7];
#pragma unroll
    for (int f = 0; f < 7; ++f) {
        const T v = v8[f + 1];
        up[f] = v >= (T)0;
        fbar[f] = dt * (qb[f + 1] * di[f + 1] - qb[f] * di[f]);
        half[f] = up[f] ? (T)0.5 * (dx[f] - v * dt) : (T)-0.5 * (dx[f + 1] + v * dt);
        qsb[f] = fbar[f] * v;
        scs[f] = qsb[f] * half[f];
    }
    // cells 1 .. 6: slope, limiter derivatives (times the gap inverses), and
    // the slope gradient each receives
    T sg[8], da[8], db[8], sb[8];
#pragma unroll
    for (int w = 1; w <= 6; ++w) {
        const T ap = (q[w + 1] - q[w]) * hv[w];
        const T bm = (q[w] - q[w - 1]) * hv[w - 1];
        sg[w] = da[w] = db[w] = (T)0;
        if (ap * bm > (T)0) {
            const T inv = (T)1 / (ap + bm);
            const T ra = ap * inv, rb = bm * inv;
            da[w] = (T)2 * rb * rb * hv[w];
            db[w] = (T)2 * ra * ra * hv[w - 1];
            sg[w] = (T)2 * ap * rb;
        }
        sb[w] = (up[w - 1] ? (T)0 : scs[w - 1]) + (up[w] ? scs[w] : (T)0);
    }
#pragma unroll
    for (int w = 2; w <= 5; ++w) {
        T g = qb[w];
        if (!up[w - 1]) g += qsb[w - 1];
        if (up[w]) g += qsb[w];
        g += sb[w - 1] * da[w - 1] + sb[w] * (db[w] - da[w]) - sb[w + 1] * db[w + 1];
        gs[w - 2] = g;
        // the cell's left face (face w-1), upwind cell w-1 or w
        const int f = w - 1;
        const int cu = up[f] ? f : f + 1;
        const T qs = q[cu] + sg[cu] * half[f];
        fb[w - 2] = fbar[f] * (qs - (T)0.5 * sg[cu] * v8[f + 1] * dt);
    }
}

template <typename T>
__device__ __forceinline__ void read8(const T *s, T (&o)[8])
{
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = s[k];
}

// (1) Mbar' = Qbar^{n+1/2} / dx of the tile's cells into smb[1 + u], zeros at
// both ends; dvbar's terms added.
template <typename TQ, bool RES>
__device__ __forceinline__ void tile_residual(const StepAdjArgs &a, const TilePos &p, int n,
                                              double *su, double *smb, int t)
{
    constexpr int NS = (kFT + 4 + kLanes - 1) / kLanes;       // slots with the two-cell halo
    constexpr int NC = kFT / kLanes;
    const MeshTab &tb = a.rows.tab;
    const int i0 = p.i0, nd = p.nd, K = nd + 4;
    const int64_t qoff = (int64_t)p.row * n;
    const TQ *qbo = (const TQ *)a.qbar_out + qoff;
    if constexpr (RES) {
        const TQ *qh = (const TQ *)a.q_half + qoff;
        const TQ *dv = (const TQ *)a.dv + qoff;
        TQ *dvb = a.dvbar ? (TQ *)a.dvbar + qoff : nullptr;
        TQ *s0 = (TQ *)su, *s1 = s0 + kSt, *s2 = s1 + kSt;
        TQ vq[NS], vb[NS], vv[NS], vi[NS], old[NC];
        typename TabT<TQ>::T2 vr[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int c = wrap1f(i0 - 2 + min(t + s * kLanes, K - 1), n);
            vq[s] = qh[c];
            vb[s] = qbo[c];
            vv[s] = dv[c];
            vr[s] = TabT<TQ>::rr(tb)[c];
            vi[s] = TabT<TQ>::dxinv(tb)[c];
        }
        if (dvb) {
#pragma unroll
            for (int s = 0; s < NC; ++s) old[s] = dvb[i0 + min(t + s * kLanes, nd - 1)];
        }
        // lanes past the last staged cell repeat it: same value, same place
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int k = min(t + s * kLanes, K - 1);
            s0[k] = vq[s];
            s1[k] = vb[s];
            s2[k] = vv[s];
        }
        wave_sync();
        const int c4 = min(4 * t, (nd - 1) & ~3);
        TQ q[8], qb[8], v8[8], dx[8], hv[8], di[8];
        read8(s0 + c4, q);
        read8(s1 + c4, qb);
        read8(s2 + c4, v8);
        wave_sync();
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int k = min(t + s * kLanes, K - 1);
            s0[k] = vr[s].x;
            s1[k] = vr[s].y;
            s2[k] = vi[s];
        }
        wave_sync();
        read8(s0 + c4, dx);
        read8(s1 + c4, hv);
        read8(s2 + c4, di);
        TQ gs[4], fb[4];
        residual_adj<TQ>(q, qb, di, dx, hv, v8, (TQ)a.dt, gs, fb);
        wave_sync();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            smb[1 + c4 + k] = (double)(gs[k] * di[2 + k]);
            s0[c4 + k] = fb[k];
        }
        wave_sync();
        if (dvb) {
#pragma unroll
            for (int s = 0; s < NC; ++s) {
                const int u = t + s * kLanes;
                if (u < nd) dvb[i0 + u] = old[s] + s0[u];
            }
        }
    } else {
        TQ vb[NC], vi[NC];
#pragma unroll
        for (int s = 0; s < NC; ++s) {
            const int c = i0 + min(t + s * kLanes, nd - 1);
            vb[s] = qbo[c];
            vi[s] = TabT<TQ>::dxinv(tb)[c];
        }
#pragma unroll
        for (int s = 0; s < NC; ++s) smb[1 + min(t + s * kLanes, nd - 1)] = (double)(vb[s] * vi[s]);
    }
    if (t == 0) {
        smb[0] = 0.0;
        smb[nd + 1] = 0.0;
    }
    wave_sync();
}

// Source cell c's stencil in the state's type.
template <int P>
__device__ __forceinline__ void tile_stencil(const MeshTab &tb, int n, int c, double (&rth)[P + 1],
                                             double (&rrd)[P + 1])
{
    node_stencil<P>(tb.stpd, n, c, rth, rrd);
}
template <int P>
__device__ __forceinline__ void tile_stencil(const MeshTab &tb, int n, int c, float (&rth)[P + 1],
                                             float (&rrd)[P + 1])
{
    node_stencil<P>(tb.stp, n, c, rth, rrd);
}

// (2), (3) of an FP32 tile in a uniform run, as the streaming adjoint takes it:
// node e in window cell LO + e at one theta, so the shift's transpose is a fixed
// stencil on Mbar' and v0bar one on Q^n (coefficients and sums in FP64).  1024 x
// 4001 uniform cells: 37 us a step of eight; with every node's FP32 weights 55 (as
// long as the general adjoint took), and their rounding in every gradient.
template <int P, bool V0>
__device__ __forceinline__ void tile_uniform(const StepAdjArgs &a, const FastTile &ft,
                                             const TilePos &p, int n, double *sw, const double *smb,
                                             int t)
{
    constexpr int NW = (kFT + P + kLanes - 1) / kLanes;       // window slots
    constexpr int LO = (P - 1) / 2;
    const MeshTab &tb = a.rows.tab;
    const int nd = p.nd, W = ft.w, base = ft.base;
    const int64_t qoff = (int64_t)p.row * n;
    const double dx = TabT<double>::dx(tb)[base];
    // the theta of the first node, in window cell LO, as the plan forms it: the
    // record's is rounded to FP32, one error for the whole tile
    const double *x = a.rows.edges;
    const double x0 = x[0], xN = x[n];
    const RowShift rs = row_shift(a.v0[p.row] * a.dt, xN - x0, tb.scal[1]);
    int dk;
    const double xt = node_wrap(x[p.i0], rs, x0, xN, dk);
    const double th = cell_theta(tb.stpd, base + LO >= n ? base + LO - n : base + LO, xt, xN - x0, false);
    float *qbi = (float *)a.qbar_in + qoff;
    float *edge = (float *)a.edge + (int64_t)ft.pad[0] * (2 * P);
    float wq[NW];
    if constexpr (V0) {
#pragma unroll
        for (int u = 0; u < NW; ++u) {
            const int c = base + min(t + u * kLanes, W - 1);
            wq[u] = ((const float *)a.q_fwd + qoff)[c >= n ? c - n : c];
        }
    }
    double cs[P + 1];
    uniform_stencil<double, P>(th, cs);
#pragma unroll
    for (int u = 0; u < NW; ++u) {
        const int j = t + u * kLanes;
        if (j >= W) continue;
        double acc = 0.0;
#pragma unroll
        for (int d = 0; d <= P; ++d) {
            const int i = j - d;
            if (i >= 0 && i < nd) acc += cs[d] * smb[1 + i];
        }
        const int c = base + j;
        put_cell<P, float>(qbi, edge, c >= n ? c - n : c, j, W, (float)(acc * dx));
    }
    if constexpr (V0) {
#pragma unroll
        for (int u = 0; u < NW; ++u) sw[min(t + u * kLanes, W - 1)] = (double)wq[u];
        double dw[P + 1], gd[P + 2];
        uniform_dweights<double, P>(th, 1.0, dw);
        outward_sums<double, P>(dw, gd);
        wave_sync();
        double vp = 0.0;
#pragma unroll
        for (int u = 0; u < kFT / kLanes; ++u) {
            const int i = t + u * kLanes;
            if (i >= nd) continue;
            double dq = 0.0;
#pragma unroll
            for (int d = 0; d <= P; ++d) dq += (gd[d] - gd[d + 1]) * sw[i + d];
            vp -= smb[1 + i] * dq;
        }
        vp = wave_sum(vp);
        if (t == 0) a.v0part[ft.pad[0]] = a.dt * vp;
    }
}

// (2), (3) of a tile whose window fits in LDS.  False, and nothing done: a node is not
// in the window.
template <typename TQ, int P, bool V0>
__device__ __forceinline__ bool tile_shift(const StepAdjArgs &a, const FastTile &ft, const TilePos &p,
                                           int n, double *sw, const double *smb, short *sjc, int t)
{
    constexpr int LO = (P - 1) / 2;
    constexpr int NS = (kFT + 1 + kLanes - 1) / kLanes;       // node slots
    constexpr int NC = kFT / kLanes;
    constexpr int NB = 5;                            // window cells a lane has in flight
    const MeshTab &tb = a.rows.tab;
    const int i0 = p.i0, nd = p.nd, NE = nd + 1;
    const int64_t qoff = (int64_t)p.row * n;
    const int W = ft.w, base = ft.base;
    const double *x = a.rows.edges;
    const double x0 = x[0], xN = x[n];
    const RowShift rs = row_shift(a.v0[p.row] * a.dt, xN - x0, tb.scal[1]);
    // (a window wraps the row at most once unless the row is shorter than it)
    const bool wraps = W + base > 2 * n;
    auto wcell = [&](int j) {
        const int c = base + j;
        return wraps ? wrap_small(c, n) : (c >= n ? c - n : c);
    };

    // ---- each node's window cell and position in it ----------------------------
    int jv[NS];
    double thv[NS];
    if (a.fast.jc)
        tile_nodes<P, NS, true>(a.fast, ft, x, n, tb, rs, x0, xN, i0, NE, wcell, t, jv, thv);
    else if (!tile_nodes<P, NS, false>(a.fast, ft, x, n, tb, rs, x0, xN, i0, NE, wcell, t, jv, thv))
        return false;
#pragma unroll
    for (int u = 0; u < NS; ++u) sjc[min(t + u * kLanes, NE - 1)] = (short)jv[u];
    wave_sync();                                     // node cells visible

    // ---- whole cells: Mbar'_i in the window cells [jc_i, jc_{i+1}), 0 outside --
    if (t < LO) sw[t] = 0.0;
    if (t < P - LO) sw[W - (P - LO) + t] = 0.0;
#pragma unroll
    for (int u = 0; u < NC; ++u) {
        const int i = t + u * kLanes;
        if (i < nd) {
            const int ja = sjc[i], jb = sjc[i + 1];
            const double mb = smb[1 + i];
            for (int j = ja; j < jb; ++j) sw[j] = mb;
        }
    }
    wave_sync();
    // ---- each node's terms: Vbar_e times its partial integral's coefficients
    // of cells jc - LO .. jc + P - LO - 1.  (The slots' loops are not unrolled:
    // unrolled, the stencils of all five take 340 registers.)
#pragma unroll 1
    for (int u = 0; u < NS; ++u) {
        const int m = t + u * kLanes, mc = min(m, NE - 1);
        const int j = jv[0], c = wcell(j);
        TQ rth[P + 1], rrd[P + 1], wk[P + 1];
        double tm[P];
        tile_stencil<P>(tb, n, c, rth, rrd);
        // the slot's nodes before this one in its source cell
        const bool first = t == 0 || (int)sjc[max(mc - 1, 0)] != j;
        const uint64_t starts = __ballot(first) & (~0ull >> (kLanes - 1 - t));
        const int rank = t - (63 - __clzll((long long)starts));
        node_weights<P>(rth, rrd, (TQ)thv[0], wk);
        const double vb = smb[mc] - smb[mc + 1];
        double s = 0.0;
#pragma unroll
        for (int b = P; b > LO; --b) {
            s += (double)wk[b];
            tm[b - 1] = s * vb;
        }
        s = 0.0;
#pragma unroll
        for (int b = 0; b < LO; ++b) {
            s += (double)wk[b];
            tm[b] = -s * vb;
        }
        double *at = sw + j - LO;
        uint64_t todo = __ballot(m < NE);
        for (int turn = 0; todo; ++turn) {
            const bool now = m < NE && rank == turn;
            if (now) {
#pragma unroll
                for (int k = 0; k < P; ++k) atomicAdd(at + k, tm[k]);
            }
            todo &= ~__ballot(now);
        }
        slot_turn(jv);
        slot_turn(thv);
    }
    wave_sync();
    // ---- Qbar^n = Mbar dx, one window cell a lane --------------------------------
    TQ *qbi = (TQ *)a.qbar_in + qoff;
    TQ *edge = (TQ *)a.edge + (int64_t)ft.pad[0] * (2 * P);
    for (int j0 = t; j0 - t < W; j0 += NB * kLanes) {
        double wd[NB];
        int cw[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            cw[u] = wcell(min(j0 + u * kLanes, W - 1));
            wd[u] = TabT<double>::dx(tb)[cw[u]];
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int j = j0 + u * kLanes;
            if (j < W) put_cell<P, TQ>(qbi, edge, cw[u], j, W, (TQ)(sw[j] * wd[u]));
        }
    }
    // ---- v0bar: q~ at the nodes from the window's masses ---------------------------
    if constexpr (V0) {
        wave_sync();                                 // the gradients are dead
        const TQ *qf = (const TQ *)a.q_fwd + qoff;
        for (int j0 = t; j0 - t < W; j0 += NB * kLanes) {
            double wq[NB], wd[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const int c = wcell(min(j0 + u * kLanes, W - 1));
                wq[u] = (double)qf[c];
                wd[u] = TabT<double>::dx(tb)[c];
            }
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if (j0 + u * kLanes < W) sw[j0 + u * kLanes] = wq[u] * wd[u];
        }
        wave_sync();
        double qt[NS];
#pragma unroll 1
        for (int u = 0; u < NS; ++u) {
            const int j = jv[0], c = wcell(j);
            TQ rth[P + 1], rrd[P + 1], dw[P + 1];
            tile_stencil<P>(tb, n, c, rth, rrd);
            node_dweights<P>(rth, rrd, (TQ)thv[0], dw);
            double dq = 0.0, up = 0.0, dn = 0.0;
#pragma unroll
            for (int b = LO + 1; b <= P; ++b) {
                up += sw[j + b - LO - 1];
                dq += (double)dw[b] * up;
            }
#pragma unroll
            for (int b = LO - 1; b >= 0; --b) {
                dn += sw[j - LO + b];
                dq -= (double)dw[b] * dn;
            }
            qt[0] = dq * tb.stpd[c].y;
            slot_turn(qt);
            slot_down(jv);
            slot_down(thv);
        }
        v0_term<NS>(a, ft.pad[0], qt, smb, nd, t);
    }
    return true;
}

// (2), (3) of a tile whose window does not fit in LDS: the sums of tile_shift, in its
// order, on pieces of the window.  A piece holds C + P cells; the nodes whose terms
// end in it are added, its first C cells are then whole and go out, and its last P
// begin the next piece.  Every node's weights are formed in FP64, whatever the state.
//
// Latency bounds it, as the tiles that fit.  512 rows refined tenfold, shifted by
// anything in their period, with every gradient: FP64 rows of 1600 and 4096 cells 48
// and 96 us, FP32 rows of 1301 and 2047 38 and 44; with every window cell's nodes
// searched and weighed from global memory 115 and 178, 68 and 82.
template <typename TQ, int P, bool V0>
__device__ __forceinline__ void tile_wide(const StepAdjArgs &a, const FastTile &ft, const TilePos &p,
                                          int n, double *su, const double *smb, int t)
{
    constexpr int LO = (P - 1) / 2;
    constexpr int NS = (kFT + 1 + kLanes - 1) / kLanes;       // node slots
    constexpr int NC = kFT / kLanes;
    constexpr int NB = 5;                            // window cells a lane has in flight
    constexpr int kNode = kFastNodes / 2;            // doubles the nodes' cells take
    constexpr int CP = kU - kNode, C = CP - P;
    const MeshTab &tb = a.rows.tab;
    const int i0 = p.i0, nd = p.nd, NE = nd + 1, base = ft.base;
    const int64_t qoff = (int64_t)p.row * n;
    const double *x = a.rows.edges;
    const double x0 = x[0], xN = x[n];
    const RowShift rs = row_shift(a.v0[p.row] * a.dt, xN - x0, tb.scal[1]);
    int *sj = (int *)su;                             // each node's window cell
    double *sw = su + kNode;                         // the piece
    // (a window is shorter than two periods and the stencil)
    auto wcell = [&](int j) { return wrap_small(base + j, n); };
    // the window: this tile's first node's stencil up to the next tile's (the row's
    // first tile one period on, for the last tile of a row)
    const int tpr = (n + kFT - 1) / kFT;
    auto wlo_of = [&](int k) {
        const FastTile &r = a.fast.rec[k];
        return (int64_t)(((uint64_t)(uint32_t)r.wlo_hi << 32) | (uint32_t)r.wlo_lo);
    };
    const int64_t wlo = wlo_of(ft.pad[0]);
    const int64_t wend = i0 + nd >= n ? wlo_of(ft.pad[0] - (tpr - 1)) + n : wlo_of(ft.pad[0] + 1);
    const int W = (int)(wend - wlo) + P;

    // ---- each node's window cell and position in it ----------------------------
    int jv[NS];
    double thv[NS];
    {
        int ce[NS], kx[NS];
        double xt[NS];
        locate_nodes<NS>(x, n, tb, rs, x0, xN, i0, NE, t, ce, kx, xt);
        const int jbase = (int)(rs.kf0 * (int64_t)n - wlo);
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            jv[u] = min(max(ce[u] + kx[u] + jbase, LO), W - (P - LO));
            thv[u] = cell_theta(tb.stpd, ce[u], xt[u], xN - x0, false);
            sj[min(t + u * kLanes, NE - 1)] = jv[u];
        }
    }
    wave_sync();                                     // node cells visible
    TQ *qbi = (TQ *)a.qbar_in + qoff;
    TQ *edge = (TQ *)a.edge + (int64_t)ft.pad[0] * (2 * P);
    for (int b = 0; b < W; b += C) {
        const bool last = b + CP >= W;
        const int end = min(b + CP, W);
        // ---- whole cells: the piece's own ones, after the P carried on ------------
        const int from = b == 0 ? 0 : b + P;
        for (int j = from + t; j < end; j += kLanes) sw[j - b] = 0.0;
        wave_sync();
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int i = t + u * kLanes;
            if (i < nd) {
                const int ja = max(sj[i], from), jb = min(sj[i + 1], end);
                const double mb = smb[1 + i];
                for (int j = ja; j < jb; ++j) sw[j - b] = mb;
            }
        }
        wave_sync();
        // ---- the terms of the nodes whose cells the piece holds ---------------------
#pragma unroll 1
        for (int u = 0; u < NS; ++u) {
            const int m = t + u * kLanes, mc = min(m, NE - 1);
            const int j = jv[0];
            const bool here = m < NE && j - LO >= b && (last || j - LO < b + C);
            uint64_t todo = __ballot(here);
            if (todo) {
                double rth[P + 1], rrd[P + 1], wk[P + 1], tm[P];
                node_stencil<P>(tb.stpd, n, wcell(j), rth, rrd);
                // the slot's nodes before this one in its source cell
                const bool first = t == 0 || sj[max(mc - 1, 0)] != j;
                const uint64_t starts = __ballot(first) & (~0ull >> (kLanes - 1 - t));
                const int rank = t - (63 - __clzll((long long)starts));
                node_weights<P>(rth, rrd, thv[0], wk);
                const double vb = smb[mc] - smb[mc + 1];
                double s = 0.0;
#pragma unroll
                for (int k = P; k > LO; --k) {
                    s += wk[k];
                    tm[k - 1] = s * vb;
                }
                s = 0.0;
#pragma unroll
                for (int k = 0; k < LO; ++k) {
                    s += wk[k];
                    tm[k] = -s * vb;
                }
                double *at = sw + (here ? j - LO - b : 0);
                for (int turn = 0; todo; ++turn) {
                    const bool now = here && rank == turn;
                    if (now) {
#pragma unroll
                        for (int k = 0; k < P; ++k) atomicAdd(at + k, tm[k]);
                    }
                    todo &= ~__ballot(now);
                }
            }
            slot_turn(jv);
            slot_turn(thv);
        }
        wave_sync();
        // ---- Qbar^n = Mbar dx, one window cell a lane -------------------------------
        const int out = last ? W : b + C;
        for (int j0 = b + t; j0 - t < out; j0 += NB * kLanes) {
            double wd[NB];
            int cw[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                cw[u] = wcell(min(j0 + u * kLanes, out - 1));
                wd[u] = TabT<double>::dx(tb)[cw[u]];
            }
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const int j = j0 + u * kLanes;
                if (j < out) put_cell<P, TQ>(qbi, edge, cw[u], j, W, (TQ)(sw[j - b] * wd[u]));
            }
        }
        if (last) break;
        const double carry = sw[C + min(t, P - 1)];
        wave_sync();
        if (t < P) sw[t] = carry;
    }
    // ---- v0bar: q~ at the nodes from the window's masses, a piece after the other ----
    if constexpr (V0) {
        const TQ *qf = (const TQ *)a.q_fwd + qoff;
        double qt[NS];
#pragma unroll
        for (int u = 0; u < NS; ++u) qt[u] = 0.0;
        for (int b = 0; b < W; b += C) {
            const bool last = b + CP >= W;
            const int len = min(CP, W - b);
            wave_sync();                             // the gradients, or the last piece, are dead
            for (int k0 = t; k0 - t < len; k0 += NB * kLanes) {
                double wq[NB], wd[NB];
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int c = wcell(b + min(k0 + u * kLanes, len - 1));
                    wq[u] = (double)qf[c];
                    wd[u] = TabT<double>::dx(tb)[c];
                }
#pragma unroll
                for (int u = 0; u < NB; ++u)
                    if (k0 + u * kLanes < len) sw[k0 + u * kLanes] = wq[u] * wd[u];
            }
            wave_sync();
#pragma unroll 1
            for (int u = 0; u < NS; ++u) {
                const int j = jv[0];
                const bool here = j - LO >= b && (last || j - LO < b + C);
                if (__any(here ? 1 : 0)) {
                    const int c = wcell(j), k = here ? j - LO - b : 0;
                    TQ rth[P + 1], rrd[P + 1], dw[P + 1];
                    tile_stencil<P>(tb, n, c, rth, rrd);
                    node_dweights<P>(rth, rrd, (TQ)thv[0], dw);
                    double dq = 0.0, up = 0.0, dn = 0.0;
#pragma unroll
                    for (int d = LO + 1; d <= P; ++d) {
                        up += sw[k + d - 1];
                        dq += (double)dw[d] * up;
                    }
#pragma unroll
                    for (int d = LO - 1; d >= 0; --d) {
                        dn += sw[k + d];
                        dq -= (double)dw[d] * dn;
                    }
                    if (here) qt[0] = dq * tb.stpd[c].y;
                }
                slot_turn(qt);
                slot_turn(jv);
                slot_turn(thv);
            }
            if (last) break;
        }
        v0_term<NS>(a, ft.pad[0], qt, smb, nd, t);
    }
}

template <typename TQ, int P, bool RES, bool V0>
__global__ __launch_bounds__(kBlock, 4) void k_adj_tile(StepAdjArgs a)
{
    __shared__ __attribute__((aligned(16))) double su[kWaves][kU];
    __shared__ __attribute__((aligned(16))) double smb_[kWaves][kFT + 8];
    __shared__ short sjc_[kWaves][kFastNodes];
    const int wid = wave_id();
    const int i = (int)blockIdx.x * kWaves + wid;
    if (i >= (int)a.rows.n_tiles) return;
    const int n = (int)a.rows.n_cols;
    const int t = (int)threadIdx.x % kLanes;
    const FastTile ft = load_rec(a.fast.rec, i);
    const TilePos p = tile_pos(i, n, 0);
    tile_residual<TQ, RES>(a, p, n, su[wid], smb_[wid], t);
    if constexpr (sizeof(TQ) == 4) {
        if (ft.kind == kFastUniform) return tile_uniform<P, V0>(a, ft, p, n, su[wid], smb_[wid], t);
    }
    if (ft.kind == kFastDirect || !tile_shift<TQ, P, V0>(a, ft, p, n, su[wid], smb_[wid], sjc_[wid], t))
        tile_wide<TQ, P, V0>(a, ft, p, n, su[wid], smb_[wid], t);
}

template <typename TQ, int P, bool RES, bool V0>
hipError_t adj_tile_kernels(const StepAdjArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL((k_adj_tile<TQ, P, RES, V0>), dim3(uniform_grid(a.rows.n_tiles)), dim3(kBlock),
                       0, st, a);
    return launch_edges<TQ, P>(a, V0, st);
}

template <typename TQ, int P>
hipError_t adj_tile_p(const StepAdjArgs &a, hipStream_t st)
{
    const bool v0 = a.v0bar != nullptr && a.q_fwd != nullptr;
    if (a.dv)
        return v0 ? adj_tile_kernels<TQ, P, true, true>(a, st)
                  : adj_tile_kernels<TQ, P, true, false>(a, st);
    return v0 ? adj_tile_kernels<TQ, P, false, true>(a, st)
              : adj_tile_kernels<TQ, P, false, false>(a, st);
}

template <typename TQ>
hipError_t adj_tile_t(const StepAdjArgs &a, int order, hipStream_t st)
{
    switch (order) {
    case 1: return adj_tile_p<TQ, 1>(a, st);
    case 3: return adj_tile_p<TQ, 3>(a, st);
    default: return adj_tile_p<TQ, 5>(a, st);
    }
}

} // namespace

hipError_t launch_step_adjoint_tile(const StepAdjArgs &a, bool f64, int order, hipStream_t stream)
{
    if (a.rows.n_tiles <= 0) return hipSuccess;
    if (a.rows.tile != kFastTile || a.rows.n_cols < kFastTile + 8 ||
        a.rows.n_tiles > INT32_MAX / 2 || !a.edge)
        return hipErrorInvalidValue;
    return f64 ? adj_tile_t<double>(a, order, stream) : adj_tile_t<float>(a, order, stream);
}

} // namespace ram
