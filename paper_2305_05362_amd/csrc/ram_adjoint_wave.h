// ram_adjoint_wave.h -- what the adjoint kernels that run a tile a wave share:
// where a window cell's gradient goes, v0bar's terms, the tiles whose window
// does not fit in LDS, and the cells several tiles add into.
#pragma once

#include "ram_adjoint_dev.h"
#include "ram_device.h"
#include "ram_wave.h"

namespace ram {
namespace dev {

// Sum of a double over the wave.
__device__ __forceinline__ double wave_sum(double v)
{
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
    return v;
}

// Store the gradient v of window cell j (of W; row cell `cell`): a cell only
// this tile's window holds goes to the state, the window's first p cells
// (head) and its last p (tail; the two overlap-free when W < 2p) to the
// tile's side buffer, for k_adjf_edges.  One store a lane, whichever it is.
template <int P, typename TQ>
__device__ __forceinline__ void put_cell(TQ *qbi, TQ *edge, int cell, int j, int W, TQ v)
{
    TQ *dst;
    if (j >= P && j < W - P) dst = qbi + cell;
    else if (j < P) dst = edge + j;
    else dst = edge + P + (j - max(P, W - P));
    *dst = v;
}

// v0bar of a tile from q~ at its nodes (node m = t + 64u in slot u) and Mbar'
// in smb: -dt sum_i Mbar'_i (q~_{i+1} - q~_i), one term a tile.
template <int NS, typename MT>
__device__ __forceinline__ void v0_term(const StepAdjArgs &a, int tile, const double (&qt)[NS],
                                        const MT *smb, int nd, int t)
{
    double vp = 0.0;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int m = t + u * kLanes;
        // q~ of node m + 1: the next lane's, lane 63 the next slot's lane 0
        double qn = __shfl_down(qt[u], 1);
        if (u + 1 < NS) {
            const double q0 = __shfl(qt[u + 1 < NS ? u + 1 : u], 0);
            if (t == kLanes - 1) qn = q0;
        }
        if (m < nd) vp -= (double)smb[1 + m] * (qn - qt[u]);
    }
    vp = wave_sum(vp);
    if (t == 0) a.v0part[tile] = a.dt * vp;
}

// The reconstruction q~ at a node in cell c from global memory: the weights'
// x-derivatives dw on the cumulative differences C(c - lo + b) - C(c), from
// the masses of cells c-lo .. c+p-lo-1 (FP64).
template <int P, typename TQ>
__device__ __forceinline__ double qtilde_global(const double *x, const TQ *q, int n,
                                                const double (&dw)[P + 1], int c)
{
    constexpr int LO = (P - 1) / 2;
    double m[P];
#pragma unroll
    for (int k = 0; k < P; ++k) m[k] = cell_mass(x, q, n, (int64_t)c - LO + k);
    double dq = 0.0, up = 0.0, dn = 0.0;
#pragma unroll
    for (int b = LO + 1; b <= P; ++b) {
        up += m[b - 1];
        dq += dw[b] * up;
    }
#pragma unroll
    for (int b = LO - 1; b >= 0; --b) {
        dn += m[b];
        dq -= dw[b] * dn;
    }
    return dq;
}

// The streaming adjoint's shift of a tile whose window does not fit, from Mbar' of its
// cells in smb[1 ..] (zeros at both ends); su holds 16 kFastNodes bytes.
template <typename TQ, int P, bool V0, typename MT>
__device__ __forceinline__ void direct_shift(const StepAdjArgs &a, const FastTile &ft, void *su,
                                             const MT *smb, int t)
{
    constexpr int LO = (P - 1) / 2;
    constexpr int NS = (kFastNodes + kLanes - 1) / kLanes;
    const Rows &R = a.rows;
    const MeshTab &tb = R.tab;
    const int n = (int)R.n_cols;
    const int tile = ft.pad[0];
    const TilePos p = tile_pos(tile, n, 0);
    const int i0 = p.i0, nd = p.nd, NE = nd + 1;
    const int64_t qoff = (int64_t)p.row * n;
    TQ *qbi = (TQ *)a.qbar_in + qoff;
    const double *x = R.edges;
    const double len = x[n] - x[0];
    const RowShift rs = row_shift(a.v0[p.row] * a.dt, len, tb.scal[1]);

    int64_t *sgd = (int64_t *)su;                    // node m's extended source index
    double *svb = (double *)(sgd + kFastNodes);      // and its Vbar
    double qt[NS];
#pragma unroll 1
    for (int u = 0; u < NS; ++u) {
        const int m = t + u * kLanes;
        qt[0] = 0.0;
        if (m < NE) {
            const int en = i0 + m;
            const int kx = en >= n ? 1 : 0;
            TQ w[P + 1];
            double xh;
            int c;
            sgd[m] = node_eval_adj<TQ, P, true>(x, n, tb, rs, len, x[en - kx * n], kx, w, c, xh);
            svb[m] = (double)smb[m] - (double)smb[m + 1];
            if constexpr (V0) {
                double dwd[P + 1];
                node_dweights<TQ, P>(tb, c, xh, dwd);
                qt[0] = qtilde_global<P>(x, (const TQ *)a.q_fwd + qoff, n, dwd, c);
            }
        }
        slot_turn(qt);
    }
    wave_sync();
    // the window: this tile's first node's stencil up to the next tile's
    // (the row's first tile one period on, for the last tile of a row)
    const int tpr = (n + kFastTile - 1) / kFastTile;
    const bool last = i0 + nd >= n;
    auto wlo_of = [&](int k) {
        const FastTile &r = a.fast.rec[k];
        return (int64_t)(((uint64_t)(uint32_t)r.wlo_hi << 32) | (uint32_t)r.wlo_lo);
    };
    const int64_t wl = wlo_of(tile);
    const int64_t wend = (last ? wlo_of(tile - (tpr - 1)) + n : wlo_of(tile + 1)) + P;
    const int Wd = (int)(wend - wl);
    TQ *edge = (TQ *)a.edge + (int64_t)tile * (2 * P);
    for (int j = t; j < Wd; j += kLanes) {
        const int64_t target = wl + j + LO;
        int lo = 0, hi = NE;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sgd[mid] > target) hi = mid; else lo = mid + 1;
        }
        // nodes lo.. lie wholly above the cell: their Vbar telescopes to Mbar'_{lo-1}
        double S = (lo >= 1 && lo <= nd) ? (double)smb[lo] : 0.0;
        for (int e = lo - 1; e >= 0 && sgd[e] > target - P; --e) {
            const int en = i0 + e;
            const int kx = en >= n ? 1 : 0;
            double ww[P + 1], xh2;
            int c2;
            node_eval_adj<double, P, true>(x, n, tb, rs, len, x[en - kx * n], kx, ww, c2, xh2);
            // the share of the node's weights on cumulative nodes above the
            // cell, the own weight taken as one minus the others
            const int bmin = (int)min((int64_t)P, max((int64_t)1, target - sgd[e] + 1));
            double h = 0.0;
            if (bmin > LO) {
                for (int b = P; b >= bmin; --b) h += ww[b];
            } else {
                for (int b = 0; b < bmin; ++b) h += ww[b];
                h = 1.0 - h;
            }
            S += svb[e] * h;
        }
        const int mm = wrapi(wl + j, n);
        put_cell<P>(qbi, edge, mm, j, Wd, (TQ)(S * (double)TabT<TQ>::dx(tb)[mm]));
    }
    if constexpr (V0) v0_term<NS>(a, tile, qt, smb, nd, t);
}

namespace {

// The window cells that several tiles add into: the first p of every tile's
// window (a tile's window ends p cells past the next tile's start).  Boundary
// T (one thread) writes the cells from its window start up to p cells on or
// the next tile's start, each the sum, tile T first and then down, of the
// terms the tiles whose windows hold it stored (head or tail; tile k's window
// is [A_k, A_{k+1} + p), and across the row's ends the row's tiles one period
// away).  Usually two terms; more where a tile's nodes fall in fewer than p
// source cells.
template <typename TQ, int P, bool V0>
__global__ __launch_bounds__(256) void k_adjf_edges(StepAdjArgs a, unsigned boundary_blocks)
{
    // workgroups past the boundaries' add up v0bar, a row a wave (one launch
    // instead of two; disjoint outputs)
    if (V0 && blockIdx.x >= boundary_blocks) {
        v0_reduce_row(a.rows, a.v0part, a.v0bar,
                      (int64_t)(blockIdx.x - boundary_blocks) * kWaves + threadIdx.x / kLanes);
        return;
    }
    const int64_t tile = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (tile >= a.rows.n_tiles) return;
    const int n = (int)a.rows.n_cols;
    const int tpr = (n + kFastTile - 1) / kFastTile;
    const int64_t row = (int)tile / tpr;             // (fewer than 2^31 tiles)
    const int k0 = (int)(tile - row * tpr);
    // window start of the row's k-th tile, any k (k mod tpr, one period per wrap)
    auto start = [&](int k, int64_t &id) {
        const int q = k >= 0 ? k / tpr : -((-k + tpr - 1) / tpr);
        id = row * tpr + (k - q * tpr);
        const FastTile &r = a.fast.rec[id];
        const int64_t w = (int64_t)(((uint64_t)(uint32_t)r.wlo_hi << 32) | (uint32_t)r.wlo_lo);
        return w + (int64_t)q * n;
    };
    int64_t idp, id0, idn;
    const int64_t ap = start(k0 - 1, idp), a0 = start(k0, id0), a1 = start(k0 + 1, idn);
    TQ *qbi = (TQ *)a.qbar_in + row * n;
    if (a1 - a0 >= P && a0 - ap >= P) {
        // two terms a cell: this tile's head and the previous tile's tail
        // (its window [ap, a0 + p) of at least 2p cells ends its tail there)
        const TQ *e0 = (const TQ *)a.edge + id0 * (2 * P);
        const TQ *ep = (const TQ *)a.edge + idp * (2 * P);
        TQ v[P];
#pragma unroll
        for (int k = 0; k < P; ++k) v[k] = ((TQ)0 + e0[k]) + ep[P + k];
        // (the record's start in the row: a0's remainder)
        const int b0 = a.fast.rec[id0].base;
#pragma unroll
        for (int k = 0; k < P; ++k) qbi[b0 + k >= n ? b0 + k - n : b0 + k] = v[k];
        return;
    }
    const int64_t mend = min(a0 + P, a1);
    for (int64_t m = a0; m < mend; ++m) {
        TQ sum = (TQ)0;
        int64_t at = a0, an = a1, id = id0;
        for (int k = k0; k > k0 - tpr - 1; --k) {
            if (k != k0) {
                an = at;
                at = start(k, id);
            }
            const int64_t W = an - at + P;
            if (at + W <= m) break;
            const int pos = (int)(m - at);
            const TQ *e = (const TQ *)a.edge + id * (2 * P);
            sum += pos < P ? e[pos] : e[P + pos - (int)max((int64_t)P, W - P)];
        }
        qbi[wrapi(m, n)] = sum;
    }
}

// Its launch, after the tiles' kernels.
template <typename TQ, int P>
hipError_t launch_edges(const StepAdjArgs &a, bool v0, hipStream_t st)
{
    const unsigned gb = (unsigned)((a.rows.n_tiles + 255) / 256);
    const unsigned gv = (unsigned)((a.rows.n_rows + kWaves - 1) / kWaves);
    if (v0) hipLaunchKernelGGL((k_adjf_edges<TQ, P, true>), dim3(gb + gv), dim3(256), 0, st, a, gb);
    else hipLaunchKernelGGL((k_adjf_edges<TQ, P, false>), dim3(gb), dim3(256), 0, st, a, gb);
    return hipGetLastError();
}

} // namespace

} // namespace dev
} // namespace ram
