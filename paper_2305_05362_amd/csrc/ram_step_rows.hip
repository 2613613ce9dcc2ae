// ram_step_rows.hip -- the RAM step on rows of their own meshes (gfx950): the
// bulk shift (Section 3, Steps 1-3, Eqs. Qmass_i, condition_p,
// mass_shift_algo, step3), optionally fused with the residual upwind step (Eq.
// splitting_second, van Leer slope of Section 3.1), nothing planned ahead.
//
// One tile a wave, 255 cells of a row (251 with the residual and its two-cell
// halo a side), whose 256 shifted nodes are four slots of the wave's lanes; no
// workgroup barrier.  A wave
//   (A) locates its end nodes in the row and so its source window, whose node
//       coordinates it reads once into LDS, where every node finds its cell
//       and its Lagrange weights (rows_locate, rows_weights);
//   (B) forms the window's masses M = Q dx, and for the FP32 prefix modes
//       their cumulative over the nodes' LDS (compensated or plain: four masses
//       a lane, scanned across the wave in DPP steps);
//   (C) takes each node's partial integral of the reconstruction, the Lagrange
//       interpolant of the window cumulative, from the cumulative's differences
//       (FP64: from sums of the few masses between, which no cancellation
//       touches);
//   (D) each destination cell's mass, the whole source cells in between plus
//       two partial integrals, over its size;
//   (E) the residual from the shifted state in LDS, one face, then one cell a
//       lane.
// A window beyond kRowsCap cells, or of a row so short that it crosses its end
// more than twice, is summed from global memory.
//
// VALU issue bounds it, with the chain of dependent loads that starts a wave
// (the table, the row, its ends and nodes, two rounds of the window search, the
// window): 1,726 VALU instructions a tile at order 5 with the residual, of
// which the weights of its 256 nodes take about 500 and their search in LDS
// 300.  1024 rows of 64 .. 4096 cells, FP32, two-sum, with the residual: 44 us
// (26 of them VALU issue); with 1019-cell tiles a workgroup (27 KB of LDS,
// seven barriers, two lanes searching the row for the window while the others
// wait) 74.  Five waves a SIMD spill (51 us).  Small batches take two node slots
// a lane instead of four: the chain of one wave is what they cost.
#include "ram_rows.h"

#include <type_traits>

namespace ram {
namespace {

using namespace dev;

constexpr int kRowsCap = 448;        // LDS window, cells

// LDS of one wave: window nodes, later the cumulative; masses; partial
// integrals; window cells of the nodes.  The residual's five arrays reuse it.
template <typename TQ, int S> struct RowsLds {
    using M = typename Acc<S>::M;
    using A = typename Acc<S>::A;
    using D = typename std::conditional<std::is_same<TQ, double>::value, double,
                                        typename Acc<S>::D>::type;
    static constexpr size_t xs = 8 * (kRowsCap + 8);
    static constexpr size_t sm = sizeof(M) * (kRowsCap + 8);
    static constexpr size_t sell = sizeof(D) * (kLanes * 4);
    static constexpr size_t res = 5 * sizeof(TQ) * (kLanes * 4);
    static constexpr size_t sum = xs + sm + sell;
    static constexpr size_t bytes = sum > res ? sum : res;
    static_assert(sizeof(A) <= 8 && 8 * kLanes * 4 <= xs, "the nodes' bytes hold the cumulative");
};

// sub: wave tiles a table tile holds (R.tile = sub times the wave's tile).
// NS: node slots a lane.
template <typename TQ, int P, int S, int H, int NS>
__global__ __launch_bounds__(kBlock) void k_rows(StepArgs a, int sub)
{
    using AC = Acc<S>;
    using L = RowsLds<TQ, S>;
    using M = typename L::M;
    using A = typename L::A;
    using D = typename L::D;
    using CT = TQ;
    constexpr int LO = (P - 1) / 2;
    constexpr bool kLocal = S == kScanF64;           // sums of the FP64 masses between
    constexpr int NDT = kLanes * NS - 1 - 2 * H;     // destination cells
    constexpr int NQ = 5;                            // window slots loaded ahead
    __shared__ __attribute__((aligned(16))) unsigned char su_[kWaves][L::bytes];
    __shared__ short sjc_[kWaves][kLanes * NS];
    const int wid = wave_id();
    const int t = (int)threadIdx.x % kLanes;
    const int64_t wave = (int64_t)blockIdx.x * kWaves + wid;
    const Rows &R = a.rows;
    const int64_t tile = sub == 1 ? wave : wave / sub;
    if (tile >= R.n_tiles) return;
    Tile ti;
    if (!get_tile(R, tile, ti)) return;
    const int n = ti.n;
    const int i0 = ti.i0 + (int)(wave - tile * sub) * NDT;
    if (n < P + 1 || i0 >= n) return;
    const int nd = min(NDT, n - i0);
    const int NC = nd + 2 * H;                       // shifted cells
    const int NE = NC + 1;                           // shifted nodes
    const double *x = ti.x;
    const TQ *q = (const TQ *)a.q_in + ti.qoff;
    TQ *qo = (TQ *)a.q_out + ti.qoff;
    const double s = rows_shift(a.v0[ti.row], a.dt);
    const double x0 = x[0], xN = x[n];
    const double len = xN - x0;
    const double invlen = 1.0 / len;
    unsigned char *su = su_[wid];
    double *xs = (double *)su;                       // window nodes
    A *sp = (A *)su;                                 // exclusive cumulative
    M *sm = (M *)(su + L::xs);                       // masses
    D *sell = (D *)(su + L::xs + L::sm);             // partial integrals
    short *sjc = sjc_[wid];

    // ---- the nodes (and, node m being cell m's left one, the cells) -----------
    double xe[NS], xr[NS];
    int kx[NS], cell[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        int e = i0 - H + min(t + u * kLanes, NE - 1);
        kx[u] = 0;
        if (e < 0) { e += n; kx[u] = -1; }
        while (e >= n) { e -= n; kx[u] += 1; }
        cell[u] = e;
        xe[u] = x[e];
        xr[u] = x[e + 1];
    }
    CT v[NS];                                        // face velocity of the cell's left face
    if constexpr (H != 0) {
#pragma unroll
        for (int u = 0; u < NS; ++u) v[u] = (CT)((const TQ *)a.dv + ti.qoff)[cell[u]];
    }

    // ---- (A) -------------------------------------------------------------------
    RowsWindow win;
    double xh[NS];
    int j[NS];
    TQ qv[NQ];
    const bool windowed = rows_locate<P, NS>(
        x, n, s, x0, xN, len, invlen, NE, t, kRowsCap, xe, kx, xs, win, xh, j, [&] {
#pragma unroll
            for (int u = 0; u < NQ; ++u) qv[u] = q[win.at(min(t + u * kLanes, win.w - 1), n)];
        });
    CT qs[NS];
    double x2[NS];                                   // the residual's: the next cell's right node
    if constexpr (H != 0) {
#pragma unroll
        for (int u = 0; u < NS; ++u) x2[u] = x[cell[u] + 2 <= n ? cell[u] + 2 : 1];
    }
    if (windowed) {
        const int W = win.w;
        TQ w[NS][P + 1];
        if (win.seam > W) {
#pragma unroll
            for (int u = 0; u < NS; ++u) rows_weights<TQ, P, false>(xs, win, len, xh[u], j[u], w[u]);
        } else {
#pragma unroll 1
            for (int u = 0; u < NS; ++u) {
                // (one copy of the code: the slots move past it)
                slot_down(w);
                rows_weights<TQ, P, true>(xs, win, len, xh[0], j[0], w[NS - 1]);
                slot_turn(xh);
                slot_turn(j);
            }
        }
        // ---- (B) -----------------------------------------------------------------
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int i = t + u * kLanes;
            if (i < W) sm[i] = AC::template mass<TQ>(qv[u], rows_size(xs, win, xN, i));
        }
        for (int i = t + NQ * kLanes; i < W; i += kLanes)
            sm[i] = AC::template mass<TQ>(q[win.at(i, n)], rows_size(xs, win, xN, i));
        wave_sync();                                 // the nodes are dead
        if constexpr (!kLocal) {
            rows_prefix<S>(sp, sm, W, t);
            wave_sync();
        }
        // ---- (C) -----------------------------------------------------------------
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            D ell = (D)0;
            if constexpr (kLocal) {
                D up = (D)0, dn = (D)0;
#pragma unroll
                for (int b = LO + 1; b <= P; ++b) {
                    up += sm[j[u] + b - LO - 1];
                    ell += (D)w[u][b] * up;
                }
#pragma unroll
                for (int b = LO - 1; b >= 0; --b) {
                    dn += sm[j[u] - LO + b];
                    ell -= (D)w[u][b] * dn;
                }
            } else {
                const A pc = sp[j[u]];
#pragma unroll
                for (int b = 0; b <= P; ++b)
                    if (b != LO) ell += (D)w[u][b] * (D)AC::diff(sp[j[u] - LO + b], pc);
            }
            const int m = min(t + u * kLanes, NE - 1);
            sell[m] = ell;
            sjc[m] = (short)j[u];
        }
        wave_sync();
        // ---- (D) (slots past the last cell repeat it) ------------------------------
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int ci = min(t + u * kLanes, NC - 1);
            const int ja = sjc[ci], jb = sjc[ci + 1];
            D whole;
            if constexpr (kLocal) {
                whole = jb > ja ? sm[ja] : (D)0;
                for (int i = ja + 1; i < jb; ++i) whole += sm[i];
            } else {
                whole = jb - ja == 1 ? (D)sm[ja] : (D)AC::diff(sp[jb], sp[ja]);
            }
            qs[u] = (CT)((whole + (sell[ci + 1] - sell[ci])) / (D)(xr[u] - xe[u]));
        }
    } else {
        // masses summed from global memory in FP64
        wave_sync();
        int64_t *sg = (int64_t *)su;
#pragma unroll 1
        for (int m = t; m < NE; m += kLanes) {
            int e = i0 - H + m, k1 = 0;
            if (e < 0) { e += n; k1 = -1; }
            while (e >= n) { e -= n; k1 += 1; }
            double xn;
            int64_t k;
            shifted_node_inv(x, n, s, e, invlen, len, xn, k);
            const int64_t g = (int64_t)find_cell(x, n, xn) + (k + k1) * (int64_t)n;
            sg[m] = g;
            sell[m] = (D)direct_partial<TQ, P>(x, q, n, len, s, invlen, i0 - H + m, g);
        }
        wave_sync();
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int ci = min(t + u * kLanes, NC - 1);
            const double wh = direct_whole<TQ>(x, q, n, sg[ci], sg[ci + 1]);
            qs[u] = (CT)((D)(wh + ((double)sell[ci + 1] - (double)sell[ci])) / (D)(xr[u] - xe[u]));
        }
    }
    if constexpr (H == 0) {
#pragma unroll
        for (int u = 0; u < NS; ++u)
            if (t + u * kLanes < nd) qo[i0 + t + u * kLanes] = (TQ)qs[u];
        return;
    } else {
        // ---- (E) -------------------------------------------------------------------
        constexpr int NL = kLanes * NS;
        CT *sq = (CT *)su, *sdx = sq + NL, *shv = sdx + NL, *sdi = shv + NL, *sf = sdi + NL;
        TQ *qmid = a.q_mid ? (TQ *)a.q_mid + ti.qoff : nullptr;
        wave_sync();
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int ci = t + u * kLanes;
            if (ci < NC) {
                // centre of the next cell minus this one's
                const double c1 = cell[u] == n - 1 ? 0.5 * (x0 + x2[u]) + len : 0.5 * (xr[u] + x2[u]);
                const double dx = xr[u] - xe[u];
                sq[ci] = qs[u];
                sdx[ci] = (CT)dx;
                shv[ci] = (CT)(1.0 / (c1 - 0.5 * (xe[u] + xr[u])));
                sdi[ci] = (CT)(1.0 / dx);
                if (qmid && ci >= H && ci < H + nd) qmid[cell[u]] = (TQ)qs[u];
            }
        }
        wave_sync();
        // face f, left of shifted cell f (f = 2 .. nd + 2), with cell f's face velocity
        const CT dt = (CT)a.dt;
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int f = t + u * kLanes;
            if (f >= H && f <= nd + H) {
                const bool up = v[u] >= (CT)0;
                const int c = up ? f - 1 : f;        // upwind cell
                const CT qm = sq[c - 1], q0 = sq[c], qp = sq[c + 1];
                const CT dp = (qp - q0) * shv[c];
                const CT dm = (q0 - qm) * shv[c - 1];
                const CT sg = (dp * dm <= (CT)0) ? (CT)0 : harmonic2(dp, dm);
                const CT qf = up ? q0 + (CT)0.5 * sg * (sdx[c] - v[u] * dt)
                                 : q0 - (CT)0.5 * sg * (sdx[c] + v[u] * dt);
                sf[f] = v[u] * qf;
            }
        }
        wave_sync();
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int ci = t + u * kLanes;
            if (ci >= H && ci < H + nd)
                qo[cell[u]] = (TQ)(sq[ci] - dt * (sf[ci + 1] - sf[ci]) * sdi[ci]);
        }
    }
}

template <typename TQ, int P, int S, int NS>
hipError_t rows_ns(const StepArgs &a, int sub, hipStream_t st)
{
    const dim3 g((unsigned)((a.rows.n_tiles * sub + kWaves - 1) / kWaves)), b(kBlock);
    if (a.dv) hipLaunchKernelGGL((k_rows<TQ, P, S, 2, NS>), g, b, 0, st, a, sub);
    else hipLaunchKernelGGL((k_rows<TQ, P, S, 0, NS>), g, b, 0, st, a, sub);
    return hipGetLastError();
}

template <typename TQ, int P, int S>
hipError_t rows_h(const StepArgs &a, hipStream_t st)
{
    const bool fused = a.dv != nullptr;
    if (a.rows.tile == rows_tile(fused, 2)) return rows_ns<TQ, P, S, 2>(a, 1, st);
    const int tile = rows_tile(fused);
    if (a.rows.tile % tile != 0) return hipErrorInvalidValue;
    return rows_ns<TQ, P, S, 4>(a, a.rows.tile / tile, st);
}

template <int P>
hipError_t rows_p(const StepArgs &a, bool f64, int scan, hipStream_t st)
{
    if (f64) return rows_h<double, P, kScanF64>(a, st);
    switch (scan) {
    case kScanF64:
    case kSumDirect: return rows_h<float, P, kScanF64>(a, st);
    case kScanTwoSum: return rows_h<float, P, kScanTwoSum>(a, st);
    default: return rows_h<float, P, kScanF32>(a, st);
    }
}

} // namespace

hipError_t launch_step(const StepArgs &a, bool f64, int scan, int order, hipStream_t stream)
{
    if (a.rows.n_tiles <= 0) return hipSuccess;
    if (a.rag.rec) {
        if (f64) return hipErrorInvalidValue;
        return launch_step_rag(a, order, scan, stream);
    }
    switch (order) {
    case 1: return rows_p<1>(a, f64, scan, stream);
    case 3: return rows_p<3>(a, f64, scan, stream);
    default: return rows_p<5>(a, f64, scan, stream);
    }
}

} // namespace ram
