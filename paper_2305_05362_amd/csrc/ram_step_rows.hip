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
// A window beyond the LDS, or of a row so short that it crosses its end
// more than twice, passes through LDS in pieces (rows_wide).
//
// VALU issue bounds it, with the chain of dependent loads that starts a wave
// (the table, the row, its ends and nodes, two rounds of the window search, the
// window): 2,034 VALU instructions a tile at order 5 with the residual, more than
// half of them the weights of its 256 nodes (an FP64 and five FP32 divisions each)
// and their search in LDS.  1024 rows of 64 .. 4096 cells, FP32, two-sum, with the
// residual: 46 us (31 of them VALU issue); with 1019-cell tiles a workgroup (27 KB
// of LDS, seven barriers, two lanes searching the row for the window while the
// others wait) 74.  Five waves a SIMD spill (51 us; 44 at four then).  Small batches take two node
// slots a lane instead of four: the chain of one wave is what they cost.
#include "ram_rows.h"

#include <type_traits>

namespace ram {
namespace {

using namespace dev;

// Waves a SIMD that the registers allow: only rows_wide spills.
template <typename TQ, int S, int NS> constexpr int rows_waves()
{
    return sizeof(TQ) == 8 ? 3 : (S == kScanF64 || NS == 4 ? 4 : 5);
}

// LDS of one wave: window nodes, later the cumulative; masses; partial
// integrals; window cells of the nodes.  The residual's five arrays reuse it.
// The window takes what that many waves leave of the CU's 160 KB (in allocations of
// 1280 bytes): 704 cells for FP32 prefix sums with four slots, 668 for FP64, 464 for
// FP32 states summed in FP64.
template <typename TQ, int S, int NS> struct RowsLds {
    using M = typename Acc<S>::M;
    using A = typename Acc<S>::A;
    using D = typename std::conditional<std::is_same<TQ, double>::value, double,
                                        typename Acc<S>::D>::type;
    static constexpr size_t wave = 163840 / rows_waves<TQ, S, NS>() / 1280 * 1280 / kWaves;
    static constexpr size_t sell = sizeof(D) * (kLanes * NS);
    static constexpr size_t sjc = sizeof(short) * (kLanes * NS);
    static constexpr int cap = (int)((wave - sell - sjc) / (8 + sizeof(M))) / 4 * 4 - 8;  // cells
    static constexpr size_t xs = 8 * (cap + 8);
    static constexpr size_t sm = sizeof(M) * (cap + 8);
    static constexpr size_t res = 5 * sizeof(TQ) * (kLanes * NS);
    static constexpr size_t bytes = xs + sm + sell;
    static_assert(sizeof(A) <= 8 && 8 * kLanes * NS <= xs && res <= bytes, "the nodes' bytes are used again");
};

// A tile whose window does not fit in LDS: the window in pieces of up to SPAN
// cells, each staged whole (nodes and masses) and starting p - 1 cells before
// the last one's end.  The nodes whose stencil a piece holds get their partial
// integral from it, and every cell adds the piece's share of its whole source
// cells, so that a cell of the row is read once, in whole lines, and nothing but
// those sums outlives a piece.  FP64 throughout; cell ci's mass goes to sell[ci].
// Nodes e0 .. e0 + NE - 1 of the row; the window's start from rows_locate.
//
// Latency bounds it: two or three pieces for a tile of 251 cells on a mesh refined
// tenfold.  A shift of 2.1 M cells in such rows by anything in their period, rows of
// 700, 1000 and 2000 cells, FP32 two-sum: 43, 45 and 59 us, FP64 48, 50 and 65; with
// 448 cells of LDS window and every wider one summed from global memory, a search a
// node and a remainder a cell, 68, 61 and 64, FP64 85, 80 and 82.
template <typename TQ, int P, int NS, int SPAN, typename D>
__device__ __forceinline__ void rows_wide(const double *x, const TQ *q, int n, double s, double x0,
                                          double xN, double len, double invlen, int e0, int NE, int t,
                                          RowsWindow win, double *xs, D *sell, short *sjc)
{
    constexpr int LO = (P - 1) / 2;
    constexpr int NQ = 5;                            // staged cells a lane has in flight
    constexpr int kAhead = 0x7fff;                   // a node of a later piece
    double *sm = xs + SPAN + 1;
    double xh[NS], whole[NS];
    int per[NS], in[NS];                             // period; 0: ahead, 1: in this piece, 2: done
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int m = min(t + u * kLanes, NE - 1);
        int e = e0 + m, kx = 0;
        if (e < 0) { e += n; kx = -1; }
        while (e >= n) { e -= n; kx += 1; }
        int64_t k;
        wrap_node(x[e], s, x0, xN, len, invlen, xh[u], k);
        per[u] = (int)min(max(k + kx - win.k0, (int64_t)-1), (int64_t)1 << 30);
        in[u] = 0;
        whole[u] = 0.0;
        sell[m] = (D)__builtin_nan("");
    }
    // (a tile's nodes span less than two periods, so its window less than 3 n cells)
    int64_t left = min(win.wide, 3 * (int64_t)n);
    int p0 = 0;                                      // the piece's first cell: its period
    bool all = false;
    while (!all && left > 0) {
        const int span = (int)min((int64_t)SPAN, 3 * (int64_t)n - win.base);
        const int step = span - P + 1;
        win.seam = n - win.base;
        win.seam2 = win.seam + n;
        // ---- nodes and masses (lanes past the last cell repeat it) -----------------
#pragma unroll 1
        for (int i0 = t; i0 - t < span; i0 += NQ * kLanes) {
            double xv[NQ], xw[NQ];
            TQ qv[NQ];
#pragma unroll
            for (int u = 0; u < NQ; ++u) {
                const int c = win.at(min(i0 + u * kLanes, span - 1), n);
                xv[u] = x[c];
                xw[u] = x[c + 1];
                qv[u] = q[c];
            }
#pragma unroll
            for (int u = 0; u < NQ; ++u) {
                const int i = min(i0 + u * kLanes, span - 1);
                xs[i] = xv[u];
                sm[i] = (double)qv[u] * (xw[u] - xv[u]);
                // (the node after the last cell: the row's first again past its end)
                if (i == span - 1) xs[span] = win.at(span, n) == 0 ? x0 : xw[u];
            }
        }
        wave_sync();
        // ---- which nodes, and where ------------------------------------------------
        int dk[NS], j[NS];
#pragma unroll
        for (int u = 0; u < NS; ++u) dk[u] = min(max(per[u] - p0, 0), 2);
        rows_search<NS>(xs, win, span, xh, dk, j);
        bool done = true;
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const bool here = in[u] == 0 && dk[u] == per[u] - p0 && j[u] >= LO && j[u] < LO + step &&
                              xs[j[u]] <= xh[u];
            in[u] = here ? 1 : (in[u] != 0 ? 2 : 0);
            j[u] = min(max(j[u], LO), LO + step - 1);
            sjc[min(t + u * kLanes, NE - 1)] = (short)(in[u] == 1 ? j[u] : (in[u] == 2 ? 0 : kAhead));
            done = done && in[u] != 0;
        }
        // ---- their partial integrals (one copy of the code: the slots move past it) --
#pragma unroll 1
        for (int u = 0; u < NS; ++u) {
            if (__any(in[0] == 1 ? 1 : 0)) {
                double w[P + 1];
                rows_weights<double, P, true>(xs, win, len, xh[0], j[0], w);
                double ell = 0.0, up = 0.0, dn = 0.0;
#pragma unroll
                for (int b = LO + 1; b <= P; ++b) {
                    up += sm[j[0] + b - LO - 1];
                    ell += w[b] * up;
                }
#pragma unroll
                for (int b = LO - 1; b >= 0; --b) {
                    dn += sm[j[0] - LO + b];
                    ell -= w[b] * dn;
                }
                if (in[0] == 1) sell[min(t + u * kLanes, NE - 1)] = (D)ell;
            }
            slot_turn(xh);
            slot_turn(in);
            slot_turn(j);
        }
        wave_sync();
        // ---- the piece's share of the whole source cells -----------------------------
        all = __all(done ? 1 : 0) != 0;
        left -= step;
        win.base += step;
        const int over = win.base / n;
        win.base -= over * n;
        p0 += over;
        int ja[NS], jb[NS];
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int ci = min(t + u * kLanes, NE - 2);
            ja[u] = max((int)sjc[ci], LO);
            jb[u] = min((int)sjc[ci + 1], LO + step);
        }
        // (every slot's next two cells at once)
        for (;;) {
            bool more = false;
            double m0[NS], m1[NS];
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                const int i = min(ja[u], LO + step - 1);
                m0[u] = sm[i];
                m1[u] = sm[i + 1];
            }
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                if (ja[u] < jb[u]) whole[u] += m0[u];
                if (ja[u] + 1 < jb[u]) whole[u] += m1[u];
                ja[u] += 2;
                more = more || ja[u] < jb[u];
            }
            if (!__any(more ? 1 : 0)) break;
        }
        wave_sync();
    }
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int ci = min(t + u * kLanes, NE - 2);
        whole[u] += (double)sell[ci + 1] - (double)sell[ci];
    }
    wave_sync();
#pragma unroll
    for (int u = 0; u < NS; ++u) sell[min(t + u * kLanes, NE - 2)] = (D)whole[u];
    wave_sync();
}

// NS: node slots a lane.
template <typename TQ, int P, int S, int H, int NS>
__global__ __launch_bounds__(kBlock, (rows_waves<TQ, S, NS>())) void k_rows(StepArgs a)
{
    using AC = Acc<S>;
    using L = RowsLds<TQ, S, NS>;
    using M = typename L::M;
    using A = typename L::A;
    using D = typename L::D;
    using CT = TQ;
    constexpr int LO = (P - 1) / 2;
    constexpr bool kLocal = S == kScanF64;           // sums of the FP64 masses between
    constexpr int NDT = kLanes * NS - 1 - 2 * H;     // destination cells
    constexpr int NQ = 5;                            // window slots loaded ahead
    constexpr int NR = 4;                            // and of a longer one a round
    __shared__ __attribute__((aligned(16))) unsigned char su_[kWaves][L::bytes];
    __shared__ short sjc_[kWaves][kLanes * NS];
    const int wid = wave_id();
    const int t = (int)threadIdx.x % kLanes;
    const int64_t tile = (int64_t)blockIdx.x * kWaves + wid;
    const Rows &R = a.rows;
    if (tile >= R.n_tiles) return;
    Tile ti;
    if (!get_tile(R, tile, ti)) return;
    const int n = ti.n;
    const int i0 = ti.i0;
    if (n < P + 1) return;
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
        x, n, s, x0, xN, len, invlen, NE, t, L::cap, xe, kx, xs, win, xh, j, [&] {
#pragma unroll
            for (int u = 0; u < NQ; ++u) qv[u] = q[win.at(min(t + u * kLanes, win.w - 1), n)];
        });
    CT qs[NS];
    double x2[NS];                                   // the residual's: the next cell's right node
    if constexpr (H != 0) {
#pragma unroll
        for (int u = 0; u < NS; ++u) x2[u] = x[cell[u] + 2 <= n ? cell[u] + 2 : 1];
    }
    if (__builtin_expect(windowed, 1)) {
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
        for (int i0 = t + NQ * kLanes; i0 - t < W; i0 += NR * kLanes) {
            TQ v[NR];
#pragma unroll
            for (int u = 0; u < NR; ++u) v[u] = q[win.at(min(i0 + u * kLanes, W - 1), n)];
#pragma unroll
            for (int u = 0; u < NR; ++u) {
                const int i = i0 + u * kLanes;
                if (i < W) sm[i] = AC::template mass<TQ>(v[u], rows_size(xs, win, xN, i));
            }
        }
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
        constexpr int kSpan = (int)((L::xs + L::sm) / 16) - 1;
        wave_sync();
        // (the nodes, their cells' geometry and velocities are read again, at an offset
        // of 0 that the compiler does not see: held in registers all along, they would
        // be spilled, by the other tiles too)
        int zero = 0;
        asm volatile("" : "+s"(zero));
        const double *xz = x + zero;
        rows_wide<TQ, P, NS, kSpan, D>(xz, q, n, s, x0, xN, len, invlen, i0 - H, NE, t, win, xs, sell, sjc);
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int c = cell[u];
            xe[u] = xz[c];
            xr[u] = xz[c + 1];
            if constexpr (H != 0) {
                x2[u] = xz[c + 2 <= n ? c + 2 : 1];
                v[u] = (CT)((const TQ *)a.dv + ti.qoff + zero)[c];
            }
        }
#pragma unroll
        for (int u = 0; u < NS; ++u) qs[u] = (CT)(sell[min(t + u * kLanes, NC - 1)] / (D)(xr[u] - xe[u]));
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
hipError_t rows_ns(const StepArgs &a, hipStream_t st)
{
    const dim3 g((unsigned)((a.rows.n_tiles + kWaves - 1) / kWaves)), b(kBlock);
    if (a.dv) hipLaunchKernelGGL((k_rows<TQ, P, S, 2, NS>), g, b, 0, st, a);
    else hipLaunchKernelGGL((k_rows<TQ, P, S, 0, NS>), g, b, 0, st, a);
    return hipGetLastError();
}

template <typename TQ, int P, int S>
hipError_t rows_h(const StepArgs &a, hipStream_t st)
{
    const bool fused = a.dv != nullptr;
    if (a.rows.tile == rows_tile(fused, 2)) return rows_ns<TQ, P, S, 2>(a, st);
    if (a.rows.tile == rows_tile(fused, 4)) return rows_ns<TQ, P, S, 4>(a, st);
    return hipErrorInvalidValue;
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
