// ram_step_fast.hip -- the FP32 RAM step on rows that share one mesh, with the
// cumulative differences summed directly from the window masses (gfx950).
//
// Same computation as k_step_sh with direct sums (bulk shift of Section 3,
// Steps 1-3, Eqs. Qmass_i, condition_p, mass_shift_algo, step3, then the
// residual upwind step with the van Leer slope of Section 3.1), laid out for
// streaming rather than for the node search:
//
//   * one tile of kFastTile = 256 destination cells per wave, four
//     consecutive cells a lane, whose residual-velocity loads and final
//     stores are 16-byte vector accesses; each wave has its own LDS and never
//     waits on the other waves of its workgroup (no workgroup barrier);
//   * everything about a tile that does not change between steps is planned
//     once per call: its source window, whether it lies in one of the mesh's
//     uniform runs (then the stencil weights and the run's geometry), and if
//     not each shifted node's window index and position in its cell;
//   * a tile in a uniform run (every node of the tile in the next source cell
//     at one theta) needs no search and no masses: the shifted value of a
//     cell is a fixed (P+1)-point stencil on the window's cell values.  Those
//     tiles run in their own kernel (k_step_uni, 26 registers, eight waves a
//     SIMD) as straight-line code: the window and face loads issued together,
//     the window through the wave's LDS once, each lane reading the thirteen
//     values its eight cells need (its four and the residual's two-cell halo
//     a side) with 16-byte LDS reads, and the residual on registers;
//   * the other tiles (k_step_gen) stage the window masses M = Q dx in LDS,
//     read their nodes' planned window index and theta, then each node's
//     stencil record for its Lagrange weights and partial integral, then the
//     destination masses one cell per lane, and the same register residual on
//     four consecutive cells; a tile whose window exceeds the LDS capacity
//     sums from global memory.
// Tiles of 256 cells keep the searching tiles to the cells near the mesh's
// non-uniform stretches.
#include "ram_node64.h"
#include "ram_rows.h"

#include <type_traits>

namespace ram {
namespace {

using namespace dev;

constexpr int kFT = kFastTile;                      // destination cells per tile (wave)
constexpr int kFPad = 16;                           // slack for vector over-reads

// LDS of one wave.  The window (values or masses), the direct path's extended
// node indices and the shifted state share bytes (the wave moves from one to
// the next after a wave-level fence); node partials and their window indices
// have arrays of their own.
struct WaveLds {
    static constexpr int nodes = kFT + 5 + 3;       // up to 261 nodes, padded
    static constexpr size_t win = sizeof(float) * (kFastWin + kFPad);
    static constexpr size_t gidx = sizeof(int64_t) * nodes;
    static constexpr size_t shifted = sizeof(float) * (kFT + 4 + kFPad);
    static constexpr size_t u0 = win > gidx ? win : gidx;
    static constexpr size_t u = u0 > shifted ? u0 : shifted;
    // the prefix modes keep the window's cumulative (8-byte values: FP64, or
    // a two-sum pair) instead of its masses
    static constexpr size_t pre = 8 * (kFastWin + 16);
    static constexpr size_t u_pre = pre > u ? pre : u;
};
template <int S> constexpr size_t wave_lds_bytes()
{
    return S == kSumDirect ? WaveLds::u : WaveLds::u_pre;
}


// The record of each tile: which path, its window, and for a uniform tile the
// stencil and the run's geometry; and of each group which tiles are in no run.
// A wave plans kPlanGroup tiles, two lanes each (plan_tile).  About six
// dependent loads bound it, whatever the size.
template <int P>
__global__ __launch_bounds__(kLanes) void k_plan_fast(StepArgs a, FastPlan pl)
{
    static_assert(2 * kPlanGroup == kLanes, "two lanes a tile");
    __shared__ FastTile srec[kPlanGroup];
    const int nt = (int)a.rows.n_tiles;
    const int first = (int)blockIdx.x * kPlanGroup;
    const int t = (int)threadIdx.x;
    const bool valid = first + (t >> 1) < nt;
    const FastTile ft = plan_tile<P>(a, min(first + (t >> 1), nt - 1), a.dv ? 2 : 0, t);
    if ((t & 1) == 0) srec[t >> 1] = ft;
    uint64_t mo = __ballot(ft.kind != kFastUniform && valid);           // bits 2 u and 2 u + 1: tile first + u
    mo &= 0x5555555555555555ull;
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {               // even bits together
        const uint64_t keep = d == 1 ? 0x3333333333333333ull : d == 2 ? 0x0f0f0f0f0f0f0f0full
                            : d == 4 ? 0x00ff00ff00ff00ffull : d == 8 ? 0x0000ffff0000ffffull
                                                                      : 0x00000000ffffffffull;
        mo = (mo | mo >> d) & keep;
    }
    if (t == 0) pl.mask[blockIdx.x] = (uint32_t)mo;
    wave_sync();
    // the records out, kWords lanes a record
    constexpr int kWords = (int)(sizeof(FastTile) / 4);
    constexpr int kPer = kLanes / kWords;
#pragma unroll
    for (int k = 0; k < kPlanGroup / kPer; ++k) {
        const int u = k * kPer + t / kWords, wd = t % kWords;
        if (first + u < nt) ((int32_t *)(pl.rec + first + u))[wd] = ((const int32_t *)&srec[u])[wd];
    }
}

// Residual step on four consecutive cells of a lane from the shifted state
// s[0..7] of cells i0+4l-2 .. i0+4l+5 (Section 3.1's upwind step with the van
// Leer slope, the face state the upwind linear profile averaged over the
// interval the face velocity sweeps in dt): fluxes on the
// five faces i0+4l .. i0+4l+4 with the upwind cell's van Leer slope and the
// swept-interval average, then the conservative update of the four cells.
// rr(c) gives (dx, 1/centre gap to the right) of s-index c, dxi(k) 1/dx of
// own cell k.
template <typename RR, typename DXI>
__device__ __forceinline__ void residual4(const float *s, const float *dvv, float dt, RR rr,
                                          DXI dxi, float *out)
{
    float F[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const float v = dvv[k];
        const bool up = v >= 0.0f;
        // upwind cell: s-index k+1 (left of the face) or k+2
        const float qm = up ? s[k] : s[k + 1];
        const float q0 = up ? s[k + 1] : s[k + 2];
        const float qp = up ? s[k + 2] : s[k + 3];
        const float2 rc = up ? rr(k + 1) : rr(k + 2);
        const float gm = up ? rr(k).y : rr(k + 1).y;
        const float dp = (qp - q0) * rc.y;
        const float dm = (q0 - qm) * gm;
        const float sig = (dp * dm <= 0.0f) ? 0.0f : harmonic2(dp, dm);
        const float half = up ? 0.5f * (rc.x - v * dt) : -0.5f * (rc.x + v * dt);
        F[k] = v * (q0 + sig * half);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) out[k] = s[k + 2] - dt * (F[k + 1] - F[k]) * dxi(k);
}


// Four consecutive cells at any cell of a row: global loads and stores need
// only their word's alignment, so rows whose length is not a multiple of four
// (VEC false below) take 16-byte accesses too, wherever the four cells lie in
// the row (`full`: the tile and one cell beyond do, for every lane).
struct f4u {
    float __attribute__((ext_vector_type(4), aligned(4))) v;
};
struct f2u {
    float __attribute__((ext_vector_type(2), aligned(4))) v;
};

// Residual velocity of faces i0+4l .. i0+4l+4 of a row (face n is face 0);
// lanes past the tile read its last faces again (every load issued, no
// branch).
template <bool VEC>
__device__ __forceinline__ void load_faces(const float *dvp, int n, int i0, int nd, int c4,
                                           float *dvv)
{
    const int cc = min(c4, nd - 1);
    if constexpr (VEC) {
        const float4 v4 = ld_at<float4>(dvp + i0, 4u * (uint32_t)(cc & ~3));
        dvv[0] = v4.x;
        dvv[1] = v4.y;
        dvv[2] = v4.z;
        dvv[3] = v4.w;
    } else if (nd == kFT) {                          // cells i0 .. i0 + 255 in the row
        const auto v4 = ld_at<f4u>(dvp + i0, 4u * (uint32_t)c4).v;
        dvv[0] = v4.x;
        dvv[1] = v4.y;
        dvv[2] = v4.z;
        dvv[3] = v4.w;
    } else {
        // faces up to the tile's right face i0 + nd
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int f = i0 + min(cc + k, nd);
            dvv[k] = dvp[f >= n ? f - n : f];
        }
    }
    const int f4 = i0 + min(cc + 4, nd);
    dvv[4] = dvp[f4 >= n ? f4 - n : f4];
}

template <bool VEC>
__device__ __forceinline__ void store_cells(float *qo, int i0, int nd, int c4, const float *o)
{
    if constexpr (!VEC) {
        if (nd == kFT) {
            st_at<f4u>(qo + i0, 4u * (uint32_t)c4, {{o[0], o[1], o[2], o[3]}});
            return;
        }
    }
    if (c4 >= nd) return;
    if constexpr (VEC) {
        st_at<float4>(qo + i0, 4u * (uint32_t)c4, make_float4(o[0], o[1], o[2], o[3]));
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c4 + k < nd) qo[i0 + c4 + k] = o[k];
    }
}



// ---------------------------------------------------------------------------
// A tile in a uniform run of the mesh: straight-line code (clamped indices
// instead of guards), the window's and the faces' loads issued together.
// ---------------------------------------------------------------------------

constexpr int kUniWin = 5 * kLanes + 16;            // window slots + over-read slack, floats

// A tile in a uniform run.  VEC: rows of a multiple of four cells (16-byte
// aligned vector loads of the residual velocity, vector stores of the
// result).  Rows need at least kFT + 2H + P cells (k_plan_fast sends shorter
// ones to the other path), so a window wraps the row at most once.
template <int P, int H, bool VEC>
__device__ __forceinline__ void uniform_tile(const StepArgs &a, const FastTile &r, float *sw,
                                             int t)
{
    constexpr int NV = 4 + 2 * H;                    // shifted cells a lane reads
    constexpr int NW = (NV + P + 3) / 4 * 4;         // window values, whole float4s
    constexpr int NUW = (kFT + 2 * H + P + kLanes - 1) / kLanes;  // window slots a lane
    static_assert(NUW * kLanes <= kUniWin && 4 * (kLanes - 1) + NW <= kUniWin, "window");
    const int n = (int)a.rows.n_cols;
    const float dt = (float)a.dt;
    const int c4 = 4 * t;
    const TilePos p = tile_pos(r.pad[0], n, H);
    const int64_t qoff = (int64_t)p.row * n;

    // window cells j = t + 64k (clamped into the window: the extra lanes read
    // its last cell again) and face velocities i0+4l .. i0+4l+4 (clamped into
    // the tile, face n is face 0)
    float wv[NUW];
    {
        const float *q = (const float *)a.q_in + qoff;
#pragma unroll
        for (int k = 0; k < NUW; ++k) {
            int mm = r.base + min(t + k * kLanes, r.w - 1);
            mm = mm >= n ? mm - n : mm;
            wv[k] = q[mm];
        }
    }
    float dvv[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
    if constexpr (H != 0) load_faces<VEC>((const float *)a.dv + qoff, n, p.i0, p.nd, c4, dvv);
#pragma unroll
    for (int k = 0; k < NUW; ++k) sw[t + k * kLanes] = wv[k];
    wave_sync();
    // shifted cells ci = 4l .. 4l+NV-1 of the tile (cell i0-H+ci) from window
    // cells ci .. ci+P
    float win[NW];
#pragma unroll
    for (int v = 0; v < NW / 4; ++v) {
        const float4 w4 = *(const float4 *)(sw + c4 + 4 * v);
        win[4 * v] = w4.x;
        win[4 * v + 1] = w4.y;
        win[4 * v + 2] = w4.z;
        win[4 * v + 3] = w4.w;
    }
    float s[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        float v = 0.0f;
#pragma unroll
        for (int d = 0; d <= P; ++d) v += r.cc[d] * win[c + d];
        s[c] = v;
    }
    float *qo = (float *)a.q_out + qoff;
    if constexpr (H == 0) {
        store_cells<VEC>(qo, p.i0, p.nd, c4, s);
    } else {
        if (a.q_mid) store_cells<VEC>((float *)a.q_mid + qoff, p.i0, p.nd, c4, s + 2);
        const float2 g = make_float2(r.dx, r.hinv);
        const float dxi = r.dxinv;
        float o[4];
        residual4(s, dvv, dt, [&](int) { return g; }, [&](int) { return dxi; }, o);
        store_cells<VEC>(qo, p.i0, p.nd, c4, o);
    }
}

// ---------------------------------------------------------------------------
// Every other tile.  Its nodes' source cells do not change between the steps
// of a call, so k_plan_nodes locates them once (bucket index, Eq.
// condition_p) and keeps each node's window index and theta; per step a wave
// then needs two round trips to memory: the window, node data, faces and
// geometry together, then the source cells' stencil records.
// ---------------------------------------------------------------------------

// The second half of the plan, in two parts side by side.
//
// Lists (workgroups 0 .. lists - 1, a thread a tile): the records of the
// uniform tiles in tile order without gaps, and the ids of the others.  Tile
// order, because the uniform kernel on the 2048 x 16384 disk takes 70 us in it
// and 80 when neighbouring waves run tiles of rows far apart (lists filled by
// atomics); no gaps, because a wave that finds no tile of its kind keeps its
// share of the workgroup's LDS from others (searching kernel 47 against 39 us
// there).
//
// Nodes (the other workgroups, kNodeTiles tiles each, whose searching tiles
// its waves take in turn): window index and FP32 theta of nodes i0-H ..
// i0+nd+H, and in the slots past the last node (up to kFastNodes) the last node
// again, so that whole 16-byte groups of slots can be read; a node outside the
// window (not expected: the plan sized it from the end nodes) turns the tile
// into a direct one.
constexpr int kNodeTiles = 8;

// Rows a multiple of eight workgroups long have their searching tiles in the
// same workgroups of every row, and workgroups go to the chip's eight XCDs in
// turn: each run of eight is rotated by its number (and by the number's higher
// octal digits), so that every XCD gets its share.
__device__ __forceinline__ int spread8(int b)
{
    const int o = b >> 3;
    return (b & ~7) | ((b + o + (o >> 3) + (o >> 6) + (o >> 9)) & 7);
}

__device__ __forceinline__ void plan_lists(const FastPlan &pl, int nt, int block)
{
    __shared__ int sred[kWaves];
    const int t = (int)threadIdx.x;
    constexpr int kGroups = kBlock / kPlanGroup;     // groups of this workgroup's tiles
    const int g0 = block * kGroups, ng = (nt + kPlanGroup - 1) / kPlanGroup;
    // the other tiles before this workgroup's
    int before = 0;
    for (int g = t; g < g0; g += kBlock) before += __popc(pl.mask[g]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) before += __shfl_xor(before, d);
    if (t % kLanes == 0) sred[t / kLanes] = before;
    uint32_t m[kGroups];
#pragma unroll
    for (int k = 0; k < kGroups; ++k) m[k] = g0 + k < ng ? pl.mask[g0 + k] : 0;
    __syncthreads();
    before = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) before += sred[w];
    const int tile = block * kBlock + t;
    const int bit = t % kPlanGroup;
    bool other = false;
    int all = before;
#pragma unroll
    for (int k = 0; k < kGroups; ++k) {
        if (k == t / kPlanGroup) {
            before = all + __popc(m[k] & ((1u << bit) - 1u));
            other = (m[k] >> bit & 1u) != 0;
        }
        all += __popc(m[k]);
    }
    if (tile < nt) {
        if (other) {
            pl.oid[before] = tile;
        } else {
            const float4 *from = (const float4 *)(pl.rec + tile);
            float4 *to = (float4 *)(pl.urec + (tile - before));
            const float4 v0 = from[0], v1 = from[1], v2 = from[2], v3 = from[3];
            to[0] = v0;
            to[1] = v1;
            to[2] = v2;
            to[3] = v3;
        }
        if (tile == nt - 1) {
            pl.totals[0] = nt - all;
            pl.totals[1] = all;
        }
    }
}

template <int P>
__global__ __launch_bounds__(kBlock) void k_plan_nodes(StepArgs a, int lists)
{
    constexpr int LO = (P - 1) / 2;
    constexpr int NS = (kFastNodes + kLanes - 1) / kLanes;
    const int nt = (int)a.rows.n_tiles;
    if ((int)blockIdx.x < lists) {
        plan_lists(a.fast, nt, (int)blockIdx.x);
        return;
    }
    const int first = spread8((int)blockIdx.x - lists) * kNodeTiles;
    if (first >= nt) return;
    uint32_t todo = a.fast.mask[first / kPlanGroup] >> (first % kPlanGroup) & ((1u << kNodeTiles) - 1u);
    const int wid = wave_id();
    const MeshTab &tb = a.rows.tab;
    const int n = (int)a.rows.n_cols;
    const int H = a.dv ? 2 : 0;
    const int t = (int)threadIdx.x % kLanes;
    const double *x = a.rows.edges;
    const double x0 = x[0], xN = x[n];
    const double len = xN - x0;
    for (int turn = 0; todo != 0; ++turn) {
        const int tile = first + __ffs((int)todo) - 1;
        todo &= todo - 1;
        if (turn % kWaves != wid) continue;
        const FastTile ft = load_rec(a.fast.rec, tile);
        if (ft.kind != kFastWindow) continue;
        const TilePos tp = tile_pos(tile, n, H);
        const int NE = tp.nd + 2 * H + 1;
        const RowShift rs = row_shift(a.v0[tp.row] * a.dt, len, tb.scal[1]);
        const int64_t wlo = (int64_t)(((uint64_t)(uint32_t)ft.wlo_hi << 32) | (uint32_t)ft.wlo_lo);
        const int jbase = (int)(rs.kf0 * (int64_t)n - wlo);
        float *th = a.fast.theta + (int64_t)tile * kFastNodes;
        int16_t *jcw = a.fast.jc + (int64_t)tile * kFastNodes;
        // (lanes past the last slot repeat it)
        int ce[NS], kx[NS];
        double xt[NS];
        locate_nodes<NS>(x, n, tb, rs, x0, xN, tp.i0 - H, NE, t, ce, kx, xt);
        double xc[NS], di[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            xc[s] = x[ce[s]];
            di[s] = tb.dxinv[ce[s]];
        }
        bool ok = true;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int m = min(t + s * kLanes, kFastNodes - 1);
            const int j = ce[s] + kx[s] + jbase;
            ok = ok && j >= LO && j + P - LO <= ft.w;
            th[m] = (float)((xt[s] - xc[s]) * di[s]);
            jcw[m] = (int16_t)min(max(j, 0), kFastWin);
        }
        if (!__all(ok ? 1 : 0) && t == 0) a.fast.rec[tile].kind = kFastDirect;
    }
}

// The window index and FP32 theta of a searching tile's nodes, as the tile's code
// takes them when it needs them: from the call's node plan, or (one step) located
// before by the same arithmetic.
template <int H> constexpr int kNodeSlots = (kFT + 2 * H + 1 + kLanes - 1) / kLanes;
template <int H> struct PlannedNodes {
    const float *theta;
    const int16_t *jc;
    __device__ __forceinline__ PlannedNodes(const StepArgs &a, const FastTile &ft)
        : theta(a.fast.theta + (int64_t)ft.pad[1] * kFastNodes),
          jc(a.fast.jc + (int64_t)ft.pad[1] * kFastNodes)
    {
    }
    __device__ __forceinline__ void get(int t, float (&thv)[kNodeSlots<H>], int (&jv)[kNodeSlots<H>]) const
    {
#pragma unroll
        for (int u = 0; u < kNodeSlots<H>; ++u) {
            const int m = min(t + u * kLanes, kFastNodes - 1);
            thv[u] = theta[m];
            jv[u] = jc[m];
        }
    }
};
template <int H> struct LocatedNodes {
    float th[kNodeSlots<H>];
    int j[kNodeSlots<H>];
    // false: a node is not in the window
    template <int P> __device__ __forceinline__ bool locate(const StepArgs &a, const FastTile &ft, int t)
    {
        constexpr int NS = kNodeSlots<H>;
        const MeshTab &tb = a.rows.tab;
        const int n = (int)a.rows.n_cols;
        const TilePos tp = tile_pos(ft.pad[0], n, H);
        const double *x = a.rows.edges;
        const double x0 = x[0], xN = x[n];
        const RowShift rs = row_shift(a.v0[tp.row] * a.dt, xN - x0, tb.scal[1]);
        int ce[NS], kx[NS];
        double xt[NS];
        locate_nodes<NS>(x, n, tb, rs, x0, xN, tp.i0 - H, tp.nd + 2 * H + 1, t, ce, kx, xt);
#pragma unroll
        for (int u = 0; u < NS; ++u) th[u] = (float)((xt[u] - x[ce[u]]) * tb.dxinv[ce[u]]);
        return window_indices<P, NS>(ce, kx, rs, n, ft, j);
    }
    __device__ __forceinline__ void get(int, float (&thv)[kNodeSlots<H>], int (&jv)[kNodeSlots<H>]) const
    {
#pragma unroll
        for (int u = 0; u < kNodeSlots<H>; ++u) {
            thv[u] = th[u];
            jv[u] = j[u];
        }
    }
};

// LDS window of the limited step's searching tiles, in cells: four arrays of
// it (masses; averages, later the cubics' C; slopes or PLM kappa, later A;
// PPM interface values).  Wider windows take the global-memory path.
constexpr int kGenLimWin = 400;
constexpr size_t kGenLimLds = 4 * sizeof(float) * (kGenLimWin + 8);

// A searching tile's window for the limited step (Section 3.1, App. A): the
// window's masses and averages in LDS, then one pass a stage over the window
// cells -- the limited slopes (PPM; PLM: kappa = sigma dx^2 / 2), the PPM
// interface values, each cell's constrained parabola as the cubic
// ell(theta) = theta (A + theta (B + theta C)), B = M - A - C -- with the
// mesh's weights of each cell, then each node's cubic at its planned theta.
// Node m's window index goes to sjc[m], its partial integral to sell[m].
template <int LR, int NS>
__device__ __forceinline__ void lim_window_partials(const StepArgs &a, const MeshTab &tb, int n,
                                                    int base, int W, int NE, int64_t qoff,
                                                    int t, const float (&thv)[NS],
                                                    const int (&jv)[NS], float *su,
                                                    float *sell, short *sjc)
{
    constexpr int CAP = kGenLimWin + 8;
    float *sw = su;                                  // masses
    float *sq = su + CAP;                            // averages, then C
    float *sd = su + 2 * CAP;                        // slopes or kappa, then A
    float *si = su + 3 * CAP;                        // PPM interface values
    const float *q = (const float *)a.q_in + qoff;
    auto cell = [&](int j) { const int c = base + j; return c >= n ? c - n : c; };
    for (int j = t; j < W; j += kLanes) {
        const int c = cell(j);
        const float qv = q[c];
        sq[j] = qv;
        sw[j] = qv * tb.dxf[c];
    }
    wave_sync();
    const float *pw = tb.ppmf;
    for (int j = t; j < W; j += kLanes) {
        if (j < 1 || j > W - 2) continue;
        const int c = cell(j);
        if constexpr (LR == kReconPPM) {
            sd[j] = ppm_delta<float>(sq[j - 1], sq[j], sq[j + 1], pw[c], pw[n + c]);
        } else {
            const float gp = tb.hinvf[c], gm = tb.hinvf[c == 0 ? n - 1 : c - 1];
            const float dp = (sq[j + 1] - sq[j]) * gp, dm = (sq[j] - sq[j - 1]) * gm;
            const float sig = (dp * dm <= 0.0f) ? 0.0f : harmonic2(dp, dm);
            const float h = tb.dxf[c];
            sd[j] = 0.5f * sig * h * h;
        }
    }
    wave_sync();
    if constexpr (LR == kReconPPM) {
        // interface values between window cells j and j+1, j = 1 .. W-3
        for (int j = t; j < W; j += kLanes) {
            if (j < 1 || j > W - 3) continue;
            const int c = cell(j);
            si[j] = sq[j] + pw[2 * n + c] * (sq[j + 1] - sq[j]) + pw[3 * n + c] * sd[j + 1] +
                    pw[4 * n + c] * sd[j];
        }
        wave_sync();
        // constrained parabolas of window cells 2 .. W-3: A into sd, C into sq
        for (int j = t; j < W; j += kLanes) {
            if (j < 2 || j > W - 3) continue;
            float pa, pb, pc;
            ppm_cubic<float>(sq[j], si[j - 1], si[j], tb.dxf[cell(j)], pa, pb, pc);
            sd[j] = pa;
            sq[j] = pc;
        }
        wave_sync();
    }
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int m = min(t + u * kLanes, NE - 1);
        const int k = jv[u];
        const float th = thv[u];
        float ell;
        if constexpr (LR == kReconPPM) {
            const float pa = sd[k], pc = sq[k];
            const float pb = sw[k] - pa - pc;
            ell = th * (pa + th * (pb + th * pc));
        } else {
            const float kap = sd[k];
            ell = th * (sw[k] - kap + th * kap);
        }
        sell[m] = ell;
        sjc[m] = (short)k;
    }
    wave_sync();
}

// LR != 0: the limited reconstruction LR (PLM / PPM, P its plan order): a
// window of at most kGenLimWin cells is tabulated in LDS (lim_window_partials,
// su then holds kGenLimLds bytes); wider ones take the global-memory path,
// each node's partial integral the limited profile of its cell (Section 3.1).
template <int P, int H, bool VEC, int LR, class Nodes>
__device__ __forceinline__ void general_tile(const StepArgs &a, const FastTile &ft, bool located,
                                             const Nodes &nodes, unsigned char *su, float *sell,
                                             short *sjc, int t)
{
    constexpr int LO = (P - 1) / 2;
    constexpr int NV = 4 + 2 * H;                    // shifted cells a lane reads
    constexpr int NCS = (kFT + 2 * H + kLanes - 1) / kLanes;      // cell slots
    constexpr int NS = (kFT + 2 * H + 1 + kLanes - 1) / kLanes;   // node slots
    const Rows &R = a.rows;
    float *sw = (float *)su;                         // window masses
    int64_t *sg = (int64_t *)su;                     // direct path: node indices
    float *sq = (float *)su;                         // shifted state
    const MeshTab &tb = R.tab;
    const int n = (int)R.n_cols;
    const int c4 = 4 * t;
    const float dt = (float)a.dt;
    const TilePos tp = tile_pos(ft.pad[0], n, H);
    const int row = tp.row, i0 = tp.i0, nd = tp.nd;
    const bool inner = tp.inner;
    const int NC = nd + 2 * H;
    const int NE = NC + 1;
    const int64_t qoff = (int64_t)row * n;
    const float *q = (const float *)a.q_in + qoff;
    float *qo = (float *)a.q_out + qoff;
    float *qmid = a.q_mid ? (float *)a.q_mid + qoff : nullptr;
    const int W = ft.w, base = ft.base;
    const bool windowed =
        located && (LR == 0 || (ft.w <= kGenLimWin && ft.w + ft.base <= 2 * n));

    if (windowed) {
        // ---- round trip 1: window masses, the nodes' window index and theta
        float thv[NS];
        int jv[NS];
        nodes.get(t, thv, jv);
        if constexpr (LR != 0) {
            lim_window_partials<LR, NS>(a, tb, n, base, W, NE, qoff, t, thv, jv, (float *)su,
                                        sell, sjc);
        } else {
        // window masses M = Q dx, four slots of loads at a time, every load
        // issued (clamped into the window) so that no per-slot branch makes
        // the wave wait for each load in turn
        const int nws = (W + kLanes - 1) / kLanes;
        if (W + base <= 2 * n) {
            for (int r0 = 0; r0 < nws; r0 += 4) {
                float wq[4], wd[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    int mm = base + min(t + (r0 + u) * kLanes, W - 1);
                    mm = mm >= n ? mm - n : mm;
                    wq[u] = q[mm];
                    wd[u] = tb.dxf[mm];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (r0 + u < nws) sw[t + (r0 + u) * kLanes] = wq[u] * wd[u];
            }
        } else {
            // rows shorter than the window: it wraps several times
            for (int j = t; j < W; j += kLanes) {
                const int mm = wrap_small(base + j, n);
                sw[j] = q[mm] * tb.dxf[mm];
            }
        }
        wave_sync();
        // ---- round trip 2: each node's stencil record, then its partial
        // integral C~(x) - C(c) from the masses between (summed outward)
        // (the lanes past the last node repeat it: same values, same LDS slot)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int m = min(t + s * kLanes, NE - 1);
            {
                const int j = jv[s];
                int c = base + j;
                c = c >= n ? c - n : c;
                c = c >= n ? wrap_small(c, n) : c;
                const CellRec<float> &rc = RecT<float>::get(tb)[c];
                float wk[P + 1];
                {
                    const float th = thv[s];
                    float tt[P + 1], pre[P + 1], suf[P + 1];
#pragma unroll
                    for (int b = 0; b <= P; ++b) tt[b] = th - rc.th[b];
                    pre[0] = 1.0f;
#pragma unroll
                    for (int b = 1; b <= P; ++b) pre[b] = pre[b - 1] * tt[b - 1];
                    suf[P] = 1.0f;
#pragma unroll
                    for (int b = P - 1; b >= 0; --b) suf[b] = suf[b + 1] * tt[b + 1];
#pragma unroll
                    for (int b = 0; b <= P; ++b) wk[b] = rc.rd[b] * (pre[b] * suf[b]);
                }
                float ell = 0.0f, up = 0.0f, dn = 0.0f;
#pragma unroll
                for (int b = LO + 1; b <= P; ++b) {
                    up += sw[j + b - LO - 1];
                    ell += wk[b] * up;
                }
#pragma unroll
                for (int b = LO - 1; b >= 0; --b) {
                    dn += sw[j - LO + b];
                    ell -= wk[b] * dn;
                }
                sell[m] = ell;
                sjc[m] = (short)j;
            }
        }
        wave_sync();
        }
    } else {
        // window wider than the LDS buffer: nodes located here, partial
        // integrals and whole-cell sums from global memory, in FP64
        const double *x = R.edges;
        const double x0 = x[0], xN = x[n];
        const double len = xN - x0;
        const double sh = a.v0[row] * a.dt;
        const RowShift rs = row_shift(sh, len, tb.scal[1]);
        for (int m = t; m < NE; m += kLanes) {
            int e = i0 - H + m;
            const int kx = e < 0 ? -n : (e >= n ? n : 0);
            e -= kx;
            const NodePos np = node_pos_same(x[e], rs, x0, xN, tb.scal[0], tb.scal[2], tb.nb);
            const double2 nx = tb.bnext[np.b];
            int c = cell_from_bucket(tb.bucket[np.b], nx, np.xt);
            if (np.xt >= nx.y) c = cell_walk(x, n, c, np.xt);
            const int64_t g = (int64_t)c + (rs.kf0 + np.dk) * (int64_t)n + kx;
            sg[m] = g;
            if constexpr (LR == kReconPPM)
                sell[m] = (float)ppm_partial_tab<float>(tb, x, q, n, c, np.xt);
            else if constexpr (LR == kReconPLM)
                sell[m] = (float)lim_partial_global<float, LR>(x, q, n, c, np.xt);
            else
                sell[m] = (float)direct_partial<float, P>(x, q, n, len, sh, tb.scal[1], i0 - H + m, g);
        }
        wave_sync();
    }

    // ---- destination cells, one per lane: whole cells + two partials, / dx --
    // (the lanes past the last cell repeat it: same values, same places)
    float qs[NCS];
#pragma unroll
    for (int kk = 0; kk < NCS; ++kk) {
        const int ci = min(t + kk * kLanes, NC - 1);
        {
            const int c0 = i0 - H + ci;
            const int cell = inner ? c0 : wrap1f(c0, n);
            float mp;
            if (windowed) {
                const int ja = sjc[ci], jb = sjc[ci + 1];
                const float m0 = sw[ja], m1 = sw[ja + 1];
                float whole = jb > ja ? m0 : 0.0f;
                whole += jb > ja + 1 ? m1 : 0.0f;
                for (int mm = ja + 2; mm < jb; ++mm) whole += sw[mm];
                mp = whole + (sell[ci + 1] - sell[ci]);
            } else {
                mp = (float)(direct_whole<float>(R.edges, q, n, sg[ci], sg[ci + 1]) +
                             ((double)sell[ci + 1] - (double)sell[ci]));
            }
            qs[kk] = mp * tb.dxinvf[cell];
            if constexpr (H == 0) qo[cell] = qs[kk];
            else if (qmid && ci >= H && ci < H + nd) qmid[cell] = qs[kk];
        }
    }
    if constexpr (H != 0) {
        float dvv[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
        load_faces<VEC>((const float *)a.dv + qoff, n, i0, nd, c4, dvv);
        // per-cell geometry of cells i0+4l-2 .. i0+4l+5: (dx, 1/gap), and 1/dx
        // of the four own cells
        float2 rrv[NV];
        float dxi[4];
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const int cg = i0 + min(c4, nd - 1) - 2 + c;
            rrv[c] = tb.rrf[wrap1f(cg, n)];
        }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) dxi[kk] = tb.dxinvf[min(i0 + c4 + kk, n - 1)];
        wave_sync();                                 // the window is dead
#pragma unroll
        for (int kk = 0; kk < NCS; ++kk) sq[min(t + kk * kLanes, NC - 1)] = qs[kk];
        wave_sync();
        if (c4 < nd) {
            float sv[NV];
#pragma unroll
            for (int v = 0; v < NV / 4; ++v) {
                const float4 q4 = *(const float4 *)(sq + c4 + 4 * v);
                sv[4 * v] = q4.x;
                sv[4 * v + 1] = q4.y;
                sv[4 * v + 2] = q4.z;
                sv[4 * v + 3] = q4.w;
            }
            float o[4];
            residual4(sv, dvv, dt, [&](int c) { return rrv[c]; }, [&](int kk) { return dxi[kk]; },
                      o);
            store_cells<VEC>(qo, i0, nd, c4, o);
        }
    }
}

// ---------------------------------------------------------------------------
// A searching tile whose window fits the wave's LDS, with every load of a phase
// in flight at once:
//   1. the nodes' plan (window index, theta), the window's values and cell
//      sizes in 16-byte groups, the faces' residual velocity;
//   2. the window masses into LDS; the stencil data of all the lane's
//      nodes' source cells (three planes of the mesh table);
//   3. each node's Lagrange weights and partial integral (from the masses
//      beside its window cell) into LDS;
//   4. each shifted cell's mass (the whole window cells between its nodes
//      plus the difference of the two partial integrals), while the cell
//      geometry of the residual is on its way;
//   5. the masses through LDS to four consecutive cells a lane and their
//      residual neighbourhoods, the residual, 16-byte stores.
// Nodes and shifted cells go to lanes in turn (node m, cell ci on lane
// m mod 64, counted from the tile's first halo node/cell), so that the LDS
// gathers of neighbouring lanes fall on neighbouring words: four consecutive
// nodes a lane put their gathers 16 bytes apart, eight lanes on each bank.
// VEC: rows of a multiple of four cells, 16-byte aligned: the window is stored
// from the 16-byte boundary at or below its start (LDS index j + off for
// window cell j), so that its groups go in whole, also across the row's end.
// Other rows read the groups from the window's start (off = 0) at a word's
// alignment, the group that straddles the row's end cell by cell beside them, and
// the mesh's sizes past its end from their continuation there; their cumulative
// differences are always summed directly.  At 1000 x 6001 cells, all searching,
// 39 us a step (38 at 6000); 58 with the whole window cell by cell, a round of
// loads after the other, where it crosses the row's end, and 80 with one node's
// 64-byte record and one word a load (general_tile).
//
// Latency bounds it (four round trips), so registers count: at five waves a SIMD
// (96 registers at order 5) 1000 x 6000 cells take 36 us a step, at four 40; at
// six the rows not a multiple of four spill (70 against 58).
// ---------------------------------------------------------------------------

template <int P, int H, int S, bool VEC, class Nodes>
__device__ __forceinline__ void window_tile(const StepArgs &a, const FastTile &ft, const Nodes &nodes,
                                            unsigned char *su, float *sell, short *sjc, int t)
{
    using AC = Acc<S == kSumDirect ? kScanF32 : S>;
    using A = typename AC::A;
    using M = typename AC::M;
    constexpr bool kDirect = S == kSumDirect;
    static_assert(VEC || kDirect, "rows not a multiple of four sum directly");
    constexpr int LO = (P - 1) / 2;
    constexpr int NG = 2;                            // window groups of 4 a lane loads first
    constexpr int NS = (kFT + 2 * H + 1 + kLanes - 1) / kLanes;   // node slots
    constexpr int NCS = (kFT + 2 * H + kLanes - 1) / kLanes;      // shifted-cell slots
    const Rows &R = a.rows;
    const MeshTab &tb = R.tab;
    const int n = (int)R.n_cols;
    const int c4 = 4 * t;
    const TilePos tp = tile_pos(ft.pad[0], n, H);
    const int i0 = tp.i0, nd = tp.nd;
    const int NC = nd + 2 * H;
    const int64_t qoff = (int64_t)tp.row * n;
    const float *q = (const float *)a.q_in + qoff;
    float *qo = (float *)a.q_out + qoff;
    const int W = ft.w, base = ft.base;
    const int a0 = VEC ? base & ~3 : base, off = base - a0;
    const int gl = (W + off - 1) >> 2;               // last window group
    float *sw = (float *)su;                         // window mass j at sw[j + off]
    // rows not a multiple of four: the one group that straddles the row's end
    // (its cells are put in one by one afterwards)
    const int left = n - base, split = left & ~3;
    const bool cross = !VEC && split != left && split <= 4 * gl;

    // ---- 1. node plan, window, faces ------------------------------------------
    float thv[NS];
    int jv[NS];
    nodes.get(t, thv, jv);
    // window values and cell sizes (FP64 sizes for the FP64 prefix)
    constexpr bool kDx64 = S == kScanF64;
    float4 wq[NG], wd[NG];
    double2 wd2[kDx64 ? NG : 1][2];
    auto load4 = [&](const float *p, int c) {
        if constexpr (VEC) {
            return ld_at<float4>(p, 4u * (uint32_t)c);
        } else {
            const auto v = ld_at<f4u>(p, 4u * (uint32_t)c).v;
            return make_float4(v.x, v.y, v.z, v.w);
        }
    };
#pragma unroll
    for (int u = 0; u < NG; ++u) {
        int c = a0 + 4 * min(t + u * kLanes, gl);
        c = c >= n ? c - n : c;
        wq[u] = load4(q, VEC ? c : min(c, n - 4));
        if constexpr (kDx64) {
            wd2[u][0] = ld_at<double2>(tb.dx, 8u * (uint32_t)c);
            wd2[u][1] = ld_at<double2>(tb.dx, 8u * (uint32_t)c + 16u);
        } else {
            wd[u] = load4(tb.dxf, c);
        }
    }
    float over = 0.0f;
    if (cross) {
        int c = base + split + (t & 3);
        c = c >= n ? c - n : c;
        over = q[c] * tb.dxf[c];
    }
    float dvv[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
    if constexpr (H != 0) load_faces<VEC>((const float *)a.dv + qoff, n, i0, nd, c4, dvv);
    float4 di4 = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (H == 0) {
        if (VEC || nd == kFT) {
            di4 = *(const float4 *)(tb.dxinvf + i0 + (VEC ? min(c4, nd - 4) : c4));
        } else {
            float *d = &di4.x;
#pragma unroll
            for (int k = 0; k < 4; ++k) d[k] = tb.dxinvf[i0 + min(c4 + k, nd - 1)];
        }
    }
    A *sp = (A *)su;                                 // prefix modes: cumulative at j + off
    if constexpr (kDirect) {
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            const int g = min(t + u * kLanes, gl);
            *(float4 *)(sw + 4 * g) = make_float4(wq[u].x * wd[u].x, wq[u].y * wd[u].y,
                                                  wq[u].z * wd[u].z, wq[u].w * wd[u].w);
        }
        // windows longer than NG groups a lane (compressing stretches of mesh)
        for (int u = NG; u * kLanes <= gl; ++u) {
            const int g = min(t + u * kLanes, gl);
            int c = a0 + 4 * g;
            c = c >= n ? c - n : c;
            const float4 vq = load4(q, VEC ? c : min(c, n - 4));
            const float4 vd = load4(tb.dxf, c);
            *(float4 *)(sw + 4 * g) = make_float4(vq.x * vd.x, vq.y * vd.y, vq.z * vd.z, vq.w * vd.w);
        }
        if (cross && t < 4) sw[split + t] = over;
    } else {
        A carry = AC::zero();
        auto masses = [&](const float4 &vq, const float4 &vd, const double2 (&v2)[2], M (&m)[4]) {
            if constexpr (kDx64) {
                m[0] = AC::mass(vq.x, v2[0].x);
                m[1] = AC::mass(vq.y, v2[0].y);
                m[2] = AC::mass(vq.z, v2[1].x);
                m[3] = AC::mass(vq.w, v2[1].y);
            } else {
                m[0] = (M)(vq.x * vd.x);
                m[1] = (M)(vq.y * vd.y);
                m[2] = (M)(vq.z * vd.z);
                m[3] = (M)(vq.w * vd.w);
            }
        };
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            if (u * kLanes > gl) break;
            M m[4];
            masses(wq[u], wd[u], wd2[kDx64 ? u : 0], m);
            wave_prefix<S == kSumDirect ? kScanF32 : S>(sp, m, t + u * kLanes, gl, carry);
        }
        for (int u = NG; u * kLanes <= gl; ++u) {
            const int g = min(t + u * kLanes, gl);
            int c = a0 + 4 * g;
            c = c >= n ? c - n : c;
            const float4 vq = *(const float4 *)(q + c);
            float4 vd = make_float4(0.f, 0.f, 0.f, 0.f);
            double2 v2[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
            if constexpr (kDx64) {
                v2[0] = *(const double2 *)(tb.dx + c);
                v2[1] = *(const double2 *)(tb.dx + c + 2);
            } else {
                vd = *(const float4 *)(tb.dxf + c);
            }
            M m[4];
            masses(vq, vd, v2, m);
            wave_prefix<S == kSumDirect ? kScanF32 : S>(sp, m, t + u * kLanes, gl, carry);
        }
    }

    // ---- 2. stencil data of the nodes' source cells, all at once -----------------
    // (planes: neighbouring lanes read neighbouring cells' data; the offsets
    // of the cell's own edges are 0 and 1 exactly, the own node's weight is not
    // needed)
    constexpr int NV = 2 * P - 1;                    // values a cell
    float rth[NS][P + 1], rrd[NS][P + 1];
    const float *stp1 = tb.stp + 4 * n, *stp2 = tb.stp + 8 * n;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        int c = base + jv[u];
        c = c >= n ? c - n : c;
        float v[12];
        const float4 A = ld_at<float4>(tb.stp, 16u * (uint32_t)c);
        v[0] = A.x; v[1] = A.y; v[2] = A.z; v[3] = A.w;
        if constexpr (NV > 4) {
            const float4 B = ld_at<float4>(stp1, 16u * (uint32_t)c);
            v[4] = B.x; v[5] = B.y; v[6] = B.z; v[7] = B.w;
        }
        if constexpr (NV > 8) v[8] = ld_at<float>(stp2, 4u * (uint32_t)c);
        int k = 0;
#pragma unroll
        for (int b = 0; b <= P; ++b)
            rth[u][b] = b == LO ? 0.0f : (b == LO + 1 ? 1.0f : v[k++]);
#pragma unroll
        for (int b = 0; b <= P; ++b) rrd[u][b] = b == LO ? 0.0f : v[k++];
    }
    wave_sync();                                     // the window masses

    // ---- 3. weights and partial integrals C~(x) - C(c), summed outward ------------
    // (lanes past the last node repeat it: the plan's padding, same slots)
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const float th = thv[u];
        float tt[P + 1], pre[P + 1], suf[P + 1], wk[P + 1];
#pragma unroll
        for (int b = 0; b <= P; ++b) tt[b] = th - rth[u][b];
        pre[0] = 1.0f;
#pragma unroll
        for (int b = 1; b <= P; ++b) pre[b] = pre[b - 1] * tt[b - 1];
        suf[P] = 1.0f;
#pragma unroll
        for (int b = P - 1; b >= 0; --b) suf[b] = suf[b + 1] * tt[b + 1];
#pragma unroll
        for (int b = 0; b <= P; ++b) wk[b] = rrd[u][b] * (pre[b] * suf[b]);
        const int j = jv[u] + off;
        float e = 0.0f;
        if constexpr (kDirect) {
            float up = 0.0f, dn = 0.0f;
#pragma unroll
            for (int b = LO + 1; b <= P; ++b) {
                up += sw[j + b - LO - 1];
                e += wk[b] * up;
            }
#pragma unroll
            for (int b = LO - 1; b >= 0; --b) {
                dn += sw[j - LO + b];
                e -= wk[b] * dn;
            }
        } else {
            const A pc = sp[j];
#pragma unroll
            for (int b = 0; b <= P; ++b)
                if (b != LO) e += wk[b] * (float)AC::diff(sp[j - LO + b], pc);
        }
        const int m = min(t + u * kLanes, kFastNodes - 1);
        sell[m] = e;
        sjc[m] = (short)j;
    }
    wave_sync();

    // ---- 4. shifted masses (lanes past the last cell repeat it) --------------------
    float ms[NCS];
#pragma unroll
    for (int u = 0; u < NCS; ++u) {
        const int ci = min(t + u * kLanes, NC - 1);
        const int ja = sjc[ci], jb = sjc[ci + 1];
        float whole;
        if constexpr (kDirect) {
            const float m0 = sw[ja], m1 = sw[ja + 1];
            whole = jb > ja ? m0 : 0.0f;
            whole += jb > ja + 1 ? m1 : 0.0f;
            for (int mm = ja + 2; mm < jb; ++mm) whole += sw[mm];
        } else {
            whole = (float)AC::diff(sp[jb], sp[ja]);
        }
        ms[u] = whole + (sell[ci + 1] - sell[ci]);
    }
    // geometry of cells i0+4l-2 .. i0+4l+5 (lanes past the tile: its last
    // cells): (dx, 1/centre gap) as four 16-byte pairs, 1/dx as 8 + 16 + 8
    // bytes (the row holds a multiple of four cells: no group straddles its end)
    float2 rr[8];
    float dxi[8];
    if constexpr (H != 0) {
        const int cb = i0 + min(c4, (nd - 1) & ~3) - 2;
        auto wr = [&](int c) { return VEC ? (c < 0 ? c + n : (c >= n ? c - n : c)) : c; };
#pragma unroll
        for (int pr = VEC ? 0 : 1; pr < 4; ++pr) {
            const float4 r2 = ld_at<float4>(tb.rrf, 8u * (uint32_t)wr(cb + 2 * pr));
            rr[2 * pr] = make_float2(r2.x, r2.y);
            rr[2 * pr + 1] = make_float2(r2.z, r2.w);
        }
        float2 d0;
        if constexpr (VEC) {
            d0 = ld_at<float2>(tb.dxinvf, 4u * (uint32_t)wr(cb));
        } else {
            // (the first pair may lie before the row's start, at any word there)
            const int c0 = cb < 0 ? cb + n : cb;
            const auto r0 = ld_at<f4u>(tb.rrf, 8u * (uint32_t)c0).v;
            const auto i0 = ld_at<f2u>(tb.dxinvf, 4u * (uint32_t)c0).v;
            rr[0] = make_float2(r0.x, r0.y);
            rr[1] = make_float2(r0.z, r0.w);
            d0 = make_float2(i0.x, i0.y);
        }
        const float4 d1 = ld_at<float4>(tb.dxinvf, 4u * (uint32_t)wr(cb + 2));
        const float2 d2 = ld_at<float2>(tb.dxinvf, 4u * (uint32_t)wr(cb + 6));
        dxi[0] = d0.x; dxi[1] = d0.y;
        dxi[2] = d1.x; dxi[3] = d1.y; dxi[4] = d1.z; dxi[5] = d1.w;
        dxi[6] = d2.x; dxi[7] = d2.y;
    }
    wave_sync();                                     // the window is dead
    float *sm = (float *)su;                         // shifted masses, index ci
#pragma unroll
    for (int u = 0; u < NCS; ++u) sm[min(t + u * kLanes, NC - 1)] = ms[u];
    wave_sync();

    // ---- 5. residual (or, without one, the shifted values) ------------------------
    if (c4 < nd) {
        if constexpr (H == 0) {
            const float4 m4 = *(const float4 *)(sm + c4);
            float o[4] = {m4.x * di4.x, m4.y * di4.y, m4.z * di4.z, m4.w * di4.w};
            store_cells<VEC>(qo, i0, nd, c4, o);
        } else {
            const float4 m0 = *(const float4 *)(sm + c4), m1 = *(const float4 *)(sm + c4 + 4);
            const float mv[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
            float sv[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) sv[c] = mv[c] * dxi[c];
            if (a.q_mid) store_cells<VEC>((float *)a.q_mid + qoff, i0, nd, c4, sv + 2);
            float o[4];
            residual4(sv, dvv, (float)a.dt, [&](int c) { return rr[c]; },
                      [&](int kk) { return dxi[kk + 2]; }, o);
            store_cells<VEC>(qo, i0, nd, c4, o);
        }
    }
}

// The step, in two kernels, one tile a wave: the uniform tiles (26 registers,
// eight waves a SIMD), then the other tiles, each from its list.  Measured
// alternatives on the refined disk: one kernel over both kinds (in tile order,
// or the other tiles spread evenly through the grid) ran the uniform tiles at
// the other path's register and LDS footprint and took 135-163 us a step
// against 123; persistent waves striding over the other tiles, 128-157; the
// two kernels on two streams with an event pair around every eager step, 342.
// Inside a captured step loop the two kernels are parallel branches of the
// graph (fork / join events, ForkJoin): the latency-bound searching tiles then
// run beside the HBM-bound uniform ones.  Fewer than kTogether tiles take one
// launch for both kinds (k_step_both).
template <int P, int H, bool VEC>
__global__ __launch_bounds__(kBlock, 8) void k_step_uni(StepArgs a)
{
    __shared__ __attribute__((aligned(16))) float swin[kWaves][kUniWin];
    const int wid = wave_id();
    const int i = (int)blockIdx.x * kWaves + wid;
    if (i >= a.fast.totals[0]) return;
    uniform_tile<P, H, VEC>(a, load_rec(a.fast.urec, i), swin[wid], (int)threadIdx.x % kLanes);
}

// A uniform-run tile of the limited step (Section 3.1's PLM / PPM, App. A),
// FP32: every node of the tile sits in the next window cell at the tile's
// theta, so shifted cell ci is the average of window cell LO + ci plus the
// difference of the limited cubics of window cells LO + ci + 1 and LO + ci
// at theta (in value units: the run's cells are all of one size).  Each lane
// forms, from its window values in registers, the slopes, the PPM interface
// values and the constrained parabolas its eight shifted cells need (the
// mesh's weights of window cell 1, whose neighbours lie in the run, serve the
// whole tile), then the residual as in uniform_tile.
template <int R, int H, bool VEC>
__device__ __forceinline__ void uniform_tile_lim(const StepArgs &a, const FastTile &r, float *sw,
                                                 int t)
{
    constexpr int LO = LimHalo<R>::lo;
    constexpr int P = 2 * LO + 1;
    constexpr int NV = 4 + 2 * H;                    // shifted cells a lane
    constexpr int NQ = NV + 2 * LO + 1;             // window values c4 .. c4 + NQ - 1
    constexpr int NW = (NQ + 3) / 4 * 4;             // whole float4s
    constexpr int NUW = (kFT + 2 * H + P + kLanes - 1) / kLanes;  // window slots a lane
    static_assert(NUW * kLanes <= kUniWin && 4 * (kLanes - 1) + NW <= kUniWin, "window");
    const MeshTab &tb = a.rows.tab;
    const int n = (int)a.rows.n_cols;
    const float dt = (float)a.dt;
    const int c4 = 4 * t;
    const TilePos p = tile_pos(r.pad[0], n, H);
    const int64_t qoff = (int64_t)p.row * n;
    const float th = __int_as_float(r.pad[1]);

    float wv[NUW];
    {
        const float *q = (const float *)a.q_in + qoff;
#pragma unroll
        for (int k = 0; k < NUW; ++k) {
            int mm = r.base + min(t + k * kLanes, r.w - 1);
            mm = mm >= n ? mm - n : mm;
            wv[k] = q[mm];
        }
    }
    float pw[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
    {
        const int c1 = r.base + 1 >= n ? r.base + 1 - n : r.base + 1;
        if constexpr (R == kReconPPM) {
#pragma unroll
            for (int k = 0; k < 5; ++k) pw[k] = tb.ppmf[k * n + c1];
        }
    }
    float dvv[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
    if constexpr (H != 0) load_faces<VEC>((const float *)a.dv + qoff, n, p.i0, p.nd, c4, dvv);
#pragma unroll
    for (int k = 0; k < NUW; ++k) sw[t + k * kLanes] = wv[k];
    wave_sync();
    float win[NW];
#pragma unroll
    for (int v = 0; v < NW / 4; ++v) {
        const float4 w4 = *(const float4 *)(sw + c4 + 4 * v);
        win[4 * v] = w4.x;
        win[4 * v + 1] = w4.y;
        win[4 * v + 2] = w4.z;
        win[4 * v + 3] = w4.w;
    }
    // ell[v]: the limited cubic at theta of window cell c4 + LO + v (value units)
    float ell[NV + 1];
    if constexpr (R == kReconPPM) {
        // slope of window cell c4 + 1 + s, then the interface between window
        // cells c4 + 1 + s and c4 + 2 + s
        float dl[NV + 3], iv[NV + 2];
#pragma unroll
        for (int k = 0; k < NV + 3; ++k) dl[k] = ppm_delta<float>(win[k], win[k + 1], win[k + 2], pw[0], pw[1]);
#pragma unroll
        for (int k = 0; k < NV + 2; ++k)
            iv[k] = win[k + 1] + pw[2] * (win[k + 2] - win[k + 1]) + pw[3] * dl[k + 1] + pw[4] * dl[k];
#pragma unroll
        for (int v = 0; v <= NV; ++v) {
            float pa, pb, pc;
            ppm_cubic<float>(win[v + 2], iv[v], iv[v + 1], 1.0f, pa, pb, pc);
            pb = win[v + 2] - pa - pc;
            ell[v] = th * (pa + th * (pb + th * pc));
        }
    } else {
        const float g = r.hinv, hh = r.dx;
#pragma unroll
        for (int v = 0; v <= NV; ++v) {
            const float dp = (win[v + 2] - win[v + 1]) * g, dm = (win[v + 1] - win[v]) * g;
            const float sig = (dp * dm <= 0.0f) ? 0.0f : harmonic2(dp, dm);
            const float kap = 0.5f * sig * hh;
            ell[v] = th * (win[v + 1] - kap + th * kap);
        }
    }
    float s[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) s[v] = win[v + LO] + (ell[v + 1] - ell[v]);
    float *qo = (float *)a.q_out + qoff;
    if constexpr (H == 0) {
        store_cells<VEC>(qo, p.i0, p.nd, c4, s);
    } else {
        if (a.q_mid) store_cells<VEC>((float *)a.q_mid + qoff, p.i0, p.nd, c4, s + 2);
        const float2 g = make_float2(r.dx, r.hinv);
        const float dxi = r.dxinv;
        float o[4];
        residual4(s, dvv, dt, [&](int) { return g; }, [&](int) { return dxi; }, o);
        store_cells<VEC>(qo, p.i0, p.nd, c4, o);
    }
}

template <int R, int H, bool VEC>
__global__ __launch_bounds__(kBlock) void k_step_uni_lim(StepArgs a)
{
    __shared__ __attribute__((aligned(16))) float swin[kWaves][kUniWin];
    const int wid = wave_id();
    const int i = (int)blockIdx.x * kWaves + wid;
    if (i >= a.fast.totals[0]) return;
    const FastTile r = load_rec(a.fast.urec, i);
    uniform_tile_lim<R, H, VEC>(a, r, swin[wid], (int)threadIdx.x % kLanes);
}

// The other tiles.

// LDS of the workgroups that run them.
template <int S> struct GenLds {
    __attribute__((aligned(16))) unsigned char su[kWaves][wave_lds_bytes<S>()];
    __attribute__((aligned(16))) float sell[kWaves][WaveLds::nodes];
    __attribute__((aligned(16))) short sjc[kWaves][WaveLds::nodes];
};
template <int P, int H, bool VEC, int S, bool PLAN>
__device__ __forceinline__ void other_tile(const StepArgs &a, const FastTile &r, GenLds<S> &lds, int t)
{
    const int wid = wave_id();
    const int n = (int)a.rows.n_cols;
    auto run = [&](const auto &nodes, bool located) {
        if (located && r.base + r.w + 3 < 2 * n && (VEC || n >= 8))
            window_tile<P, H, S, VEC>(a, r, nodes, lds.su[wid], lds.sell[wid], lds.sjc[wid], t);
        else
            general_tile<P, H, VEC, 0>(a, r, located, nodes, lds.su[wid], lds.sell[wid], lds.sjc[wid], t);
    };
    if constexpr (PLAN) {
        run(PlannedNodes<H>(a, r), r.kind == kFastWindow);
    } else {
        LocatedNodes<H> nodes;
        const bool located = r.kind == kFastWindow && nodes.template locate<P>(a, r, t);
        run(nodes, located);
    }
}
// Wave `wave` of `waves`.
template <int P, int H, bool VEC, int S>
__device__ __forceinline__ void other_tiles(const StepArgs &a, GenLds<S> &lds, int wave, int waves)
{
    const int total = a.fast.totals[1];
    for (int i = wave; i < total; i += waves) {
        other_tile<P, H, VEC, S, true>(a, load_rec(a.fast.rec, load_index(a.fast.oid, i)), lds,
                                       (int)threadIdx.x % kLanes);
        wave_sync();                                 // the next tile reuses the LDS
    }
}

template <int P, int H, bool VEC, int S>
__global__ __launch_bounds__(kBlock, 5) void k_step_gen(StepArgs a)
{
    __shared__ GenLds<S> lds;
    other_tiles<P, H, VEC, S>(a, lds, (int)blockIdx.x * kWaves + wave_id(), (int)gridDim.x * kWaves);
}

// Both kinds in one launch: the first `others` workgroups the other tiles, the
// rest the uniform ones.
template <int P, int H, bool VEC, int S>
__global__ __launch_bounds__(kBlock, 5) void k_step_both(StepArgs a, int others)
{
    __shared__ GenLds<S> lds;
    const int wid = wave_id();
    if ((int)blockIdx.x < others) {
        other_tiles<P, H, VEC, S>(a, lds, (int)blockIdx.x * kWaves + wid, others * kWaves);
        return;
    }
    const int i = ((int)blockIdx.x - others) * kWaves + wid;
    if (i >= a.fast.totals[0]) return;
    static_assert(sizeof(lds.su[0]) >= sizeof(float) * kUniWin, "a uniform tile's window");
    uniform_tile<P, H, VEC>(a, load_rec(a.fast.urec, i), (float *)lds.su[wid],
                            (int)threadIdx.x % kLanes);
}

// One step of a call that has no plan: a wave takes a tile in tile order, makes
// its record and locates its nodes, by the arithmetic of the plan's kernels.  The
// call is then the mesh tables (with the copy of the state beside them) and this:
// 512 x 2048 cells on the refined disk 17 us (6.5 and 10.8), 26 with the plan's
// two launches, the lists' one and the copy of the result back.  Latency bounds
// it there, VALU issue on large searching batches.
template <int P, int H, bool VEC, int S>
__global__ __launch_bounds__(kBlock, 5) void k_step_one(StepArgs a)
{
    __shared__ GenLds<S> lds;
    const int i = spread8((int)blockIdx.x) * kWaves + wave_id();
    if (i >= (int)a.rows.n_tiles) return;
    const int t = (int)threadIdx.x % kLanes;
    const FastTile r = plan_wave<P>(a, i, H, t);
    if (r.kind == kFastUniform) uniform_tile<P, H, VEC>(a, r, (float *)lds.su[wave_id()], t);
    else other_tile<P, H, VEC, S, false>(a, r, lds, t);
}

template <int P, int H, bool VEC, int S>
hipError_t step_fast_kernels(const StepArgs &a, hipStream_t st)
{
    const int64_t nt = a.rows.n_tiles;
    const dim3 g(uniform_grid(nt)), b(kBlock), gg(other_grid(nt));
    if (a.fast.alone) {
        hipLaunchKernelGGL((k_step_one<P, H, VEC, S>), dim3((g.x + 7) / 8 * 8), b, 0, st, a);
        return hipGetLastError();
    }
    if (nt < kTogether) {
        const unsigned others = uniform_grid(nt);    // a wave a tile: it may be any of them
        hipLaunchKernelGGL((k_step_both<P, H, VEC, S>), dim3(others + g.x), b, 0, st, a, (int)others);
        return hipGetLastError();
    }
    if (const ForkJoin *fj = capture_fork) {
        // the two kinds of tile write disjoint cells and read only q_in: the
        // searching tiles' kernel on the side stream, between a fork after
        // everything before the step and a join before everything after it
        hipError_t e = hipEventRecord(fj->fork, st);
        if (e == hipSuccess) e = hipStreamWaitEvent(fj->side, fj->fork, 0);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_step_gen<P, H, VEC, S>), gg, b, 0, fj->side, a);
        e = hipEventRecord(fj->join, fj->side);
        hipLaunchKernelGGL((k_step_uni<P, H, VEC>), g, b, 0, st, a);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, fj->join, 0);
        if (e != hipSuccess) return e;
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_step_uni<P, H, VEC>), g, b, 0, st, a);
    hipLaunchKernelGGL((k_step_gen<P, H, VEC, S>), gg, b, 0, st, a);
    return hipGetLastError();
}

template <int P, int S>
hipError_t step_fast_ps(const StepArgs &a, bool vec, hipStream_t st)
{
    if constexpr (S == kSumDirect) {
        if (!vec)
            return a.dv ? step_fast_kernels<P, 2, false, S>(a, st)
                        : step_fast_kernels<P, 0, false, S>(a, st);
    }
    return a.dv ? step_fast_kernels<P, 2, true, S>(a, st) : step_fast_kernels<P, 0, true, S>(a, st);
}

template <int P>
hipError_t step_fast_p(const StepArgs &a, int scan, hipStream_t st)
{
    const bool vec = (a.rows.n_cols % 4) == 0 && ((uintptr_t)a.q_out % 16) == 0 &&
                     ((uintptr_t)a.q_in % 16) == 0 &&
                     (!a.q_mid || ((uintptr_t)a.q_mid % 16) == 0) &&
                     (!a.dv || ((uintptr_t)a.dv % 16) == 0);
    // rows not a multiple of four cells sum directly in every mode
    switch (vec ? scan : (int)kSumDirect) {
    case kScanF64: return step_fast_ps<P, kScanF64>(a, vec, st);
    case kScanTwoSum: return step_fast_ps<P, kScanTwoSum>(a, vec, st);
    case kScanF32: return step_fast_ps<P, kScanF32>(a, vec, st);
    default: return step_fast_ps<P, kSumDirect>(a, vec, st);
    }
}

// The limited step's other tiles: general_tile with the limited partials, the
// window tabulated in LDS where it fits, else every node located by the bucket
// index and its partial integral the limited profile of its cell.
struct GenLimLds {
    static constexpr size_t U = kGenLimLds > WaveLds::u ? kGenLimLds : WaveLds::u;
    __attribute__((aligned(16))) unsigned char su[kWaves][U];
    __attribute__((aligned(16))) float sell[kWaves][WaveLds::nodes];
    __attribute__((aligned(16))) short sjc[kWaves][WaveLds::nodes];
};
template <int R, int H, bool VEC>
__device__ __forceinline__ void other_tiles_lim(const StepArgs &a, GenLimLds &lds, int wave, int waves)
{
    constexpr int P = 2 * LimHalo<R>::lo + 1;
    const int wid = wave_id();
    const int t = (int)threadIdx.x % kLanes;
    const int total = a.fast.totals[1];
    for (int i = wave; i < total; i += waves) {
        const FastTile r = load_rec(a.fast.rec, load_index(a.fast.oid, i));
        general_tile<P, H, VEC, R>(a, r, r.kind == kFastWindow, PlannedNodes<H>(a, r), lds.su[wid],
                                   lds.sell[wid], lds.sjc[wid], t);
        wave_sync();                                 // the next tile reuses the LDS
    }
}

template <int R, int H, bool VEC>
__global__ __launch_bounds__(kBlock) void k_step_gen_lim(StepArgs a)
{
    __shared__ GenLimLds lds;
    other_tiles_lim<R, H, VEC>(a, lds, (int)blockIdx.x * kWaves + wave_id(), (int)gridDim.x * kWaves);
}

// Both kinds in one launch, as k_step_both.
template <int R, int H, bool VEC>
__global__ __launch_bounds__(kBlock) void k_step_both_lim(StepArgs a, int others)
{
    __shared__ GenLimLds lds;
    const int wid = wave_id();
    if ((int)blockIdx.x < others) {
        other_tiles_lim<R, H, VEC>(a, lds, (int)blockIdx.x * kWaves + wid, others * kWaves);
        return;
    }
    const int i = ((int)blockIdx.x - others) * kWaves + wid;
    if (i >= a.fast.totals[0]) return;
    static_assert(sizeof(lds.su[0]) >= sizeof(float) * kUniWin, "a uniform tile's window");
    uniform_tile_lim<R, H, VEC>(a, load_rec(a.fast.urec, i), (float *)lds.su[wid],
                                (int)threadIdx.x % kLanes);
}

template <int R, int H, bool VEC>
hipError_t step_fast_lim_kernels(const StepArgs &a, hipStream_t st)
{
    const int64_t nt = a.rows.n_tiles;
    const dim3 g(uniform_grid(nt)), b(kBlock), gg(other_grid(nt));
    if (nt < kTogether) {
        const unsigned others = uniform_grid(nt);
        hipLaunchKernelGGL((k_step_both_lim<R, H, VEC>), dim3(others + g.x), b, 0, st, a, (int)others);
        return hipGetLastError();
    }
    if (const ForkJoin *fj = capture_fork) {
        // parallel graph branches, as in step_fast_kernels
        hipError_t e = hipEventRecord(fj->fork, st);
        if (e == hipSuccess) e = hipStreamWaitEvent(fj->side, fj->fork, 0);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_step_gen_lim<R, H, VEC>), gg, b, 0, fj->side, a);
        e = hipEventRecord(fj->join, fj->side);
        hipLaunchKernelGGL((k_step_uni_lim<R, H, VEC>), g, b, 0, st, a);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, fj->join, 0);
        if (e != hipSuccess) return e;
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_step_uni_lim<R, H, VEC>), g, b, 0, st, a);
    hipLaunchKernelGGL((k_step_gen_lim<R, H, VEC>), gg, b, 0, st, a);
    return hipGetLastError();
}

template <int R>
hipError_t step_fast_lim_r(const StepArgs &a, hipStream_t st)
{
    const bool vec = (a.rows.n_cols % 4) == 0 && ((uintptr_t)a.q_out % 16) == 0 &&
                     ((uintptr_t)a.q_in % 16) == 0 &&
                     (!a.q_mid || ((uintptr_t)a.q_mid % 16) == 0) &&
                     (!a.dv || ((uintptr_t)a.dv % 16) == 0);
    if (a.dv) return vec ? step_fast_lim_kernels<R, 2, true>(a, st) : step_fast_lim_kernels<R, 2, false>(a, st);
    return vec ? step_fast_lim_kernels<R, 0, true>(a, st) : step_fast_lim_kernels<R, 0, false>(a, st);
}

// ---------------------------------------------------------------------------
// Per-row meshes (every row its own nodes, ragged or not), FP32 state, the
// shift alone.  The tiles are the ragged tile table's, kRagTile cells of one
// row, one a wave.  Per call, k_plan_rag locates every shifted node of a tile
// (a binary search of the row, Eq. condition_p), takes its Lagrange weights
// from the row's nodes (Section 3, Step 2: the cumulative's interpolant
// through the p+1 nodes around the source cell) and its source cell's index
// in the tile's window, and writes the row cells' FP32 sizes.  Per step,
// k_step_rag then needs no search and no division by the mesh: the window's
// masses into LDS (or, for the prefix modes, their cumulative), each node's
// partial integral from its planned weights, each cell's whole source cells
// and the two partials, over the cell size (Eqs. mass_shift_algo, step3).
// ---------------------------------------------------------------------------

__device__ inline RagTile load_rag(const RagTile *rec, int64_t i)
{
    RagTile r;
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const __attribute__((address_space(4))) int32_t *CI;
    const CI c = (CI)(rec + i);
    int32_t *o = (int32_t *)&r;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(RagTile) / 4); ++k) o[k] = c[k];
#else
    r = rec[i];
#endif
    return r;
}

// The plan, one wave a tile: the window's nodes once into LDS, every node
// located and weighted there (rows_locate, rows_weights).  VALU issue bounds it
// (815 instructions a tile at order 3).  16.9 M cells, order 3: 172 us; 418
// with a binary search of the row and the stencil's nodes from global
// memory a node.
template <int P>
__global__ __launch_bounds__(kBlock) void k_plan_rag(StepArgs a, RagPlan pl)
{
    constexpr int NS = (kRagTile + 1) / kLanes;
    static_assert(NS * kLanes == kRagTile + 1, "whole node slots");
    __shared__ double xs_[kWaves][kFastWin + 8];
    const Rows &R = a.rows;
    const int t = (int)threadIdx.x % kLanes;
    const int wid = wave_id();
    const int64_t tile = (int64_t)blockIdx.x * kWaves + wid;
    if (tile >= R.n_tiles) return;
    RagTile rt;
    rt.kind = -1;
    rt.row = rt.i0 = rt.nd = rt.n = rt.w = rt.base = rt.pad0 = 0;
    rt.qoff = rt.eoff = rt.wlo = 0;
    rt.pad[0] = rt.pad[1] = 0;
    Tile ti;
    if (!get_tile(R, tile, ti)) {                    // past the batch's last tile
        if (t == 0) pl.rec[tile] = rt;
        return;
    }
    const int n = ti.n, i0 = ti.i0;
    const int nd = min(R.tile, n - i0);
    const int NE = nd + 1;
    const double *x = ti.x;
    const double x0 = x[0], xN = x[n];
    const double len = xN - x0;
    const double invlen = 1.0 / len;
    const double s = rows_shift(a.v0[ti.row], a.dt);
    double xe[NS], xr[NS];
    int kx[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int m = min(t + u * kLanes, NE - 1);
        kx[u] = i0 + m >= n ? 1 : 0;
        const int e = i0 + m - (kx[u] ? n : 0);
        xe[u] = x[e];
        xr[u] = x[e + 1];
    }
#pragma unroll
    for (int u = 0; u < NS; ++u)
        if (t + u * kLanes < nd) pl.dx[ti.qoff + i0 + t + u * kLanes] = (float)(xr[u] - xe[u]);
    double *xs = xs_[wid];
    RowsWindow win;
    double xh[NS];
    int j[NS];
    const bool all = n >= P + 1 && rows_locate<P, NS>(x, n, s, x0, xN, len, invlen, NE, t, kFastWin, xe,
                                                      kx, xs, win, xh, j, [] {});
    const int64_t slot = tile * kFastNodes;
    if (all) {
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            constexpr int LO = (P - 1) / 2;
            const int m = t + u * kLanes;
            float w[P + 1], v[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
            if (win.seam > win.w) rows_weights<float, P, false>(xs, win, len, xh[u], j[u], w);
            else rows_weights<float, P, true>(xs, win, len, xh[u], j[u], w);
            int k = 0;
#pragma unroll
            for (int b = 0; b <= P; ++b)
                if (b != LO) v[k++] = w[b];
            if constexpr (P == 5) {
                ((float4 *)pl.wa)[slot + m] = make_float4(v[0], v[1], v[2], v[3]);
                pl.wb[slot + m] = v[4];
            } else if constexpr (P == 3) {
                ((float2 *)pl.wa)[slot + m] = make_float2(v[0], v[1]);
                pl.wb[slot + m] = v[2];
            } else {
                pl.wa[slot + m] = v[0];
            }
            pl.jc[slot + m] = (int16_t)j[u];
        }
    }
    if (t == 0) {
        rt.kind = all ? kFastWindow : kFastDirect;
        rt.row = (int32_t)ti.row;
        rt.i0 = i0;
        rt.nd = nd;
        rt.n = n;
        rt.w = all ? win.w : 0;
        rt.base = n >= P + 1 ? win.base : 0;
        rt.qoff = ti.qoff;
        rt.eoff = (int64_t)(x - R.edges);
        rt.wlo = n >= P + 1 ? win.wlo : 0;
        pl.rec[tile] = rt;
    }
}

// The prefix modes on per-row tiles: one window cell a lane per slot (cell j
// = l + 64 u), the slot's masses scanned across the wave, the slots before
// carried on; sp[j] = cumulative before cell j, sp[W] the total.
template <int S>
__device__ __forceinline__ void wave_prefix1(typename Acc<S>::A *sp, typename Acc<S>::M m, int j,
                                             int W, typename Acc<S>::A &carry)
{
    using AC = Acc<S>;
    using A = typename AC::A;
    const int lane = (int)threadIdx.x % kLanes;
    const bool live = j < W;
    const A inc = wave_inclusive<AC>(live ? AC::add(AC::zero(), m) : AC::zero());
    A ex = AC::template dpp<kDppWaveShr1, 0xf, 0xf>(inc);
    if (lane == 0) ex = AC::zero();
    if (live) {
        sp[j] = AC::comb(carry, ex);
        if (j == W - 1) sp[W] = AC::comb(carry, inc);
    }
    carry = AC::comb(carry, lane63(inc));
}

template <int P, int S>
__device__ __forceinline__ void rag_tile(const StepArgs &a, const RagTile &r, int64_t tile,
                                         unsigned char *su, float *sell, short *sjc, int t)
{
    using AC = Acc<S == kSumDirect ? kScanF32 : S>;
    using A = typename AC::A;
    using M = typename AC::M;
    constexpr bool kDirect = S == kSumDirect;
    constexpr int LO = (P - 1) / 2;
    constexpr int NS = (kRagTile + 1 + kLanes - 1) / kLanes;     // node slots
    constexpr int NCS = (kRagTile + kLanes - 1) / kLanes;        // cell slots
    constexpr int NB = 5;                                         // window slots a batch
    const int n = r.n, i0 = r.i0, nd = r.nd, W = r.w, base = r.base;
    const float *q = (const float *)a.q_in + r.qoff;
    float *qo = (float *)a.q_out + r.qoff;
    const float *dxr = a.rag.dx + r.qoff;
    const int64_t slot = tile * kFastNodes;
    float *sw = (float *)su;                         // direct sums: window masses
    A *sp = (A *)su;                                 // prefix modes: the cumulative

    // ---- plan of the nodes, sizes of the destination cells -------------------
    float wv[NS][5];
    int jv[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int64_t m = slot + t + u * kLanes;
        if constexpr (P == 5) {
            const float4 w4 = ((const float4 *)a.rag.wa)[m];
            wv[u][0] = w4.x;
            wv[u][1] = w4.y;
            wv[u][2] = w4.z;
            wv[u][3] = w4.w;
            wv[u][4] = a.rag.wb[m];
        } else if constexpr (P == 3) {
            const float2 w2 = ((const float2 *)a.rag.wa)[m];
            wv[u][0] = w2.x;
            wv[u][1] = w2.y;
            wv[u][2] = a.rag.wb[m];
        } else {
            wv[u][0] = a.rag.wa[m];
        }
        jv[u] = a.rag.jc[m];
    }
    float dxd[NCS];
#pragma unroll
    for (int u = 0; u < NCS; ++u) dxd[u] = dxr[i0 + min(t + u * kLanes, nd - 1)];

    // ---- window masses, five slots of loads at a time (a whole window of
    // up to 320 cells in one batch); the FP64 prefix widens the FP32 masses
    const bool once = base + W <= 2 * n;             // the window wraps the row at most once
    A carry = AC::zero();
    // the prefix modes: a window of one batch goes through LDS to NB consecutive
    // masses a lane, whose sums one scan of the wave accumulates (two-sum on the
    // 16.9 M cell batch at order 3: 90 us a step, 104 with a scan a slot)
    const bool batch = !kDirect && W <= NB * kLanes;
    for (int s0 = 0; s0 * kLanes < W; s0 += NB) {
        float vq[NB], vd[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int j = min(t + (s0 + u) * kLanes, W - 1);
            int c = base + j;
            c = once ? (c >= n ? c - n : c) : c % n;
            vq[u] = q[c];
            vd[u] = dxr[c];
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            if ((s0 + u) * kLanes >= W) break;
            const int j = t + (s0 + u) * kLanes;
            if (kDirect || batch) {
                if (j < W) sw[j] = vq[u] * vd[u];
            } else if constexpr (!kDirect) {
                const M m = (M)(vq[u] * vd[u]);
                wave_prefix1<S == kSumDirect ? kScanF32 : S>(sp, m, j, W, carry);
            }
        }
    }
    wave_sync();
    if constexpr (!kDirect) {
        if (batch) {
            M m[NB];
            A tot = AC::zero();
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                m[k] = NB * t + k < W ? (M)sw[NB * t + k] : (M)0;
                tot = AC::add(tot, m[k]);
            }
            wave_sync();                             // the cumulative takes the masses' place
            const A inc = wave_inclusive<AC>(tot);
            A e = AC::template dpp<kDppWaveShr1, 0xf, 0xf>(inc);
            if (t == 0) e = AC::zero();
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                if (NB * t + k <= W) sp[NB * t + k] = e;
                e = AC::add(e, m[k]);
            }
            if (t == kLanes - 1 && W == NB * kLanes) sp[W] = e;
            wave_sync();
        }
    }

    // ---- partial integrals C~(x) - C(c) of the nodes ---------------------------
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        float wk[P + 1];
        int k = 0;
#pragma unroll
        for (int b = 0; b <= P; ++b) wk[b] = b == LO ? 0.0f : wv[u][k++];
        const int j = jv[u];
        float e = 0.0f;
        if constexpr (kDirect) {
            float up = 0.0f, dn = 0.0f;
#pragma unroll
            for (int b = LO + 1; b <= P; ++b) {
                up += sw[j + b - LO - 1];
                e += wk[b] * up;
            }
#pragma unroll
            for (int b = LO - 1; b >= 0; --b) {
                dn += sw[j - LO + b];
                e -= wk[b] * dn;
            }
        } else {
            const A pc = sp[j];
#pragma unroll
            for (int b = 0; b <= P; ++b)
                if (b != LO) e += wk[b] * (float)AC::diff(sp[j - LO + b], pc);
        }
        const int m = min(t + u * kLanes, kFastNodes - 1);
        sell[m] = e;
        sjc[m] = (short)j;
    }
    wave_sync();

    // ---- destination cells: whole source cells + two partials, / dx ----------
#pragma unroll
    for (int u = 0; u < NCS; ++u) {
        const int ci = t + u * kLanes;
        if (ci < nd) {
            const int ja = sjc[ci], jb = sjc[ci + 1];
            float whole;
            if constexpr (kDirect) {
                const float m0 = sw[ja], m1 = sw[ja + 1];
                whole = jb > ja ? m0 : 0.0f;
                whole += jb > ja + 1 ? m1 : 0.0f;
                for (int mm = ja + 2; mm < jb; ++mm) whole += sw[mm];
            } else {
                whole = (float)AC::diff(sp[jb], sp[ja]);
            }
            qo[i0 + ci] = (whole + (sell[ci + 1] - sell[ci])) / dxd[u];
        }
    }
}

// A per-row tile whose window exceeds the LDS: nodes located again and the
// masses summed from global memory, FP64.
template <int P>
__device__ __forceinline__ void rag_direct(const StepArgs &a, const RagTile &r,
                                           unsigned char *su, float *sell, int t)
{
    const int n = r.n, i0 = r.i0, nd = r.nd;
    const float *q = (const float *)a.q_in + r.qoff;
    float *qo = (float *)a.q_out + r.qoff;
    const double *x = a.rows.edges + r.eoff;
    const double len = x[n] - x[0];
    const double invlen = 1.0 / len;
    const double s = a.v0[r.row] * a.dt;
    int64_t *sg = (int64_t *)su;
    for (int m = t; m <= nd; m += kLanes) {
        int e = i0 + m, kx = 0;
        if (e >= n) {
            e -= n;
            kx = 1;
        }
        double xh;
        int64_t k;
        shifted_node_inv(x, n, s, e, invlen, len, xh, k);
        const int64_t g = (int64_t)find_cell(x, n, xh) + (k + kx) * (int64_t)n;
        sg[m] = g;
        sell[m] = (float)direct_partial<float, P>(x, q, n, len, s, invlen, i0 + m, g);
    }
    wave_sync();
    for (int ci = t; ci < nd; ci += kLanes) {
        const int c = i0 + ci;
        const double mp = direct_whole<float>(x, q, n, sg[ci], sg[ci + 1]) +
                          ((double)sell[ci + 1] - (double)sell[ci]);
        qo[c] = (float)(mp / (x[c + 1] - x[c]));
    }
}

template <int P, int S>
__global__ __launch_bounds__(kBlock) void k_step_rag(StepArgs a)
{
    __shared__ __attribute__((aligned(16))) unsigned char su[kWaves][wave_lds_bytes<S>()];
    __shared__ __attribute__((aligned(16))) float sell_[kWaves][WaveLds::nodes];
    __shared__ __attribute__((aligned(16))) short sjc_[kWaves][WaveLds::nodes];
    const int wid = wave_id();
    const int64_t tile = (int64_t)blockIdx.x * kWaves + wid;
    if (tile >= a.rows.n_tiles) return;
    const RagTile r = load_rag(a.rag.rec, tile);
    const int t = (int)threadIdx.x % kLanes;
    if (r.kind == kFastWindow) rag_tile<P, S>(a, r, tile, su[wid], sell_[wid], sjc_[wid], t);
    else if (r.kind == kFastDirect) rag_direct<P>(a, r, su[wid], sell_[wid], t);
}

template <int P>
hipError_t step_rag_p(const StepArgs &a, int scan, hipStream_t st)
{
    const dim3 g((unsigned)((a.rows.n_tiles + kWaves - 1) / kWaves)), b(kBlock);
    switch (scan) {
    case kScanF64: hipLaunchKernelGGL((k_step_rag<P, kScanF64>), g, b, 0, st, a); break;
    case kScanTwoSum: hipLaunchKernelGGL((k_step_rag<P, kScanTwoSum>), g, b, 0, st, a); break;
    case kScanF32: hipLaunchKernelGGL((k_step_rag<P, kScanF32>), g, b, 0, st, a); break;
    default: hipLaunchKernelGGL((k_step_rag<P, kSumDirect>), g, b, 0, st, a); break;
    }
    return hipGetLastError();
}

} // namespace

hipError_t launch_plan_fast(const StepArgs &a, int order, const FastPlan &plan, bool nodes,
                            hipStream_t stream)
{
    if (a.rows.n_tiles <= 0) return hipSuccess;
    if (a.rows.tile != kFastTile || a.rows.n_tiles > INT32_MAX / 2) return hipErrorInvalidValue;
    StepArgs b = a;
    b.fast = plan;
    const int64_t nt = a.rows.n_tiles;
    const int lists = (int)((nt + kBlock - 1) / kBlock);
    const int64_t groups = ((nt + kNodeTiles - 1) / kNodeTiles + 7) / 8 * 8;
    const dim3 g0((unsigned)plan_groups(nt)), b0(kLanes), g1((unsigned)(lists + groups)), b1(kBlock);
    switch (order) {
    case 1:
        hipLaunchKernelGGL(k_plan_fast<1>, g0, b0, 0, stream, a, plan);
        if (nodes) hipLaunchKernelGGL(k_plan_nodes<1>, g1, b1, 0, stream, b, lists);
        break;
    case 3:
        hipLaunchKernelGGL(k_plan_fast<3>, g0, b0, 0, stream, a, plan);
        if (nodes) hipLaunchKernelGGL(k_plan_nodes<3>, g1, b1, 0, stream, b, lists);
        break;
    default:
        hipLaunchKernelGGL(k_plan_fast<5>, g0, b0, 0, stream, a, plan);
        if (nodes) hipLaunchKernelGGL(k_plan_nodes<5>, g1, b1, 0, stream, b, lists);
        break;
    }
    return hipGetLastError();
}

hipError_t launch_step_fast(const StepArgs &a, int order, int scan, hipStream_t stream)
{
    if (a.rows.n_tiles <= 0) return hipSuccess;
    if (a.rows.tile != kFastTile) return hipErrorInvalidValue;
    switch (order) {
    case 1: return step_fast_p<1>(a, scan, stream);
    case 3: return step_fast_p<3>(a, scan, stream);
    default: return step_fast_p<5>(a, scan, stream);
    }
}

hipError_t launch_step_fast_lim(const StepArgs &a, int recon, hipStream_t stream)
{
    if (a.rows.n_tiles <= 0) return hipSuccess;
    if (a.rows.tile != kFastTile) return hipErrorInvalidValue;
    return recon == kReconPLM ? step_fast_lim_r<kReconPLM>(a, stream)
                              : step_fast_lim_r<kReconPPM>(a, stream);
}

hipError_t launch_plan_rag(const StepArgs &a, int order, const RagPlan &plan,
                           hipStream_t stream)
{
    if (a.rows.n_tiles <= 0) return hipSuccess;
    if (a.rows.tile != kRagTile || a.dv) return hipErrorInvalidValue;
    const dim3 g((unsigned)((a.rows.n_tiles + kWaves - 1) / kWaves)), b(kBlock);
    switch (order) {
    case 1: hipLaunchKernelGGL(k_plan_rag<1>, g, b, 0, stream, a, plan); break;
    case 3: hipLaunchKernelGGL(k_plan_rag<3>, g, b, 0, stream, a, plan); break;
    default: hipLaunchKernelGGL(k_plan_rag<5>, g, b, 0, stream, a, plan); break;
    }
    return hipGetLastError();
}

hipError_t launch_step_rag(const StepArgs &a, int order, int scan, hipStream_t stream)
{
    if (a.rows.n_tiles <= 0) return hipSuccess;
    if (a.rows.tile != kRagTile || a.dv) return hipErrorInvalidValue;
    switch (order) {
    case 1: return step_rag_p<1>(a, scan, stream);
    case 3: return step_rag_p<3>(a, scan, stream);
    default: return step_rag_p<5>(a, scan, stream);
    }
}

} // namespace ram
