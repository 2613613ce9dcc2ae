// ram_kernels.hip -- the residual step alone and the tables of a mesh (gfx950).
//
// Rows are independent periodic lines (paper Section 2).
//
//   k_residual   the residual step alone.
//   k_mesh_prep  mesh-only tables of a shared mesh.
//   k_tiles_prep tile table of a ragged batch.
#include "ram_device.h"

#include <algorithm>

#include <type_traits>

namespace ram {
namespace {

using namespace dev;


// ---------------------------------------------------------------------------
// residual step alone
// ---------------------------------------------------------------------------

template <typename TQ>
__global__ __launch_bounds__(kBlock) void k_residual(ResidualArgs a)
{
    // Staged once (index j <-> cell i0-2+j, and face i0-2+j between cells
    // j-1 and j): the state, the face velocities and the mesh data (dx,
    // 1/centre gap, 1/dx); every lane issues its loads before the first LDS
    // store.  Then one face per lane (fluxes on faces i0 .. i0+nd, with the
    // upwind cell's van Leer slope) and one cell per lane (the conservative
    // update), lane-consecutive in LDS, so no access conflicts on a bank.
    using CT = TQ;
    using CT2 = typename TabT<CT>::T2;
    constexpr int NP = kStepNodes + 8;
    __shared__ __attribute__((aligned(16))) CT sq[NP];
    __shared__ __attribute__((aligned(16))) CT sdx[NP];
    __shared__ __attribute__((aligned(16))) CT shv[NP];
    __shared__ __attribute__((aligned(16))) CT sdi[NP];
    __shared__ __attribute__((aligned(16))) CT sf[NP];

    const Rows &R = a.rows;
    Tile ti;
    if (!get_tile(R, blockIdx.x, ti)) return;
    const int n = ti.n;
    const double *x = ti.x;
    const TQ *q = (const TQ *)a.q_in + ti.qoff;
    const TQ *dv = (const TQ *)a.dv + ti.qoff;
    TQ *qo = (TQ *)a.q_out + ti.qoff;
    const CT dt = (CT)a.dt;
    const int i0 = ti.i0;
    const int nd = min(R.tile, n - i0);
    const bool tab = R.has_tab != 0;
    const bool inner = (i0 - 2 >= 0) && (i0 + nd + 2 < n);
    const int t = threadIdx.x;
    const double len = x[n] - x[0];
    CT vq[kItems], vv[kItems], vdi[kItems];
    CT2 vr[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int j = min(t + k * kBlock, nd + 3);
        const int c = inner ? i0 - 2 + j : wrap_small(i0 - 2 + j, n);
        vq[k] = (CT)q[c];
        vv[k] = (CT)dv[c];
        if (tab) {
            vr[k] = TabT<CT>::rr(R.tab)[c];
            vdi[k] = TabT<CT>::dxinv(R.tab)[c];
        }
    }
    CT vd[kItems];                       // face velocity of the face j (cell j's left)
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int j = t + k * kBlock;
        if (j < nd + 4) {
            const int c = inner ? i0 - 2 + j : wrap_small(i0 - 2 + j, n);
            if (!tab) {
                const double d = x[c + 1] - x[c];
                vr[k].x = (CT)d;
                vr[k].y = (CT)(1.0 / centre_gap(x, n, len, c));
                vdi[k] = (CT)(1.0 / d);
            }
            sq[j] = vq[k];
            sdx[j] = vr[k].x;
            shv[j] = vr[k].y;
            sdi[j] = vdi[k];
        }
        vd[k] = vv[k];
    }
    __syncthreads();
    // face f (0 .. nd) lies between cells f+1 and f+2; its velocity is the
    // one staged with cell f+2
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int f = t + k * kBlock - 2;
        if (f >= 0 && f <= nd) {
            const CT v = vd[k];
            const bool up = v >= (CT)0;
            const int c = up ? f + 1 : f + 2;             // upwind cell
            const CT qm = sq[c - 1], q0 = sq[c], qp = sq[c + 1];
            const CT dp = (qp - q0) * shv[c];
            const CT dm = (q0 - qm) * shv[c - 1];
            const CT sg = (dp * dm <= (CT)0) ? (CT)0 : harmonic2(dp, dm);
            const CT qf = up ? q0 + (CT)0.5 * sg * (sdx[c] - v * dt)
                             : q0 - (CT)0.5 * sg * (sdx[c] + v * dt);
            sf[f] = v * qf;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int u = t + k * kBlock;
        if (u < nd) qo[i0 + u] = (TQ)(sq[u + 2] - dt * (sf[u + 1] - sf[u]) * sdi[u + 2]);
    }
}

// ---------------------------------------------------------------------------
// mesh-only tables of a shared mesh
// ---------------------------------------------------------------------------

struct MeshTabW {
    double *dx, *dxinv, *hinv;
    float *dxf, *dxinvf, *hinvf;
    int32_t *bucket;
    double2 *bnext;
    int32_t nb;
    double *scal;
    CellRec<float> *crf;
    CellRec<double> *crd;
    float2 *rrf;
    float *stp;
    double2 *rrd;
    double2 *stpd;
    float *stdv;
    double *ppmd;
    float *ppmf;
    int32_t *nonu;
    int32_t *nonu_min;
    double2 *runs_size;
    int2 *runs_cnt;
};

// Every table of the mesh in one launch of B-thread workgroups, each with one
// part: the uniform-run counts (workgroup 0, when they are asked for), then
// per B cells the sizes, gaps and PPM weights, then the stencils, then per B
// buckets the search index.  Short dependent chains bound it (FP64 divisions,
// node loads of about a microsecond when first touched), not bytes, so the
// parts run side by side instead of one after the other in one thread, and
// the run counts do not wait for a launch of their own.  B: the run counts'
// one workgroup sets the time of rows up to kRunsAlone (it keeps its cells in registers,
// 32 a lane at 16384 cells), four waves a workgroup are quicker to start on
// short ones: 256 threads against 512 4.6 and 6.2 us at 2048 cells, 5.9 and
// 6.3 at 4096, 15.5 and 7.5 at 6001, 20.5 and 12.2 at 16384.  One thread a
// cell and bucket, then the run counts in a launch of their own: 10.2 us at
// 256 cells (now 4.7), 11.1 at 2048, 22.0 at 16384.
constexpr int kPrepShort = 4096;                     // longest row of 256-thread workgroups

// Cell sizes, reciprocals, centre gaps and PPM interface weights of cell j.
__device__ __forceinline__ void prep_sizes(const double *x, int n, int j, const MeshTabW &T)
{
    const double len = x[n] - x[0];
    const double dx = x[j + 1] - x[j];
    const double h = centre_gap(x, n, len, j);
    const double dxi = 1.0 / dx, hi = 1.0 / h;
    T.dx[j] = dx;
    T.dxinv[j] = dxi;
    T.hinv[j] = hi;
    // (the FP32 sizes, their reciprocals and (dx, 1/gap) go on past the row's end)
    for (int k = j; k < n + kMeshPad; k += n) {
        T.dxf[k] = (float)dx;
        T.dxinvf[k] = (float)dxi;
        T.rrf[k] = make_float2((float)dx, (float)hi);
    }
    T.hinvf[j] = (float)hi;
    T.rrd[j] = make_double2(dx, hi);
    const PpmW pw = ppm_weights(x[wrap_small(j - 1, n) + 1] - x[wrap_small(j - 1, n)], dx,
                                x[wrap_small(j + 1, n) + 1] - x[wrap_small(j + 1, n)],
                                x[wrap_small(j + 2, n) + 1] - x[wrap_small(j + 2, n)]);
    const double pv[5] = {pw.d1, pw.d2, pw.e1, pw.e2, pw.e3};
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        T.ppmd[k * n + j] = pv[k];
        T.ppmf[k * n + j] = (float)pv[k];
    }
}

// Stencil data of cell j (order P) in the layouts the kernels read.
template <int P>
__device__ __forceinline__ void prep_stencil(const double *x, int n, int j, const MeshTabW &T)
{
    constexpr int LO = (P - 1) / 2;
    const double len = x[n] - x[0];
    const double dx = x[j + 1] - x[j];
    double th[P + 1];
    const double xc = x[j];
#pragma unroll
    for (int a = 0; a <= P; ++a) th[a] = (node_x(x, n, len, j - LO + a) - xc) / dx;
    // the cell's own edges, exactly (the streaming kernels rely on it)
    th[LO] = 0.0;
    th[LO + 1] = 1.0;
    CellRec<float> rf;
    CellRec<double> rd;
    rf.xc = rd.xc = xc;
    rf.dxinv = rd.dxinv = 1.0 / dx;
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        rf.th[a] = rf.rd[a] = 0.0f;
        rd.th[a] = rd.rd[a] = 0.0;
    }
#pragma unroll
    for (int a = 0; a <= P; ++a) {
        double den = 1.0;
#pragma unroll
        for (int b = 0; b <= P; ++b)
            if (b != a) den *= th[a] - th[b];
        rd.th[a] = th[a];
        rd.rd[a] = 1.0 / den;
        rf.th[a] = (float)th[a];
        rf.rd[a] = (float)rd.rd[a];
    }
    T.crf[j] = rf;
    T.crd[j] = rd;
    {
        float v[9];
        int k = 0;
#pragma unroll
        for (int a = 0; a <= P; ++a)
            if (a != LO && a != LO + 1) v[k++] = rf.th[a];
#pragma unroll
        for (int a = 0; a <= P; ++a)
            if (a != LO) v[k++] = rf.rd[a];
        for (; k < 9; ++k) v[k] = 0.0f;
        float4 *p4 = (float4 *)T.stp;
        p4[j] = make_float4(v[0], v[1], v[2], v[3]);
        p4[n + j] = make_float4(v[4], v[5], v[6], v[7]);
        T.stp[8 * n + j] = v[8];
    }
    {
        // FP64: the cell's left edge and 1/dx, then the same values, in
        // pairs (six planes of double2)
        double v[12];
        int k = 0;
        v[k++] = xc;
        v[k++] = rd.dxinv;
#pragma unroll
        for (int a = 0; a <= P; ++a)
            if (a != LO && a != LO + 1) v[k++] = rd.th[a];
#pragma unroll
        for (int a = 0; a <= P; ++a)
            if (a != LO) v[k++] = rd.rd[a];
        for (; k < 12; ++k) v[k] = 0.0;
#pragma unroll
        for (int pl = 0; pl < 6; ++pl) T.stpd[pl * n + j] = make_double2(v[2 * pl], v[2 * pl + 1]);
        // the same offsets and denominators as FP32 deviations from those
        // of equally spaced nodes (offset b - LO, denominator 1 / prod_{a != b}
        // (b - a)): th_b - (b - LO), and rd_b / rd_eq_b - 1
        float dv9[9];
        int m = 0;
#pragma unroll
        for (int a = 0; a <= P; ++a)
            if (a != LO && a != LO + 1) dv9[m++] = (float)(rd.th[a] - (double)(a - LO));
#pragma unroll
        for (int a = 0; a <= P; ++a) {
            if (a == LO) continue;
            double eq = 1.0;
#pragma unroll
            for (int b = 0; b <= P; ++b)
                if (b != a) eq *= (double)(a - b);
            dv9[m++] = (float)(rd.rd[a] * eq - 1.0);
        }
        for (; m < 9; ++m) dv9[m] = 0.0f;
        float4 *d4 = (float4 *)T.stdv;
        d4[j] = make_float4(dv9[0], dv9[1], dv9[2], dv9[3]);
        d4[n + j] = make_float4(dv9[4], dv9[5], dv9[6], dv9[7]);
        T.stdv[8 * n + j] = dv9[8];
    }
}

// The search index: the lower-bound cell of bucket j, taken a hair below the
// bucket start so that a bucket number rounded up by one still bounds the
// cell from below; then the next two nodes (+inf past the last cell).  Two
// loads deep on rows of up to 64 B cells (a binary search of 16384 nodes is
// fourteen): B nodes sampled evenly over the row, shared by
// the workgroup, place a wave's first bucket within 64 cells; the cells of
// its 64 neighbouring buckets are then found among the kPrepWin nodes from
// there in LDS.  Longer rows narrow 64-fold a load until there; a lane whose
// cell lies beyond the window (a mesh far finer here than on average)
// searches the rest of the row by itself.
constexpr int kPrepWin = 192;
template <int B>
__device__ __forceinline__ void prep_buckets(const double *x, int n, int j, const MeshTabW &T,
                                             double *smp, double *win)
{
    const int t = (int)threadIdx.x, lane = t & 63;
    const double inf = __builtin_huge_val();
    const int step0 = (n + B - 1) / B;
    smp[t] = t * step0 < n ? x[t * step0] : inf;
    const double len = x[n] - x[0];
    const double w = len / (double)T.nb;
    const double tj = x[0] + ((double)j - 1e-6) * w;
    __syncthreads();
    if (j - lane >= T.nb) return;                    // (whole waves)
    const double t0 = __shfl(tj, 0);
    // x[lo] <= t0 (or lo == 0), x[hi] > t0 (or hi == n)
    int k = 0;
#pragma unroll
    for (int i = 0; i < B / 64; ++i) k += __popcll(__ballot(smp[64 * i + lane] <= t0));
    int lo = min(max(k - 1, 0) * step0, n - 1), hi = min(n, lo + step0);
    while (hi - lo > 64) {
        const int step = (hi - lo + 63) / 64;
        const int at = lo + lane * step;
        const int m = __popcll(__ballot((at < hi ? x[at] : inf) <= t0));
        lo = min(lo + max(m - 1, 0) * step, n - 1);
        hi = min(hi, lo + step);
    }
    double v[kPrepWin / 64];
#pragma unroll
    for (int i = 0; i < kPrepWin / 64; ++i) {
        const int at = lo + lane + 64 * i;
        v[i] = at < n ? x[at] : inf;
    }
#pragma unroll
    for (int i = 0; i < kPrepWin / 64; ++i) win[lane + 64 * i] = v[i];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    int cnt = 0;                                     // of the first 128 nodes: at or below tj
#pragma unroll
    for (int d = 64; d > 0; d >>= 1)
        if (win[cnt + d - 1] <= tj) cnt += d;
    if (cnt == 127 && win[127] <= tj) cnt = 128;
    if (j >= T.nb) return;
    int c = max(lo + cnt - 1, 0);
    double2 nx;
    if (cnt < 128) {
        const int d = c - lo;
        nx = make_double2(win[d + 1], win[d + 2]);
    } else {                                         // x[c] <= tj
        int b = n - 1;
        c = min(c, b);
        while (c < b) {
            const int mid = c + (b - c + 1) / 2;
            if (x[mid] <= tj) c = mid;
            else b = mid - 1;
        }
        nx = make_double2(c + 1 < n ? x[c + 1] : inf, c + 2 < n ? x[c + 2] : inf);
    }
    T.bucket[j] = min(c, n - 1);
    T.bnext[j] = nx;
}

// Uniform runs of a shared mesh: prefix counts of the cells whose size
// differs from the largest (nonu) and from the smallest (nonu_min) by more
// than kUniformTol of it.  One workgroup (rows of up to B KEEP cells): each of its
// waves takes one contiguous segment of the row, whose cells it keeps in registers
// (one load of the nodes); both sizes by a block reduction, then each lane flags its
// cells, and after one scan of the waves' counts a wave writes its segment's prefix
// 64 cells at a time from one ballot per flag.
template <int B, int KEEP>
__device__ __forceinline__ void prep_uniform(const double *x, int n, int32_t *nonu,
                                             int32_t *nonu_min, double *sx)
{
    constexpr int kPrepWaves = B / 64;
    double *smax = sx, *smin = sx + kPrepWaves;
    int32_t *soff = (int32_t *)(sx + 2 * kPrepWaves);          // [2][kPrepWaves]
    const int t = (int)threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int seg = (n + kPrepWaves - 1) / kPrepWaves;
    const int a0 = min(n, wv * seg), a1 = min(n, a0 + seg);
    double keep[KEEP];
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        const int j = min(a0 + 64 * k + lane, n - 1);
        keep[k] = x[j + 1] - x[j];
    }
    double mx = 0.0, mn = __builtin_huge_val();
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        mx = fmax(mx, keep[k]);                      // (clamped lanes: cells of the row as well)
        mn = fmin(mn, keep[k]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, o, 64));
        mn = fmin(mn, __shfl_xor(mn, o, 64));
    }
    if (lane == 0) {
        smax[wv] = mx;
        smin[wv] = mn;
    }
    __syncthreads();
    double hx = smax[0], hn = smin[0];
#pragma unroll
    for (int w = 1; w < kPrepWaves; ++w) {
        hx = fmax(hx, smax[w]);
        hn = fmin(hn, smin[w]);
    }
    // a lane's flags: bit k of fx (fn) where its cell k is off the largest (smallest)
    static_assert(KEEP <= 32, "a bit a cell");
    uint32_t fx = 0, fn = 0;
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        const bool in = a0 + 64 * k + lane < a1;
        fx |= in && fabs(keep[k] - hx) > kUniformTol * hx ? 1u << k : 0u;
        fn |= in && fabs(keep[k] - hn) > kUniformTol * hn ? 1u << k : 0u;
    }
    // (held as bits, the lane's cells counted by them: as masks they are 3 KEEP scalar
    // pairs, which spill; the tables of 11,840 cells 8.7 us, 11.6 so)
    int lw = lane;
    asm volatile("" : "+v"(fx), "+v"(fn), "+v"(lw));
    int32_t cx = 0, cn = 0;
    if constexpr (KEEP <= 4) {                       // (few masks; 0.2 us less of a row of 256)
#pragma unroll
        for (int k = 0; k < KEEP; ++k) {
            cx += __popcll(__ballot((fx >> k & 1u) != 0));
            cn += __popcll(__ballot((fn >> k & 1u) != 0));
        }
    } else {
        int32_t c = __popc(fx) | __popc(fn) << 16;   // (64 KEEP cells at most)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
        cx = c & 0xffff;
        cn = c >> 16;
    }
    if (lane == 0) {
        soff[wv] = cx;
        soff[kPrepWaves + wv] = cn;
    }
    __syncthreads();
    int32_t bx = 0, bn = 0, tx = 0, tn = 0;
#pragma unroll
    for (int w = 0; w < kPrepWaves; ++w) {
        const int32_t ux = soff[w], un = soff[kPrepWaves + w];
        bx += w < wv ? ux : 0;
        bn += w < wv ? un : 0;
        tx += ux;
        tn += un;
    }
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        if (a0 + 64 * k >= a1) break;
        const int j = a0 + 64 * k + lw;
        const uint64_t kx = __ballot((fx >> k & 1u) != 0), kn = __ballot((fn >> k & 1u) != 0);
        if (j < a1) {
            nonu[j] = bx + __popcll(kx & below);
            nonu_min[j] = bn + __popcll(kn & below);
        }
        bx += __popcll(kx);
        bn += __popcll(kn);
    }
    if (t == 0) {
        nonu[n] = tx;
        nonu_min[n] = tn;
    }
}

// The same of a row beyond kRunsAlone cells, shared out: every workgroup takes one
// contiguous segment.  Here its largest and smallest size; in k_runs_count the
// row's, and its waves' flagged cells; in k_runs_write the prefix.  One shift of a
// row of 2^20 cells: FP32 189 us, 2160 with the counts as one workgroup; three rows
// of 100,001 cells 64 and 157.
constexpr int kRunsB = 64 * kRunsWaves;
__device__ __forceinline__ int runs_segment(int n, int groups)
{
    return ((n + groups - 1) / groups + kRunsB - 1) / kRunsB * kRunsB;
}

__device__ __forceinline__ double2 runs_reduce(double mx, double mn, double *sx)
{
    const int t = (int)threadIdx.x;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, o, 64));
        mn = fmin(mn, __shfl_xor(mn, o, 64));
    }
    if ((t & 63) == 0) {
        sx[t >> 6] = mx;
        sx[kRunsWaves + (t >> 6)] = mn;
    }
    __syncthreads();
    mx = sx[0];
    mn = sx[kRunsWaves];
#pragma unroll
    for (int w = 1; w < kRunsWaves; ++w) {
        mx = fmax(mx, sx[w]);
        mn = fmin(mn, sx[kRunsWaves + w]);
    }
    return make_double2(mx, mn);
}

__device__ __forceinline__ void prep_runs_size(const double *x, int n, int b, int groups,
                                               double2 *size, double *sx)
{
    const int seg = runs_segment(n, groups);
    const int64_t a0 = (int64_t)b * seg;
    const int a1 = (int)min((int64_t)n, a0 + seg);
    double mx = 0.0, mn = __builtin_huge_val();
#pragma unroll 4
    for (int64_t j = a0 + threadIdx.x; j < a1; j += kRunsB) {
        const double d = x[j + 1] - x[j];
        mx = fmax(mx, d);
        mn = fmin(mn, d);
    }
    const double2 m = runs_reduce(mx, mn, sx);
    if (threadIdx.x == 0) size[b] = m;
}

// Cell j's flags: its size is not the largest, not the smallest (to kUniformTol of it).
__device__ __forceinline__ void run_flags(const double *x, int64_t j, int a1, double2 h, uint64_t &fx,
                                          uint64_t &fn)
{
    const bool in = j < a1;
    const int64_t c = min(j, (int64_t)a1 - 1);
    const double d = x[c + 1] - x[c];
    fx = __ballot(in && fabs(d - h.x) > kUniformTol * h.x);
    fn = __ballot(in && fabs(d - h.y) > kUniformTol * h.y);
}

__global__ __launch_bounds__(kRunsB) void k_runs_count(const double *x, int n, int groups,
                                                       double2 *size, int2 *cnt)
{
    __shared__ double sx[2 * kRunsWaves];
    const int t = (int)threadIdx.x, lane = t & 63, wv = t >> 6, b = (int)blockIdx.x;
    static_assert(kRunsGroups <= kRunsB, "a group's sizes a thread");
    double2 m = make_double2(0.0, __builtin_huge_val());
    if (t < groups) m = size[t];
    m = runs_reduce(m.x, m.y, sx);
    if (b == 0 && t == 0) size[kRunsGroups] = m;
    const int seg = runs_segment(n, groups), part = seg / kRunsWaves;
    const int64_t a0 = min((int64_t)n, (int64_t)b * seg + wv * part);
    const int a1 = (int)min((int64_t)n, a0 + part);
    int2 c = make_int2(0, 0);
#pragma unroll 4
    for (int64_t j0 = a0; j0 < a1; j0 += 64) {
        uint64_t fx, fn;
        run_flags(x, j0 + lane, a1, m, fx, fn);
        c.x += __popcll(fx);
        c.y += __popcll(fn);
    }
    if (lane == 0) cnt[b * kRunsWaves + wv] = c;
}

__global__ __launch_bounds__(kRunsB) void k_runs_write(const double *x, int n, int groups,
                                                       const double2 *size, const int2 *cnt,
                                                       int32_t *nonu, int32_t *nonu_min)
{
    __shared__ int2 sc[kRunsWaves];
    const int t = (int)threadIdx.x, lane = t & 63, wv = t >> 6, b = (int)blockIdx.x;
    const double2 m = size[kRunsGroups];
    // the flagged cells before this wave's
    int2 c = make_int2(0, 0);
    for (int i = t; i < b * kRunsWaves; i += kRunsB) {
        c.x += cnt[i].x;
        c.y += cnt[i].y;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        c.x += __shfl_xor(c.x, o, 64);
        c.y += __shfl_xor(c.y, o, 64);
    }
    if (lane == 0) sc[wv] = c;
    __syncthreads();
    int32_t bx = 0, bn = 0;
#pragma unroll
    for (int w = 0; w < kRunsWaves; ++w) {
        bx += sc[w].x;
        bn += sc[w].y;
        if (w < wv) {
            bx += cnt[b * kRunsWaves + w].x;
            bn += cnt[b * kRunsWaves + w].y;
        }
    }
    const int seg = runs_segment(n, groups), part = seg / kRunsWaves;
    const int64_t a0 = min((int64_t)n, (int64_t)b * seg + wv * part);
    const int a1 = (int)min((int64_t)n, a0 + part);
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll 2
    for (int64_t j0 = a0; j0 < a1; j0 += 64) {
        uint64_t fx, fn;
        run_flags(x, j0 + lane, a1, m, fx, fn);
        if (j0 + lane < a1) {
            nonu[j0 + lane] = bx + __popcll(fx & below);
            nonu_min[j0 + lane] = bn + __popcll(fn & below);
        }
        bx += __popcll(fx);
        bn += __popcll(fn);
    }
    if (b == groups - 1 && wv == kRunsWaves - 1 && lane == 0) {
        nonu[n] = bx;
        nonu_min[n] = bn;
    }
}

// runs: workgroups that take the uniform-run counts (0: not asked for).
template <int P, int B>
__global__ __launch_bounds__(B) void k_mesh_prep(const double *x, int n, MeshTabW T,
                                                 int runs, unsigned groups, CopyJob copy)
{
    if (blockIdx.x >= groups) return copy_part(copy, blockIdx.x - groups, gridDim.x - groups);
    __shared__ double sx[B];
    __shared__ double swin[B / 64][kPrepWin];
    const int t = (int)threadIdx.x;
    const int nc = (n + B - 1) / B;
    int b = (int)blockIdx.x;
    if (b < runs) {
        constexpr int K1 = B == 256 ? 4 : 12, K2 = B == 256 ? 16 : 32;
        if (B == kRunsB && runs > 1) prep_runs_size(x, n, b, runs, T.runs_size, sx);
        else if (n <= B * K1) prep_uniform<B, K1>(x, n, T.nonu, T.nonu_min, sx);
        else prep_uniform<B, K2>(x, n, T.nonu, T.nonu_min, sx);
        return;
    }
    b -= runs;
    if (b < nc) {
        const int j = b * B + t;
        if (j < n) prep_sizes(x, n, j, T);
    } else if (b < 2 * nc) {
        const int j = (b - nc) * B + t;
        if (j < n) prep_stencil<P>(x, n, j, T);
        if (j == 0) {
            const double len = x[n] - x[0];
            T.scal[0] = (double)T.nb / len;
            T.scal[1] = 1.0 / len;
            T.scal[2] = x[0] * ((double)T.nb / len);
        }
    } else {
        prep_buckets<B>(x, n, (b - 2 * nc) * B + t, T, sx, swin[t >> 6]);
    }
}

// ---------------------------------------------------------------------------
// ragged-row tile table: tile_ptr[r] = sum_{r'<r} ceil(N_r'/tile) and
// tile_row[t] = row of tile t.
// ---------------------------------------------------------------------------

// Every workgroup scans all the rows' tile counts (consecutive rows a thread;
// the same first tiles written by each), then fills in its own share of the
// tiles' rows, kFillRows rows a wave, a row at a time with consecutive tiles on
// the lanes: the fill is instruction issue, too much for one CU.  4096 rows of
// 17 tiles on average: 10 us; 48 as one workgroup, each thread writing its own
// rows' tiles one after the other.  A batch of few rows of few tiles keeps to that
// form: 3000 rows of 6 .. 200 cells 1.2 us less of a call.
constexpr int kFillRows = 8;
constexpr int64_t kFillFew = 8192, kFillTiles = 8;
__global__ __launch_bounds__(1024) void k_tiles_prep(const int64_t *row_ptr,
                                                     int64_t n_rows, int tile,
                                                     int64_t *tile_ptr,
                                                     int32_t *tile_row, unsigned groups,
                                                     CopyJob copy)
{
    if (blockIdx.x >= groups) return copy_part(copy, blockIdx.x - groups, gridDim.x - groups);
    __shared__ int64_t swt[16];
    const int t = (int)threadIdx.x, lane = t & 63, wv = t >> 6;
    const int64_t per = (n_rows + 1023) / 1024;
    const int64_t r0 = min(n_rows, (int64_t)t * per);
    const int64_t r1 = min(n_rows, r0 + per);
    int64_t run = 0, p0 = r0 < r1 ? row_ptr[r0] : 0;
    bool many = n_rows > kFillFew;
    for (int64_t r = r0; r < r1; ++r) {
        const int64_t p1 = row_ptr[r + 1];
        const int64_t k = (p1 - p0 + tile - 1) / tile;
        run += k;
        many = many || k > kFillTiles;
        p0 = p1;
    }
    int64_t inc = run;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    if (lane == 63) swt[wv] = inc;
    const bool own = __syncthreads_or(many ? 1 : 0) == 0;
    if (own && blockIdx.x > 0) return;
    int64_t acc = inc - run, total = 0;
    for (int w = 0; w < 16; ++w) {
        acc += w < wv ? swt[w] : 0;
        total += swt[w];
    }
    p0 = r0 < r1 ? row_ptr[r0] : 0;
    for (int64_t r = r0; r < r1; ++r) {
        const int64_t p1 = row_ptr[r + 1];
        const int64_t to = acc + (p1 - p0 + tile - 1) / tile;
        tile_ptr[r] = acc;
        if (own)
            for (int64_t i = acc; i < to; ++i) tile_row[i] = (int32_t)r;
        acc = to;
        p0 = p1;
    }
    if (t == 1023) tile_ptr[n_rows] = total;
    if (own) return;
    __threadfence_block();
    __syncthreads();
    const int64_t wave = (int64_t)blockIdx.x * 16 + wv;
    for (int64_t c = kFillRows * wave; c < n_rows; c += kFillRows * 16 * (int64_t)groups) {
        // the rows' first tiles at once, then one row after the other
        const int64_t r = c + min(lane, kFillRows - 1);
        const int64_t base = tile_ptr[c];
        const int first = (int)(tile_ptr[min(r, n_rows)] - base);
        const int end = (int)(tile_ptr[min(r + 1, n_rows)] - base);
        const int m = (int)min((int64_t)kFillRows, n_rows - c);
        int32_t *to = tile_row + base;
        for (int k = 0; k < m; ++k) {
            const int a = __builtin_amdgcn_readlane(first, k), b = __builtin_amdgcn_readlane(end, k);
            for (int i = a + lane; i < b; i += 64) to[i] = (int32_t)(c + k);
        }
    }
}

template <int B>
hipError_t mesh_prep_launch(const double *x, int64_t n, int order, const MeshTabW &w, bool uniform,
                            const CopyJob &c, hipStream_t st)
{
    const int64_t nc = (n + B - 1) / B;
    const int u = uniform ? (n > kRunsAlone ? runs_groups(n) : 1) : 0;
    const unsigned gp = (unsigned)(2 * nc + ((int64_t)w.nb + B - 1) / B + u);
    const dim3 g(gp + c.blocks(B)), b(B);
    switch (order) {
    case 1: hipLaunchKernelGGL((k_mesh_prep<1, B>), g, b, 0, st, x, (int)n, w, u, gp, c); break;
    case 3: hipLaunchKernelGGL((k_mesh_prep<3, B>), g, b, 0, st, x, (int)n, w, u, gp, c); break;
    default: hipLaunchKernelGGL((k_mesh_prep<5, B>), g, b, 0, st, x, (int)n, w, u, gp, c); break;
    }
    if (u > 1) {
        hipLaunchKernelGGL(k_runs_count, dim3(u), dim3(kRunsB), 0, st, x, (int)n, u, w.runs_size,
                           w.runs_cnt);
        hipLaunchKernelGGL(k_runs_write, dim3(u), dim3(kRunsB), 0, st, x, (int)n, u, w.runs_size,
                           w.runs_cnt, w.nonu, w.nonu_min);
    }
    return hipGetLastError();
}

} // namespace

hipError_t launch_mesh_prep(const double *x, int64_t n, int order, void *mem,
                            MeshTab &tab, hipStream_t stream, bool uniform, const CopyJob &copy)
{
    const MeshLayout m = mesh_layout(n);
    char *p = (char *)mem;
    MeshTabW w;
    w.dx = (double *)(p + m.dx);
    w.dxinv = (double *)(p + m.dxinv);
    w.hinv = (double *)(p + m.hinv);
    w.dxf = (float *)(p + m.dxf);
    w.dxinvf = (float *)(p + m.dxinvf);
    w.hinvf = (float *)(p + m.hinvf);
    w.bucket = (int32_t *)(p + m.bucket);
    w.nb = (int32_t)(4 * n);
    w.bnext = (double2 *)(p + m.bnext);
    w.scal = (double *)(p + m.scal);
    w.crf = (CellRec<float> *)(p + m.crf);
    w.crd = (CellRec<double> *)(p + m.crd);
    w.rrf = (float2 *)(p + m.rrf);
    w.stp = (float *)(p + m.stp);
    w.rrd = (double2 *)(p + m.rrd);
    w.stpd = (double2 *)(p + m.stpd);
    w.stdv = (float *)(p + m.stdv);
    w.ppmd = (double *)(p + m.ppmd);
    w.ppmf = (float *)(p + m.ppmf);
    w.nonu = (int32_t *)(p + m.nonu);
    w.nonu_min = (int32_t *)(p + m.nonu_min);
    w.runs_size = (double2 *)(p + m.runs_size);
    w.runs_cnt = (int2 *)(p + m.runs_cnt);
    tab.dx = w.dx; tab.dxinv = w.dxinv; tab.hinv = w.hinv;
    tab.dxf = w.dxf; tab.dxinvf = w.dxinvf; tab.hinvf = w.hinvf;
    tab.bucket = w.bucket;
    tab.nb = w.nb;
    tab.scal = w.scal;
    tab.bnext = w.bnext;
    tab.crf = w.crf;
    tab.crd = w.crd;
    tab.rrf = w.rrf;
    tab.stp = w.stp;
    tab.rrd = w.rrd;
    tab.stpd = w.stpd;
    tab.stdv = w.stdv;
    tab.ppmd = w.ppmd;
    tab.ppmf = w.ppmf;
    tab.nonu = uniform ? w.nonu : nullptr;
    tab.nonu_min = uniform ? w.nonu_min : nullptr;
    if (n <= kPrepShort) return mesh_prep_launch<256>(x, n, order, w, uniform, copy, stream);
    return mesh_prep_launch<512>(x, n, order, w, uniform, copy, stream);
}

hipError_t launch_tiles_prep(const int64_t *row_ptr, int64_t n_rows, int tile,
                             int64_t *tile_ptr, int32_t *tile_row,
                             hipStream_t stream, const CopyJob &copy)
{
    // (more than 64 workgroups only repeat the scan)
    const unsigned g = (unsigned)std::min<int64_t>((n_rows + 16 * kFillRows - 1) / (16 * kFillRows), 64);
    hipLaunchKernelGGL(k_tiles_prep, dim3(g + copy.blocks(1024)), dim3(1024), 0, stream, row_ptr,
                       n_rows, tile, tile_ptr, tile_row, g, copy);
    return hipGetLastError();
}

hipError_t launch_residual(const ResidualArgs &a, bool f64, hipStream_t stream)
{
    if (a.rows.n_tiles <= 0) return hipSuccess;
    // the staged window (tile + 4 cells) must fit kItems slots a lane
    if (a.rows.tile > kResTile) return hipErrorInvalidValue;
    const dim3 grid((unsigned)a.rows.n_tiles), block(kBlock);
    if (f64)
        hipLaunchKernelGGL(k_residual<double>, grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL(k_residual<float>, grid, block, 0, stream, a);
    return hipGetLastError();
}

// Plain copy kernel (16-byte words, then the tail bytes): also usable inside
// a captured graph, where it keeps copy nodes out.
__global__ __launch_bounds__(256) void k_copy(const unsigned char *src, unsigned char *dst,
                                              int64_t bytes)
{
    const int64_t nw = bytes / 16;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = i0; i < nw; i += stride)
        ((uint4 *)dst)[i] = ((const uint4 *)src)[i];
    for (int64_t b = nw * 16 + i0; b < bytes; b += stride) dst[b] = src[b];
}

hipError_t launch_copy(const void *src, void *dst, int64_t bytes,
                       hipStream_t stream)
{
    if (bytes <= 0) return hipSuccess;
    if ((((uintptr_t)src | (uintptr_t)dst) & 15) != 0)
        return hipMemcpyAsync(dst, src, (size_t)bytes, hipMemcpyDeviceToDevice, stream);
    const int64_t nw = (bytes + 15) / 16;
    const unsigned grid = (unsigned)std::min<int64_t>((nw + 255) / 256, 8192);
    hipLaunchKernelGGL(k_copy, dim3(grid), dim3(256), 0, stream,
                       (const unsigned char *)src, (unsigned char *)dst, bytes);
    return hipGetLastError();
}

} // namespace ram
