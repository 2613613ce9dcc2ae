// ram_mesh_layout.h -- where the tables of a shared mesh lie in their device
// memory.  The one place that knows their sizes: what is reserved and what is
// carved are the same offsets.  (No HIP types, so that the host can check it.)
#pragma once

#include <cstddef>
#include <cstdint>

namespace ram {

// Cells past the row's end that the FP32 sizes, their reciprocals and the (size,
// inverse gap) pairs go on for, for loads of several cells.
constexpr int kMeshPad = 16;
// Bytes of one record of a cell's stencil (CellRec).
constexpr size_t kCellRecF32 = 64, kCellRecF64 = 112;

// Uniform-run counts: one workgroup up to kRunsAlone cells, else runs_groups of them,
// each with its largest and smallest size and its waves' counts kept (then the two
// sizes of the row).
constexpr int64_t kRunsAlone = 16384;
constexpr int kRunsGroups = 512, kRunsWaves = 8;
inline int runs_groups(int64_t n)
{
    const int64_t g = (n + 4095) / 4096;
    return (int)(g < kRunsGroups ? g : kRunsGroups);
}

// Byte offsets, 256-byte aligned each, and the bytes of all.
struct MeshLayout {
    size_t dx, dxinv, hinv;          // FP64 a cell
    size_t dxf, dxinvf, hinvf;       // FP32, the first two padded
    size_t bucket, bnext;            // the search index: four buckets a cell
    size_t scal;                     // three FP64
    size_t crf, crd;                 // stencil records
    size_t rrf, rrd;                 // (size, inverse gap); FP32 padded
    size_t stp, stpd, stdv;          // stencil planes: FP32, FP64, FP32 deviations
    size_t ppmd, ppmf;               // PPM interface weights, five planes
    size_t nonu, nonu_min;           // uniform-run counts, one more than cells
    size_t runs_size, runs_cnt;      // their groups' sizes and counts (long rows)
    size_t bytes;
};

inline MeshLayout mesh_layout(int64_t n_cells)
{
    const size_t n = (size_t)n_cells, np = n + kMeshPad, nb = 4 * n;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += (bytes + 255) & ~size_t(255);
        return at;
    };
    MeshLayout m;
    m.dx = take(8 * n);
    m.dxinv = take(8 * n);
    m.hinv = take(8 * n);
    m.dxf = take(4 * np);
    m.dxinvf = take(4 * np);
    m.hinvf = take(4 * n);
    m.bucket = take(4 * nb);
    m.bnext = take(16 * nb);
    m.scal = take(24);
    m.crf = take(kCellRecF32 * n);
    m.crd = take(kCellRecF64 * n);
    m.rrf = take(8 * np);
    m.rrd = take(16 * n);
    m.stp = take(36 * n);
    m.stpd = take(96 * n);
    m.stdv = take(36 * n);
    m.ppmd = take(40 * n);
    m.ppmf = take(20 * n);
    m.nonu = take(4 * (n + 1));
    m.nonu_min = take(4 * (n + 1));
    const size_t groups = n_cells > kRunsAlone ? (size_t)kRunsGroups : 0;
    m.runs_size = take(groups ? 16 * (groups + 1) : 0);
    m.runs_cnt = take(8 * groups * kRunsWaves);
    m.bytes = off;
    return m;
}

} // namespace ram
