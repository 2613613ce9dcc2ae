// ram_wave.h -- wave-level helpers of the kernels that run one tile of
// kFastTile destination cells a wave (the FP32 streaming step and its
// adjoint): LDS visibility inside a wave, DPP prefix sums, records read with
// scalar loads, tile positions.
#pragma once

#include "ram_device.h"

namespace ram {
namespace dev {

constexpr int kLanes = 64;
constexpr int kWaves = kBlock / kLanes;             // tiles per workgroup

// Every lane's LDS writes visible to the whole wave (a wave executes its LDS
// instructions in order; the fences keep the compiler from moving accesses
// across).
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline int wrap1f(int j, int n) { return j < 0 ? j + n : (j >= n ? j - n : j); }

// Tile id -> row and first cell (tiles of kFastTile cells, row by row).
struct TilePos {
    int row, i0, nd;
    bool inner;          // the tile and its halo do not wrap the row
};
__device__ inline TilePos tile_pos(int tile, int n, int H)
{
    const int tpr = (n + kFastTile - 1) / kFastTile;
    TilePos p;
    p.row = tile / tpr;
    p.i0 = (tile - p.row * tpr) * kFastTile;
    p.nd = min(kFastTile, n - p.i0);
    p.inner = (p.i0 - H >= 0) && (p.i0 + p.nd + H < n);
    return p;
}

// A record, read through the constant address space: with a wave-uniform
// address these are scalar loads (the host pass, which only checks device
// code, reads it plainly).
__device__ inline FastTile load_rec(const FastTile *rec, int64_t i = 0)
{
    FastTile r;
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const __attribute__((address_space(4))) int32_t *CI;
    const CI c = (CI)(rec + i);
    int32_t *o = (int32_t *)&r;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(FastTile) / 4); ++k) o[k] = c[k];
#else
    r = rec[i];
#endif
    return r;
}

// A word of a table the same way.
__device__ inline int load_index(const int32_t *p, int i)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return ((const __attribute__((address_space(4))) int32_t *)p)[i];
#else
    return p[i];
#endif
}

// The step kernels' grids: the host does not know how the tiles split, so the
// uniform kernels' has a wave for every tile (the ones past totals[0] return
// at once) and the others' a wave for every second, each stepping through the
// list by the grid's size.  On 24000 searching tiles a wave for every fourth,
// second and one takes 66, 57 and 58 us a step (whole rounds of the chip's
// waves are left over); on the 2048 x 16384 disk, one tile in six searching,
// 1995, 1990 and 2032 us for twenty steps (waves without a tile).
inline unsigned uniform_grid(int64_t n_tiles) { return (unsigned)((n_tiles + kWaves - 1) / kWaves); }
inline unsigned other_grid(int64_t n_tiles)
{
    return (unsigned)((n_tiles + 2 * kWaves - 1) / (2 * kWaves));
}

// Wave index inside the workgroup, in a scalar register (so that what it
// selects is read with scalar loads).
__device__ inline int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x / kLanes); }

// Load / store at a 32-bit byte offset from a wave-uniform base: the access
// takes the scalar-base form (base in SGPRs, one 32-bit offset a lane)
// instead of a 64-bit address formed in every lane.  The streaming kernels
// run on rows of fewer than kFastMaxCols cells, so no offset wraps.
template <class T>
__device__ __forceinline__ T ld_at(const void *base, uint32_t byte_off)
{
    return *(const T *)((const char *)base + byte_off);
}
template <class T>
__device__ __forceinline__ void st_at(void *base, uint32_t byte_off, const T &v)
{
    *(T *)((char *)base + byte_off) = v;
}

// Inclusive scan of one value a lane over the wave in DPP steps (row shifts,
// then the row-15 and row-31 broadcasts; lanes without a source read zero),
// and lane 63's value read back as a scalar.
template <class AC>
__device__ __forceinline__ typename AC::A wave_inclusive(typename AC::A inc)
{
    inc = AC::comb(AC::template dpp<kDppRowShr1, 0xf, 0xf>(inc), inc);
    inc = AC::comb(AC::template dpp<kDppRowShr2, 0xf, 0xf>(inc), inc);
    inc = AC::comb(AC::template dpp<kDppRowShr4, 0xf, 0xf>(inc), inc);
    inc = AC::comb(AC::template dpp<kDppRowShr8, 0xf, 0xf>(inc), inc);
    inc = AC::comb(AC::template dpp<kDppBcast15, 0xa, 0xf>(inc), inc);
    inc = AC::comb(AC::template dpp<kDppBcast31, 0xc, 0xf>(inc), inc);
    return inc;
}
__device__ __forceinline__ float lane63(float v)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kLanes - 1));
}
__device__ __forceinline__ float2 lane63(float2 v) { return make_float2(lane63(v.x), lane63(v.y)); }
__device__ __forceinline__ double lane63(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), kLanes - 1);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), kLanes - 1);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The prefix modes (S other than kSumDirect): the window's exclusive
// cumulative of the masses, in the mode's precision (Acc<S>), at LDS index
// j + off for window cell j and one past the window's last group; partial
// integrals and whole-cell sums are then its differences (only differences:
// the cells below the window start in the first group cancel).  Masses of
// groups g = l + 64 s (s = 0, 1, ...), four a lane: each group's lane totals
// scanned across the wave, the groups before carried on.
template <int S>
__device__ __forceinline__ void wave_prefix(typename Acc<S>::A *sp, const typename Acc<S>::M (&m)[4],
                                            int g, int gl, typename Acc<S>::A &carry)
{
    using AC = Acc<S>;
    using A = typename AC::A;
    const int lane = (int)threadIdx.x % kLanes;
    const bool live = g <= gl;
    A tot = AC::zero();
    if (live) {
#pragma unroll
        for (int k = 0; k < 4; ++k) tot = AC::add(tot, m[k]);
    }
    // inclusive scan of the lane totals over the wave
    const A inc = wave_inclusive<AC>(tot);
    A ex = AC::template dpp<kDppWaveShr1, 0xf, 0xf>(inc);
    if (lane == 0) ex = AC::zero();
    A e = AC::comb(carry, ex);
    if (live) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            sp[4 * g + k] = e;
            e = AC::add(e, m[k]);
        }
        if (g == gl) sp[4 * g + 4] = e;
    }
    carry = AC::comb(carry, lane63(inc));
}

// Moves a small per-lane array down one slot (v[0] = v[1], ...), for loops
// over slots that are not unrolled: they read slot 0 each trip, since an
// array indexed at run time is placed in scratch memory, whose stores reach
// HBM.
template <class T, int N>
__device__ __forceinline__ void slot_down(T (&v)[N])
{
#pragma unroll
    for (int i = 0; i + 1 < N; ++i) v[i] = v[i + 1];
}
template <class T, int N, int M>
__device__ __forceinline__ void slot_down(T (&v)[N][M])
{
#pragma unroll
    for (int i = 0; i + 1 < N; ++i)
#pragma unroll
        for (int k = 0; k < M; ++k) v[i][k] = v[i + 1][k];
}

// The same, the first slot's value going to the last (after N turns every slot
// is back in its place).
template <class T, int N>
__device__ __forceinline__ void slot_turn(T (&v)[N])
{
    const T first = v[0];
#pragma unroll
    for (int i = 0; i + 1 < N; ++i) v[i] = v[i + 1];
    v[N - 1] = first;
}
} // namespace dev
} // namespace ram
