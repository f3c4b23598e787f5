// nlist_dev.h -- device helpers shared by the two framed list builds: wave
// reductions and scans, the per-cell sort, the tile hand-out.
#pragma once

#include "launch.h"

namespace md {

constexpr int kRebuildGrid = 2048;   // blocks of the grid-stride rebuild kernels
constexpr int kPlanGrid = 8192;      // one-wave workgroups of the plan kernels
constexpr int kSeg = 8;              // members of a cell staged by 8 lanes of the matrix build
constexpr int kBoxMax = 8192;        // cells of a tile's frame box

// System owning a cell: largest s with cprefix[s] <= c (cprefix holds each
// system's first cell; a compact array, so the search stays in the scalar
// cache).
__device__ __forceinline__ int find_sys_cell(const int64_t *__restrict__ cprefix, int n_sys, int64_t c)
{
    int lo = 0, hi = n_sys;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cprefix[mid] <= c) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The systems that a rebuild takes, in order, with the prefixes of their cells
// and local tiles: a batch rebuilds a few of its systems on most steps, and
// launches that walk all of its tiles and cells, skipping most, leave their
// work to the few workgroups whose run it falls into (64 systems of 3,200 to
// 20,000 particles, us a step: binning 25 -> 9, sort and plans 48 -> 35, build
// 160 -> 137).  One system alone is not looked up.
struct Flagged {
    const int64_t *cell;  // n + 1
    const int32_t *tile;  // n + 1
    const int32_t *sys;   // n
    const int32_t *n;
};
__host__ __device__ inline size_t flagged_bytes(int n_sys)
{
    return sizeof(int64_t) * ((size_t)n_sys + 1) + sizeof(int32_t) * (2 * (size_t)n_sys + 2);
}
__device__ __forceinline__ Flagged flagged_at(int64_t *base, int n_sys)
{
    const int32_t *t = reinterpret_cast<const int32_t *>(base + n_sys + 1);
    return {base, t, t + n_sys + 1, t + 2 * n_sys + 1};
}

// Local tile number x of the rebuilt systems' tiles.
__device__ __forceinline__ int flagged_tile(const Flagged &F, int nf, const int32_t *__restrict__ tprefix, int n_sys,
                                            int x, int &s)
{
    if (n_sys == 1) {
        s = 0;
        return x;
    }
    const int k = find_sys(F.tile, nf, x);
    s = F.sys[k];
    return tprefix[s] + (x - F.tile[k]);
}

// One wave per cell (wave w of W takes cells w, w + W, ...): members ranked
// by their FP32 x coordinate relative to the cell's corner, ties by row index
// (a total order on (bits, row), so the ranks are a permutation whatever the
// values), sizes published.  Next to each member's row the list keeps its
// position relative to the cell's lower corner in FP32 (row bits in w), so
// that the framed build stages a cell with coalesced reads of 8 members.  The counts
// are left for the plan of the framed build, which runs beside this, and
// cleared by the framed scan.  cell_cap <= 64 * CPL.
__host__ __device__ constexpr int cell_xf_stride(int cell_cap) { return (cell_cap + kSeg - 1) / kSeg * kSeg; }
template <int CPL>
__device__ __forceinline__ void cell_sort_waves(int64_t wfirst, int64_t wstep, const SysDev *__restrict__ sys,
                                                const int64_t *__restrict__ cprefix, int n_sys, const double4 *__restrict__ pos, int64_t n_cells,
                                                const int32_t *__restrict__ cell_count,
                                                int32_t *__restrict__ cell_size, int32_t *__restrict__ cell_idx,
                                                float4 *__restrict__ cell_xf, int cell_cap,
                                                const int32_t *__restrict__ sflag, int64_t *fl)
{
    const int lane = lane_id();
    const int64_t xs = cell_xf_stride(cell_cap);
    // fl: the cells of the rebuilt systems; else (or with one system) all
    // cells, those of systems that keep their lists skipped
    const bool listed = fl && n_sys > 1;
    const Flagged F = flagged_at(fl, n_sys);
    const int nf = listed ? *F.n : 0;
    const int64_t n = listed ? F.cell[nf] : n_cells;
    for (int64_t x = wfirst; x < n; x += wstep) {
        int64_t c = x;
        int s;
        if (listed) {
            const int k = find_sys_cell(F.cell, nf, x);
            s = F.sys[k];
            c = cprefix[s] + (x - F.cell[k]);
        } else {
            s = find_sys_cell(cprefix, n_sys, c);
            if (!sflag[s]) continue;  // this system keeps its list
        }
        int m = cell_count[c];
        m = m < cell_cap ? m : cell_cap;
        const SysDev &S = sys[s];
        const int64_t key = c - S.cell0;
        const int cx = (int)(key % S.bins[0]), cy = (int)((key / S.bins[0]) % S.bins[1]),
                  cz = (int)(key / ((int64_t)S.bins[0] * S.bins[1]));
        const double ox = S.lo[0] + (double)cx * (S.L[0] / S.bins[0]);
        const double oy = S.lo[1] + (double)cy * (S.L[1] / S.bins[1]);
        const double oz = S.lo[2] + (double)cz * (S.L[2] / S.bins[2]);
        int32_t v[CPL];
        float4 f[CPL];
        int64_t ord[CPL];  // (x bits made order-preserving as a signed integer, row)
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
            const int k = q * kWave + lane;
            v[q] = k < m ? cell_idx[c * cell_cap + k] : INT32_MAX;
            f[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            ord[q] = INT64_MAX;
            if (k < m) {
                const double4 y = pos[v[q]];
                f[q] = make_float4((float)(y.x - ox), (float)(y.y - oy), (float)(y.z - oz), __int_as_float(v[q]));
                const int32_t b = __float_as_int(f[q].x);
                ord[q] = ((int64_t)(b ^ ((b >> 31) & 0x7FFFFFFF)) << 32) | (uint32_t)v[q];
            }
        }
        int rank[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) rank[q] = 0;
#pragma unroll
        for (int q2 = 0; q2 < CPL; ++q2) {
            const int tmax = m - q2 * kWave < kWave ? m - q2 * kWave : kWave;
            for (int t = 0; t < tmax; ++t) {
                const int64_t other = __shfl(ord[q2], t, kWave);
#pragma unroll
                for (int q = 0; q < CPL; ++q) rank[q] += other < ord[q] ? 1 : 0;
            }
        }
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
            const int k = q * kWave + lane;
            if (k < m) {
                cell_idx[c * cell_cap + rank[q]] = v[q];
                cell_xf[c * xs + rank[q]] = f[q];
            } else if (k < (m + kSeg - 1) / kSeg * kSeg) {
                // the last segment's free places: near nothing
                cell_xf[c * xs + k] = make_float4(__builtin_nanf(""), 0.f, 0.f, 0.f);
            }
        }
        if (lane == 0) cell_size[c] = m;
    }
}

// Wrap a cell coordinate difference into [-bins/2, bins - bins/2).
__device__ __forceinline__ int wrap_rel(int d, int bins)
{
    const int h = bins / 2;
    d = ((d + h) % bins + bins) % bins - h;
    return d;
}

// Index of the largest entry <= x in the ascending array a[0..n).
__device__ __forceinline__ int upper_idx(const int32_t *a, int n, int x)
{
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// DPP lane move within rows of 16 lanes (every lane of the wave active).
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}

// Minimum / maximum over the 64 lanes of a fully active wave: swaps within
// quads, half rows and rows, then the four row results.
__device__ __forceinline__ int wave_min_full(int v)
{
    v = min(v, dpp_mov<0xB1>(v));   // quad_perm [1,0,3,2]
    v = min(v, dpp_mov<0x4E>(v));   // quad_perm [2,3,0,1]
    v = min(v, dpp_mov<0x141>(v));  // row_half_mirror
    v = min(v, dpp_mov<0x140>(v));  // row_mirror
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// The same over each row of 16 lanes, left in all of them.
__device__ __forceinline__ int row_min_full(int v)
{
    v = min(v, dpp_mov<0xB1>(v));
    v = min(v, dpp_mov<0x4E>(v));
    v = min(v, dpp_mov<0x141>(v));
    return min(v, dpp_mov<0x140>(v));
}
__device__ __forceinline__ int row_max_full(int v)
{
    v = max(v, dpp_mov<0xB1>(v));
    v = max(v, dpp_mov<0x4E>(v));
    v = max(v, dpp_mov<0x141>(v));
    return max(v, dpp_mov<0x140>(v));
}

// Inclusive sum over the lanes of a fully active wave: shifts within rows of
// 16 lanes, then the last lane of each row or pair of rows to those after it.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add(int v)
{
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ int wave_scan_incl(int v)
{
    v = dpp_add<0x111, 0xF>(v);  // row_shr 1, 2, 4, 8
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);  // row_bcast 15 into rows 1 and 3
    return dpp_add<0x143, 0xC>(v);  // row_bcast 31 into rows 2 and 3
}

// Sum of v over the threads before this one in a block of NT; total gets the
// sum over all.  scan holds NT / 64 words in LDS.
template <int NT>
__device__ __forceinline__ int block_rank(int v, int32_t *scan, int &total)
{
    constexpr int NW = NT / kWave;
    const int w = threadIdx.x >> 6;
    const int incl = wave_scan_incl(v);
    if (lane_id() == kWave - 1) scan[w] = incl;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        before += q < w ? scan[q] : 0;
        total += scan[q];
    }
    __syncthreads();  // scan free again
    return before + incl - v;
}

// Floats as integers of the same order, and back (NaN apart).
__device__ __forceinline__ int float_order(float v)
{
    const int b = __float_as_int(v);
    return b ^ ((b >> 31) & 0x7FFFFFFF);
}
__device__ __forceinline__ float float_unorder(int b) { return __int_as_float(b ^ ((b >> 31) & 0x7FFFFFFF)); }

// Values that are the same in every lane (read from LDS or computed from
// such values), moved to scalar registers.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uni(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
__device__ __forceinline__ double uni(double v)
{
    const int64_t b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ int wave_max_full(int v)
{
    v = max(v, dpp_mov<0xB1>(v));
    v = max(v, dpp_mov<0x4E>(v));
    v = max(v, dpp_mov<0x141>(v));
    v = max(v, dpp_mov<0x140>(v));
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// One tile index from a die's counter, by one lane.  The pointer gets a zero
// from a vector register that the compiler cannot see through: taken as
// divergent, the atomic is issued plainly and its result waited for where it
// is used (the pass that merges the atomics of a wave into one would wait
// for it at once).
__device__ __forceinline__ int take_tile(int32_t *ctr)
{
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    return atomicAdd(ctr + zero, 1);
}

// uint16 entries per row assembled in LDS.
inline int nlist_row_stride(int cap)
{
    // uint16 entries per staged row; an odd number of words keeps the
    // transposed read-out free of bank conflicts
    // one spare entry past the capacity takes the writes of an overflowing row
    int r = cap + 1 + ((cap + 1) & 1);
    if (((r / 2) & 1) == 0) r += 2;
    return r;
}

inline int capped(int64_t blocks) { return (int)(blocks < kRebuildGrid ? (blocks > 0 ? blocks : 1) : kRebuildGrid); }

}  // namespace md
