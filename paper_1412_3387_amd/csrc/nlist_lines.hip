// nlist_lines.hip -- the framed list build with line-ordered rows, which
// mixed-precision DPD keeps.
//
// The order of a row's entries decides how the FP64 sum of its forces rounds,
// so it moves every velocity in its last bit; a DPD pair's FP32 drag and noise
// follow the velocities and separations of the step before, and where such a
// bit crosses an FP32 rounding the pair's force moves by an FP32 ulp of its
// amplitude (up to 60: 4e-6, a velocity by 8e-8).  The matrix build's rows
// (nlist.hip) come in another order, and within 10 steps a few of 1,000,000
// DPD particles so leave the trajectories these rows give; LJ, whose FP32
// terms see positions only, and FP64 runs stay within 1e-12 of them.  So
// mixed DPD runs this build (0.56 ms for 1,000,000 particles, the matrix build
// 0.33 ms).
//
//   * A tile's cells are placed in one frame, as in nlist.hip; the distinct
//     cells come out in box order, so the three x-adjacent cells of a row's
//     stencil line are three consecutive distinct cells: a row's candidates
//     are nine contiguous slot ranges ("runs"), x-ordered and cut to the
//     row's x-window by binary search.
//   * One wave takes one row at a time; its 64 lanes split the nine runs in
//     proportion to their lengths (at least one lane each).  A candidate whose
//     FP32 distance lies clearly inside or outside r_list is decided there;
//     one within the tile's band of r_list^2 is decided by the exact FP64
//     test, so the list is exactly the FP64 one.
//   * Rows are assembled in LDS and written out coalesced after the halo
//     numbering.
#include <algorithm>

#include "nlist_dev.h"
#include "nlist_general.h"

namespace md {

constexpr int kLineWavesMax = 8;     // waves per workgroup at most
constexpr int kLineChunk = 2560;     // members staged at once (float4 each)
constexpr int kLineSlotMax = 8192;   // members of a framed tile's stencil cells
constexpr int kUMax = 256;           // distinct cells of a framed tile
constexpr int kBoxWords = kBoxMax / 32;
constexpr int kRuns = 9;             // x-lines of cells around a row
static_assert(kUMax <= 256, "slot map holds distinct cells as bytes");

// Exclusive scan of n <= 8 * NT values held in LDS `a` (in place) by a block
// of NT threads with wave-level shuffles; returns the total.
// The barriers order LDS accesses only (the caller's global accesses may stay
// in flight).
template <int NT>
__device__ __forceinline__ int block_scan_w(int32_t *a, int n, int32_t *wsum)
{
    constexpr int NW = NT / kWave;
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int w = tid >> 6;
    const int b = 8 * tid;
    int v[8];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        v[k] = b + k < n ? a[b + k] : 0;
        sum += v[k];
    }
    int inc = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int y = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += y;
    }
    if (lane == kWave - 1) wsum[w] = inc;
    lds_barrier();
    int before = 0, total = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        const int x = wsum[q];
        before += q < w ? x : 0;
        total += x;
    }
    int run = before + inc - sum;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (b + k < n) {
            a[b + k] = run;
            run += v[k];
        }
    lds_barrier();
    return total;
}

// Exclusive scan in place of a[0..n), n <= 4 * 64, by one fully active
// wave; returns the total.
__device__ __forceinline__ int wave_scan_excl(int32_t *a, int n)
{
    const int lane = lane_id();
    int v[4];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = lane * 4 + k;
        v[k] = i < n ? a[i] : 0;
        sum += v[k];
    }
    int inc = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int y = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += y;
    }
    const int total = __shfl(inc, kWave - 1, kWave);
    int run = inc - sum;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = lane * 4 + k;
        if (i < n) a[i] = run;
        run += v[k];
    }
    return total;
}
static_assert(kBoxWords <= 4 * kWave && kUMax <= 4 * kWave, "one-wave scans of the plan");

struct PlanShared {
    uint32_t box[kBoxWords];
    int32_t bpre[kBoxWords + 1];
    int32_t ucell[kUMax];
    int32_t ustart[kUMax + 1];
};


struct LineShared {
    float4 cp[kLineChunk];               // member position in the frame (FP32), row in w
    int32_t ucell[kUMax];                // cell index of each distinct cell
    float4 uoff[kUMax];                  // frame position of each distinct cell's corner (FP32)
    int32_t ustart[kUMax + 1];           // first slot of each distinct cell
    uint32_t used[kLineSlotMax / 32];
    int32_t wpre[kLineSlotMax / 32 + 1];
    uint32_t run[kTile][kRuns];          // slot range of each row line: lo | hi << 16
    uint32_t runc[kTile][kRuns];         // the same cut to the chunk and to the line's x-window
    float hw[kTile][kRuns];              // half width in x of each row line
    float4 xrow[kTile];                  // row position in the frame (FP32)
    int32_t rown[kTile];                 // hits of each row so far
    uint64_t lmask[kTile];               // per row: bit of the last lane of each (non-empty) line but the last
    uint8_t lb[kTile][kRuns + 1];        // per row: first lane of each (non-empty) line, then the lanes used
    int32_t scan[kLineWavesMax];         // per-wave totals of the block scans
    uint8_t smap[kLineChunk];            // distinct cell of each slot of the chunk
    double xref[3];                      // first row's position: the frame reference
    int32_t info[5];                     // distinct cells, per-pair image flag, longest row, slots,
                                         // FP32 decision band (float bits)
    int32_t grab[2];                     // tile indices taken from the die's counter
};

// Per-tile plan of the line-ordered build, written by k_cells_and_lines and read
// by k_build_lines: a header {distinct cells (-1: passed on), slots, per-pair
// image flag, 0}, then per distinct cell {cell, first slot} and its corner
// in the frame, per row its frame position, and per row line its slot range
// and the half width in x that its y-z distance leaves.
struct LinePlan {
    int4 *hdr;
    int2 *cell;
    float4 *off;
    float4 *xrow;
    uint32_t *run;
    float *hw;
};

__host__ __device__ inline LinePlan line_plan(char *base, int64_t tiles)
{
    LinePlan P;
    size_t off = 0;
    auto carve = [&](size_t bytes) {
        char *p = base + off;
        off += (bytes + 255) / 256 * 256;
        return p;
    };
    P.hdr = reinterpret_cast<int4 *>(carve(sizeof(int4) * tiles));
    P.cell = reinterpret_cast<int2 *>(carve(sizeof(int2) * tiles * kUMax));
    P.off = reinterpret_cast<float4 *>(carve(sizeof(float4) * tiles * kUMax));
    P.xrow = reinterpret_cast<float4 *>(carve(sizeof(float4) * tiles * kTile));
    P.run = reinterpret_cast<uint32_t *>(carve(sizeof(uint32_t) * tiles * kTile * kRuns));
    P.hw = reinterpret_cast<float *>(carve(sizeof(float) * tiles * kTile * kRuns));
    return P;
}

// The plan of one tile per wave: lane t takes row t, its home cell in the
// frame, its nine x-lines of three cells marked in a bitmap over the frame's
// box, the distinct cells in box order with their sizes and first slots, every
// line cut to the cells within r_list and its half width in x.
__device__ __forceinline__ void plan_lines(
    PlanShared &ps, int pb, int npb, const SysDev *__restrict__ sys, const int32_t *__restrict__ tprefix,
    int n_sys, int tiles, const double4 *__restrict__ pos, const int32_t *__restrict__ cell_count, int cell_cap,
    double4 *__restrict__ xbuild, int32_t *__restrict__ slow_list, int32_t *__restrict__ slow_n, LinePlan plan,
    const int32_t *__restrict__ sflag, int32_t *__restrict__ halo_n, int halo_lds,
    int32_t *__restrict__ rare_list, int32_t *__restrict__ rare_n)
{
    uint32_t *box = ps.box;
    int32_t *bpre = ps.bpre;
    int32_t *ucell = ps.ucell;
    int32_t *ustart = ps.ustart;
    const int lane = lane_id();
    int64_t tfirst, tend;
    int tstep;
    die_range(pb, npb, tiles, tfirst, tend, tstep);
    for (int tile = (int)tfirst; tile < tend; tile += tstep) {
        const int s = find_sys(tprefix, n_sys, tile);
        if (!sflag[s]) {
            // a system that keeps its list: its tile goes back on the list of
            // tiles that the force pass takes first if its last build put it there
            // (the binning launch before this one emptied that list)
            if (lane == 0) {
                const int32_t hn = halo_n[tile];
                if (hn < 0 || (hn & 0xFFFF) > halo_lds) rare_list[atomicAdd(rare_n, 1)] = tile;
            }
            continue;
        }
        const SysDev &S = sys[s];
        const double Ls[3] = {S.L[0], S.L[1], S.L[2]};
        const int bins[3] = {S.bins[0], S.bins[1], S.bins[2]};
        const int per[3] = {S.per[0], S.per[1], S.per[2]};
        const int64_t row0 = S.row0, cell0 = S.cell0;
        const int n_local = S.n_local;
        const double rl2 = S.rl2;
        const int r0 = (tile - S.tile0) * kTile;
        if (r0 >= n_local) {
            // a tile past the local rows (room for particles that may
            // arrive): an empty list and halo, nothing to build
            if (lane == 0) {
                plan.hdr[tile] = make_int4(0, 0, 0, 0);
                halo_n[tile] = 0;
            }
            continue;
        }
        const float cw[3] = {(float)(Ls[0] / bins[0]), (float)(Ls[1] / bins[1]), (float)(Ls[2] / bins[2])};
        auto pass_on = [&]() {
            if (lane == 0) {
                slow_list[atomicAdd(slow_n, 1)] = tile;
                plan.hdr[tile] = make_int4(-1, 0, 0, 0);
            }
        };

        // ---- rows: home cell in the frame, frame position, build position ----
        const int r = r0 + lane;
        const bool act = r < n_local;
        const double4 xi = pos[row0 + (act ? r : r0)];
        if (act) xbuild[row0 + r] = make_double4(xi.x, xi.y, xi.z, 0.0);
        const double xr[3] = {uni(xi.x), uni(xi.y), uni(xi.z)};  // row 0 of the tile
        const double xa[3] = {xi.x, xi.y, xi.z};
        int c0[3], h[3], elo[3], ehi[3];
        float xf[3], frel[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            c0[a] = uni(cell_coord(xr[a], S.lo[a], S.scale[a], bins[a]));
            const int ci = cell_coord(xa[a], S.lo[a], S.scale[a], bins[a]);
            const int d = ci - c0[a];
            const int sft = bins[a] / 2;
            const int hc[2] = {per[a] ? wrap_rel(d, bins[a]) : d, per[a] ? sft + wrap_rel(d - sft, bins[a]) : d};
            int mn[2], mx[2];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                mn[v] = wave_min_full(act ? hc[v] : INT32_MAX);
                mx[v] = wave_max_full(act ? hc[v] : INT32_MIN);
            }
            const int pick = mx[1] - mn[1] < mx[0] - mn[0] ? 1 : 0;
            h[a] = hc[pick];
            elo[a] = pick ? mn[1] : mn[0];
            ehi[a] = pick ? mx[1] : mx[0];
            // image of the row in the frame: the home cell at c0 + h
            const int kimg = per[a] ? (c0[a] + h[a] - ci) / bins[a] : 0;
            xf[a] = (float)((xa[a] + (double)kimg * Ls[a]) - xr[a]);
            frel[a] = (float)(xa[a] - S.lo[a]) - (float)ci * cw[a];
        }
        plan.xrow[(int64_t)tile * kTile + lane] = make_float4(xf[0], xf[1], xf[2], 0.f);
        // spread of the rows around row 0 per axis (xf is relative to it;
        // non-negative floats order as their bit patterns)
        float spread[3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
            spread[a] = __int_as_float(wave_max_full(act ? __float_as_int(fabsf(xf[a])) : 0));

        // ---- frame box and the stencil-cell bitmap ----------------------------
        int blo[3], X[3];
        bool pass = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            int lo_ = elo[a] - 1, hi_ = ehi[a] + 1;
            if (!per[a]) {
                lo_ = lo_ > -c0[a] ? lo_ : -c0[a];
                hi_ = hi_ < bins[a] - 1 - c0[a] ? hi_ : bins[a] - 1 - c0[a];
            } else if (bins[a] < 3 || hi_ - lo_ + 1 > bins[a]) {
                pass = true;
            }
            blo[a] = lo_;
            X[a] = hi_ - lo_ + 1;
            if ((double)X[a] * (double)cw[a] > 512.0 * sqrt(rl2)) pass = true;
        }
        const int vol = X[0] * X[1] * X[2];
        if (pass || vol > kBoxMax) {
            pass_on();
            continue;
        }
        const int nbw = (vol + 31) >> 5;
        __syncthreads();  // LDS of the previous tile no longer read
        for (int q = lane; q < nbw; q += kWave) box[q] = 0u;
        __syncthreads();
        // a row's stencil as nine x-lines of (up to) three adjacent cells:
        // consecutive bits of one box row
        if (act) {
            for (int rr = 0; rr < kRuns; ++rr) {
                const int fy = h[1] + rr % 3 - 1, fz = h[2] + rr / 3 - 1;
                if (!per[1] && (c0[1] + fy < 0 || c0[1] + fy >= bins[1])) continue;
                if (!per[2] && (c0[2] + fz < 0 || c0[2] + fz >= bins[2])) continue;
                int xa_ = h[0] - 1, xb_ = h[0] + 1;
                if (!per[0]) {
                    xa_ = c0[0] + xa_ >= 0 ? xa_ : -c0[0];
                    xb_ = c0[0] + xb_ < bins[0] ? xb_ : bins[0] - 1 - c0[0];
                }
                const int b = ((fz - blo[2]) * X[1] + (fy - blo[1])) * X[0] + (xa_ - blo[0]);
                const uint64_t bits = ((1ull << (xb_ - xa_ + 1)) - 1ull) << (b & 31);
                atomicOr(&box[b >> 5], (uint32_t)bits);
                if (bits >> 32) atomicOr(&box[(b >> 5) + 1], (uint32_t)(bits >> 32));
            }
        }
        __syncthreads();

        // ---- distinct cells (box order), sizes, first slots ----------------------
        for (int q = lane; q < nbw; q += kWave) bpre[q] = __popc(box[q]);
        __syncthreads();
        const int nu = uni(wave_scan_excl(bpre, nbw));
        __syncthreads();
        if (nu > kUMax || nu < 1) {
            pass_on();
            continue;
        }
        for (int b = lane; b < vol; b += kWave) {
            const uint32_t word = box[b >> 5];
            if ((word >> (b & 31)) & 1u) ucell[bpre[b >> 5] + __popc(word & ((1u << (b & 31)) - 1u))] = b;
        }
        __syncthreads();
        // four distinct cells per lane; every lane reads a valid cell (the
        // last one again past the end) so that the reads are in flight together
        int cells[4];
        float4 offs[4];
        int sizes[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int u = lane + k * kWave;
            const int b = ucell[u < nu ? u : nu - 1];
            const int f[3] = {b % X[0] + blo[0], (b / X[0]) % X[1] + blo[1], b / (X[0] * X[1]) + blo[2]};
            int pc[3];
            float off[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                pc[a] = c0[a] + f[a];
                const int ki = pc[a] >= bins[a] ? 1 : (pc[a] < 0 ? -1 : 0);
                pc[a] -= ki * bins[a];
                // the cell's lower corner in the frame, relative to the reference
                off[a] = (float)((S.lo[a] + (double)pc[a] * (Ls[a] / bins[a]) + (double)ki * Ls[a]) - xr[a]);
            }
            cells[k] = (int32_t)(cell0 + ((int64_t)pc[2] * bins[1] + pc[1]) * bins[0] + pc[0]);
            offs[k] = make_float4(off[0], off[1], off[2], 0.f);
            sizes[k] = cell_count[cells[k]];
        }
        __syncthreads();  // ucell no longer read
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int u = lane + k * kWave;
            if (u < nu) ustart[u] = sizes[k] < cell_cap ? sizes[k] : cell_cap;
        }
        __syncthreads();
        const int nslot = uni(wave_scan_excl(ustart, nu));
        if (lane == 0) ustart[nu] = nslot;
        __syncthreads();
        if (nslot > kLineSlotMax) {
            pass_on();
            continue;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int u = lane + k * kWave;
            if (u < nu) {
                plan.cell[(int64_t)tile * kUMax + u] = make_int2(cells[k], ustart[u]);
                plan.off[(int64_t)tile * kUMax + u] = offs[k];
            }
        }

        // ---- every row line cut to the cells within r_list; x half widths -----
        const float rl2f = (float)rl2 * 1.0001f + 1e-3f;
        float fext = 0.f;
#pragma unroll
        for (int a = 0; a < 3; ++a) fext = fmaxf(fext, (float)X[a] * cw[a]);
        // bound on the FP32 error of a frame x difference, with room to spare
        const float xmargin = 1e-3f + fext * 0x1p-18f;
        const int64_t pr = ((int64_t)tile * kTile + lane) * kRuns;
        for (int rr = 0; rr < kRuns; ++rr) {
            uint32_t v = 0u;
            float hwv = 0.f;
            if (act) {
                const int dy = rr % 3 - 1, dz = rr / 3 - 1;
                const int hx = h[0], hy = h[1] + dy, hz = h[2] + dz;
                bool in = (per[1] || (c0[1] + hy >= 0 && c0[1] + hy < bins[1])) &&
                          (per[2] || (c0[2] + hz >= 0 && c0[2] + hz < bins[2]));
                // squared distance in y and z from the row to the line's cells
                // (a lower bound for every member of the line)
                float gyz = 0.f;
                if (dy != 0) {
                    const float gg = dy < 0 ? frel[1] : cw[1] - frel[1];
                    gyz += gg > 0.f ? gg * gg : 0.f;
                }
                if (dz != 0) {
                    const float gg = dz < 0 ? frel[2] : cw[2] - frel[2];
                    gyz += gg > 0.f ? gg * gg : 0.f;
                }
                in = in && gyz <= rl2f;
                if (in) {
                    const float fx = frel[0];
                    const float gl = fx > 0.f ? fx : 0.f, gr = cw[0] - fx > 0.f ? cw[0] - fx : 0.f;
                    const bool left = (per[0] || c0[0] + hx - 1 >= 0) && gl * gl + gyz <= rl2f;
                    const bool right = (per[0] || c0[0] + hx + 1 < bins[0]) && gr * gr + gyz <= rl2f;
                    const int xa_ = hx + (left ? -1 : 0), xb_ = hx + (right ? 1 : 0);
                    const int b = ((hz - blo[2]) * X[1] + (hy - blo[1])) * X[0] + (xa_ - blo[0]);
                    const int u0 = bpre[b >> 5] + __popc(box[b >> 5] & ((1u << (b & 31)) - 1u));
                    const int u1 = u0 + (xb_ - xa_);
                    v = (uint32_t)ustart[u0] | ((uint32_t)ustart[u1 + 1] << 16);
                    hwv = sqrtf(fmaxf(rl2f - gyz, 0.f)) + xmargin;
                }
            }
            plan.run[pr + rr] = v;
            plan.hw[pr + rr] = hwv;
        }
        // One image per halo entry (the one nearest row 0, taken by the force
        // pass at every step) is every row's minimum image while, per
        // periodic axis, spread + r_list + 2 r_buff < L/2: until the next
        // build each particle moves at most r_buff/2, so a row stays within
        // spread + r_buff of row 0 and a listed pair within r_list + r_buff,
        // and the partner image nearest the row is within L/2 of row 0 (the
        // rows' FP32 offsets get a margin of 1e-5 L).  Otherwise the force
        // pass takes the minimum image per pair.
        int pp = 0;
        {
            const double rlist = sqrt(rl2), rbuff = 2.0 * sqrt(S.disp2);
            for (int a = 0; a < 3; ++a)
                if (per[a] && (double)spread[a] + rlist + 2.0 * rbuff + 1e-5 * Ls[a] >= 0.5 * Ls[a]) pp = 1;
        }
        // relative band around r_list^2 inside which the FP32 distance of a
        // candidate cannot decide the test: a bound on the FP32 rounding of
        // frame coordinates up to E in magnitude (cell-relative position,
        // cell corner, their sum, the row's position: |error| <= 2^-24 (4E +
        // |dx|) per separation), propagated through r^2 and doubled
        const double Ef = (double)fext + (double)fmaxf(cw[0], fmaxf(cw[1], cw[2]));
        const double rl = sqrt(rl2);
        const double eta = 0x1p-24 * (4.0 * Ef + 1.01 * rl);
        const double dr2 = 2.0 * sqrt(3.0) * rl * eta + 3.0 * eta * eta + 3.0 * 0x1p-24 * rl2 * 1.01;
        const float band = (float)(2.0 * (dr2 / rl2 + 3.0 * 0x1p-24));
        if (lane == 0) plan.hdr[tile] = make_int4(nu, nslot, pp, __float_as_int(band));
    }
}

// The cell sort and the plans of the line-ordered build in one launch of one-wave
// workgroups: both read only the binning results, so the first n_sort
// workgroups sort cells while the others plan tiles.
template <int CPL>
__global__ __launch_bounds__(kWave) void k_cells_and_lines(
    int n_sort, const SysDev *__restrict__ sys, const int64_t *__restrict__ cprefix, int n_sys,
    const int32_t *__restrict__ tprefix, int tiles,
    const double4 *__restrict__ pos, int64_t n_cells, const int32_t *__restrict__ cell_count,
    int32_t *__restrict__ cell_size, int32_t *__restrict__ cell_idx, float4 *__restrict__ cell_xf, int cell_cap,
    double4 *__restrict__ xbuild, int32_t *__restrict__ slow_list, int32_t *__restrict__ slow_n, LinePlan plan,
    const int32_t *__restrict__ flag, const int32_t *__restrict__ sflag, int32_t *__restrict__ halo_n,
    int halo_lds, int32_t *__restrict__ rare_list, int32_t *__restrict__ rare_n)
{
    if (*flag == 0) return;
    if ((int)blockIdx.x < n_sort) {
        cell_sort_waves<CPL>(blockIdx.x, n_sort, sys, cprefix, n_sys, pos, n_cells, cell_count, cell_size, cell_idx,
                             cell_xf, cell_cap, sflag, nullptr);
    } else {
        __shared__ PlanShared ps;
        plan_lines(ps, (int)blockIdx.x - n_sort, (int)gridDim.x - n_sort, sys, tprefix, n_sys, tiles, pos,
                   cell_count, cell_cap, xbuild, slow_list, slow_n, plan, sflag, halo_n, halo_lds, rare_list, rare_n);
    }
}

// A plan header read through the vector memory path: the index gets a zero
// from a vector register that the compiler cannot see through, so the read is
// not made a scalar one (a pending scalar read would be waited for at the
// next LDS barrier).
__device__ __forceinline__ int4 next_header(const int4 *hdr, int tile)
{
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    return hdr[tile + zero];
}

// NT threads per workgroup: NT / 64 waves share a tile, a wave scans a row at
// a time.
constexpr int kLineBytes = (int)((sizeof(LineShared) + 15) / 16 * 16);

template <bool EXCL, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_build_lines(
    const SysDev *__restrict__ sys, const int32_t *__restrict__ tprefix, int n_sys, int tiles,
    const double4 *__restrict__ pos, const int32_t *__restrict__ tag, const int32_t *__restrict__ ptag,
    const int32_t *__restrict__ cell_size, const int32_t *__restrict__ cell_idx,
    const float4 *__restrict__ cell_xf, int cell_cap, int xf_stride,
    uint16_t *__restrict__ nlist, int32_t *__restrict__ nn, int cap, int rstride,
    int32_t *__restrict__ halo, int32_t *__restrict__ halo_n, int halo_cap, LinePlan plan,
    int halo_lds, int32_t *__restrict__ rare_list, int32_t *__restrict__ rare_n, int32_t *__restrict__ tile_ctr,
    int32_t *__restrict__ cell_count, int64_t n_cells,
    double4 *__restrict__ xbuild, double4 *__restrict__ tref, const int32_t *__restrict__ slow_list,
    const int32_t *__restrict__ slow_n,
    const int32_t *__restrict__ flag, const int32_t *__restrict__ sflag, int32_t *build_count, Status *st)
{
    if (*flag == 0) return;
    // the binning counts, read by the cell sort and the plans, back to zero
    // for the next build
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n_cells; c += (int64_t)gridDim.x * blockDim.x)
        cell_count[c] = 0;
    extern __shared__ float4 lds_lines[];
    LineShared &sh = *reinterpret_cast<LineShared *>(lds_lines);
    // [kTile][rstride]: staged slot of each hit
    uint16_t *const srows = reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(lds_lines) + kLineBytes);
    // The tiles that the plan passed on, first, where their time hides (as a
    // launch of their own 54 us of most builds of 1,000,000 particles, and an
    // empty launch of every other step); staged and in the order of chunks as
    // in workgroups of 512 always.
    if constexpr (NT == kBuildThreads) {
        for (int it = blockIdx.x; it < *slow_n; it += gridDim.x)
            general_tile<EXCL, NT, kChunk>(*reinterpret_cast<GeneralShared<kChunk> *>(lds_lines), slow_list[it], sys,
                                           tprefix, n_sys, pos, tag, ptag, cell_size, cell_idx, nullptr, cell_cap,
                                           nlist, nn, cap, halo, halo_n, halo_cap, xbuild, tref, halo_lds, rare_list,
                                           rare_n, st);
    }
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wv = tid >> 6;
    constexpr int kWaves = NT / kWave;
    static_assert(kWaves >= 2 && kWaves <= kLineWavesMax, "a loader wave and at least one more");
    if (blockIdx.x == 0 && tid == 0) atomicAdd(build_count, 1);

    // Each die's workgroups walk one contiguous run of tiles.  With one
    // system every tile of the run is built, and the tiles are handed out one
    // at a time from the die's counter (cleared by the binning launch): a
    // workgroup that meets costly tiles takes fewer, so the launch ends with
    // its run.  The loader wave (which makes no global writes, so its wait
    // for the count waits for no write) takes the tile after next as a tile
    // starts.  A batch rebuilds only some systems, and a count for every tile
    // it skips would cost more than it balances: there the workgroups of a
    // die take every step-th tile of the run, and skip without a barrier.
    const bool dyn = n_sys == 1;
    const int D = (int)gridDim.x < kDies ? (int)gridDim.x : kDies;
    const int die = (int)blockIdx.x % D;
    int64_t tfirst, tend;
    int tstep;
    die_range(blockIdx.x, gridDim.x, tiles, tfirst, tend, tstep);
    const int64_t dfirst = (int64_t)tiles * die / D;
    int32_t *ctr = tile_ctr + die * kTileCtrStride;
    int grabbed = 0;
    int64_t t_next = tfirst;
    if (dyn) {
        if (tid == kWave) {
            sh.grab[0] = take_tile(ctr);
            grabbed = take_tile(ctr);
        }
        lds_barrier();
        t_next = dfirst + sh.grab[0];
    }
    int par = 0;
    // each tile's plan header is read one tile ahead, by every thread, with
    // no branch, so that the read stays in flight until its use
    int4 hd_next = next_header(plan.hdr, t_next < tend ? (int)t_next : 0);
    bool built = false;  // a tile was built since the last barrier (its LDS may still be read)
    for (;;) {
        if (dyn) {
            // the next tile's index, taken during the last tile
            par ^= 1;
            if (tid == kWave) sh.grab[par] = grabbed;
        }
        if (dyn || built) lds_barrier();  // LDS of the previous tile no longer read; the index published
        built = false;
        const int64_t t_cur = t_next;
        t_next = dyn ? dfirst + sh.grab[par] : t_cur + tstep;
        if (t_cur >= tend) break;
        if (dyn && tid == kWave) grabbed = take_tile(ctr);  // the tile after next
        const int tile = (int)t_cur;
        const int4 hd_tile = hd_next;
        hd_next = next_header(plan.hdr, t_next < tend ? (int)t_next : tile);
        const int s = find_sys(tprefix, n_sys, tile);
        if (!sflag[s]) continue;  // a system that keeps its list
        built = true;
        const SysDev &S = sys[s];
        const double Ls[3] = {S.L[0], S.L[1], S.L[2]};
        const double iL[3] = {S.invL[0], S.invL[1], S.invL[2]};
        const int64_t row0 = S.row0, nl0 = S.nl0;
        const int n_local = S.n_local;
        const double rl2 = S.rl2;
        const int r0 = (tile - S.tile0) * kTile;

        // ---- 1. the tile's plan ------------------------------------------------
        // Wave 1 does this tile's global reads and no global writes: a wave's
        // wait for a read also waits for all of its earlier writes, and the
        // other waves still have the previous tile's rows in flight.
        const bool loader = wv == 1;
        const int tr = tid - kWave;  // lane of the loader wave
        if (loader) {
            const int4 hd = hd_tile;
            if (tr == 0) {
                sh.info[0] = hd.x;
                sh.info[1] = hd.z;
                sh.info[3] = hd.y;
                sh.info[4] = hd.w;
            }
            if (hd.x > 0) {
                const int nu_ = hd.x < kUMax ? hd.x : kUMax;
                const int64_t pu = (int64_t)tile * kUMax, pr = (int64_t)tile * kTile * kRuns;
                // every read issued before the first is used: cells past the
                // end read the last one again
                int2 cs[kUMax / kWave];
                float4 os[kUMax / kWave];
                uint32_t rv[kRuns];
                float hv[kRuns];
#pragma unroll
                for (int k = 0; k < kUMax / kWave; ++k) {
                    const int u = tr + k * kWave;
                    cs[k] = plan.cell[pu + (u < nu_ ? u : nu_ - 1)];
                    os[k] = plan.off[pu + (u < nu_ ? u : nu_ - 1)];
                }
#pragma unroll
                for (int k = 0; k < kRuns; ++k) {
                    rv[k] = plan.run[pr + tr + k * kWave];
                    hv[k] = plan.hw[pr + tr + k * kWave];
                }
                const float4 xw = plan.xrow[(int64_t)tile * kTile + tr];
                const double4 x0 = pos[row0 + r0];
#pragma unroll
                for (int k = 0; k < kUMax / kWave; ++k) {
                    const int u = tr + k * kWave;
                    if (u < nu_) {
                        sh.ucell[u] = cs[k].x;
                        sh.ustart[u] = cs[k].y;
                        sh.uoff[u] = os[k];
                    }
                }
#pragma unroll
                for (int k = 0; k < kRuns; ++k) {
                    const int e = tr + k * kWave;
                    sh.run[e / kRuns][e % kRuns] = rv[k];
                    sh.hw[e / kRuns][e % kRuns] = hv[k];
                }
                sh.xrow[tr] = xw;
                if (tr == 0) {
                    sh.ustart[nu_] = hd.y;
                    sh.xref[0] = x0.x;
                    sh.xref[1] = x0.y;
                    sh.xref[2] = x0.z;
                }
            }
        } else if (wv == 0) {
            sh.rown[tid] = r0 + tid < n_local ? 0 : -1;
        }
        lds_barrier();
        const int nu = uni(sh.info[0]);
        const int nslot = uni(sh.info[3]);
        if (nu <= 0 || nu > kUMax || nslot > kLineSlotMax) continue;  // built by the general kernel
        const double xr[3] = {uni(sh.xref[0]), uni(sh.xref[1]), uni(sh.xref[2])};
        for (int q = tid; q < (nslot + 31) / 32; q += NT) sh.used[q] = 0u;
        // ---- 5. stage members a chunk at a time, scan every row's lines -------------
        const bool one_chunk = nslot <= kLineChunk;
        // FP32 distances below lo_f are hits, above hi_f misses, in between
        // the exact FP64 test decides (the band comes with the tile's plan)
        const double band = (double)__int_as_float(uni(sh.info[4]));
        const float lo_f = (float)(rl2 * (1.0 - band)), hi_f = (float)(rl2 * (1.0 + band));
        for (int q0 = 0; q0 < nslot; q0 += kLineChunk) {
            const int q1 = q0 + kLineChunk < nslot ? q0 + kLineChunk : nslot;
            lds_barrier();
            // slot -> distinct cell of the chunk: each cell writes its index
            // over its own slots
            for (int u = tid; u < nu; u += NT) {
                int qa = sh.ustart[u], qb = sh.ustart[u + 1];
                qa = qa > q0 ? qa : q0;
                qb = qb < q1 ? qb : q1;
                for (int q = qa; q < qb; ++q) sh.smap[q - q0] = (uint8_t)u;
            }
            lds_barrier();
            // staging: one coalesced read per member (cell-relative FP32
            // position and row), moved into the frame by its cell's corner;
            // four reads of a thread in flight at once
            {
                constexpr int kB = 4;
                for (int qb = q0 + tid; qb < q1; qb += kB * NT) {
                    int us[kB], qs[kB];
                    float4 cs[kB];
#pragma unroll
                    for (int k = 0; k < kB; ++k) {
                        const int q = qb + k * NT;
                        qs[k] = q;
                        us[k] = q < q1 ? (int)sh.smap[q - q0] : 0;
                    }
#pragma unroll
                    for (int k = 0; k < kB; ++k)
                        if (qs[k] < q1) cs[k] = cell_xf[(int64_t)sh.ucell[us[k]] * xf_stride + (qs[k] - sh.ustart[us[k]])];
#pragma unroll
                    for (int k = 0; k < kB; ++k) {
                        const int q = qb + k * NT;
                        if (q < q1) {
                            const float4 o = sh.uoff[us[k]];
                            sh.cp[q - q0] = make_float4(cs[k].x + o.x, cs[k].y + o.y, cs[k].z + o.z, cs[k].w);
                        }
                    }
                }
            }
            lds_barrier();
            // members of a line are ordered by x (cells in x order, each sorted
            // by x): cut every line, within this chunk, to the slots within the
            // half width that its y-z distance leaves (|dx|^2 <= r_list^2 - gap^2,
            // widened by a margin for the FP32 frame coordinates)
            for (int e = tid; e < kTile * kRuns; e += NT) {
                const int t = e / kRuns, rr = e - kRuns * (e / kRuns);
                const uint32_t v = sh.run[t][rr];
                int a = (int)(v & 0xffffu), b = (int)(v >> 16);
                a = a > q0 ? a : q0;
                b = b < q1 ? b : q1;
                if (b <= a) {
                    sh.runc[t][rr] = 0u;
                    continue;
                }
                const float hw = sh.hw[t][rr];
                const float xc = sh.xrow[t].x;
                const float tlo = xc - hw, thi = xc + hw;
                // first slot with x >= tlo, first slot with x > thi
                int pa = a, pb = a;
                int step = 1;
                while (2 * step <= b - a) step *= 2;
                for (; step > 0; step >>= 1) {
                    if (pa + step <= b && sh.cp[pa + step - 1 - q0].x < tlo) pa += step;
                    if (pb + step <= b && sh.cp[pb + step - 1 - q0].x <= thi) pb += step;
                }
                sh.runc[t][rr] = (uint32_t)pa | ((uint32_t)(pb > pa ? pb : pa) << 16);
            }
            lds_barrier();
            // lanes to lines, one thread per row: line r takes lanes [B_r, B_r+1)
            // with B_r = r + about 55 P_r / T (P_r the members of the row's lines
            // before line r in this chunk, T all of them), so every line keeps at
            // least one lane and longer lines get more.  Kept as the first lanes
            // and a mask with the last lane of every line but the last.
            if (tid < kTile) {
                int lens[kRuns];
                int tot = 0;
#pragma unroll
                for (int r = 0; r < kRuns; ++r) {
                    const uint32_t rv = sh.runc[tid][r];
                    const int x0_ = (int)(rv & 0xffffu), x1_ = (int)(rv >> 16);
                    lens[r] = x1_ > x0_ ? x1_ - x0_ : 0;
                    tot += lens[r];
                }
                const uint32_t inv = tot > 0 ? 65536u / (uint32_t)tot : 0u;  // floor(2^16 / T)
                uint64_t mask = 0;
                int pre = 0, b0 = 0;
#pragma unroll
                for (int r = 0; r < kRuns; ++r) {
                    const int pn = pre + lens[r];
                    const int b1 = r == kRuns - 1 ? kWave : r + 1 + (int)((55u * (uint32_t)pn * inv) >> 16);
                    sh.lb[tid][r] = (uint8_t)b0;
                    if (r < kRuns - 1) mask |= 1ull << (b1 - 1);
                    b0 = b1;
                    pre = pn;
                }
                sh.lb[tid][kRuns] = (uint8_t)kWave;
                sh.lmask[tid] = tot > 0 ? mask : 0ull;
                if (tot == 0 && sh.rown[tid] >= 0) sh.lb[tid][0] = 0xFF;  // nothing to scan in this chunk
            }
            lds_barrier();
            for (int t = wv; t < kTile; t += kWaves) {
                int ntot = uni(sh.rown[t]);
                if (ntot < 0) continue;  // inactive row
                if (uni((int)sh.lb[t][0]) == 0xFF) continue;  // no members in this chunk
                // this lane's line: the lines that end before it; its lanes,
                // members (cut to the chunk) and stride
                const uint64_t lm = sh.lmask[t];
                int myline = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(lm >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)lm, 0u));
                myline = myline < kRuns - 1 ? myline : kRuns - 1;
                const int blo_ = sh.lb[t][myline], bhi_ = sh.lb[t][myline + 1];
                const uint32_t rv = sh.runc[t][myline];
                const int x0_ = (int)(rv & 0xffffu), x1_ = (int)(rv >> 16);
                const int gsz = bhi_ - blo_ > 1 ? bhi_ - blo_ : 1;
                const int base = x0_ + (lane - blo_);
                const int end = x1_;
                const float4 xt0 = sh.xrow[t];
                const float4 xt = make_float4(uni(xt0.x), uni(xt0.y), uni(xt0.z), 0.f);
                const int32_t it = (int32_t)(row0 + r0 + t);
                int32_t part[kMaxBondCap];
                if constexpr (EXCL) {
                    const int64_t prow = (int64_t)it * S.bond_stride;
#pragma unroll
                    for (int bnd = 0; bnd < kMaxBondCap; ++bnd)
                        part[bnd] = bnd < S.bond_cap ? ptag[prow + bnd] : -1;
                }
                uint16_t *myrow = srows + t * rstride;
                // exact FP64 decision of a candidate whose FP32 distance is
                // within the band around r_list
                auto exact = [&](const float4 c) -> bool {
                    const int32_t j = __float_as_int(c.w);
                    const double4 xa = pos[it], xb = pos[j];
                    const double cj[3] = {(double)c.x, (double)c.y, (double)c.z};
                    const double xt3[3] = {(double)xt.x, (double)xt.y, (double)xt.z};
                    const double pa[3] = {xa.x, xa.y, xa.z}, pb[3] = {xb.x, xb.y, xb.z};
                    double d[3];
#pragma unroll
                    for (int ax = 0; ax < 3; ++ax) {
                        // frame images of both: k = round((frame - stored) / L)
                        const double kj = rint((cj[ax] + xr[ax] - pb[ax]) * iL[ax]);
                        const double ki = rint((xt3[ax] + xr[ax] - pa[ax]) * iL[ax]);
                        d[ax] = pb[ax] - pa[ax];
                        if (kj != ki) d[ax] = d[ax] + (kj - ki) * Ls[ax];
                    }
                    return norm2_exact(d[0], d[1], d[2]) < rl2 && j != it;
                };
                auto excluded = [&](bool hit, const float4 c) -> bool {
                    if constexpr (EXCL) {
                        if (hit) {
                            const int32_t tj = tag[__float_as_int(c.w)];
#pragma unroll
                            for (int bnd = 0; bnd < kMaxBondCap; ++bnd) hit = hit && part[bnd] != tj;
                        }
                    }
                    return hit;
                };
                // a hit goes to the row's next entry (entries past the
                // capacity land on the row's spare slot) and marks its slot
                auto append = [&](bool hit, uint64_t mask, int q) {
                    if (hit) {
                        const int p = ntot + (int)__builtin_amdgcn_mbcnt_hi(
                                                 (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                        myrow[p < cap ? p : cap] = (uint16_t)q;
                        atomicOr(&sh.used[q >> 5], 1u << (q & 31));
                    }
                    ntot += __popcll(mask);
                };
                // every lane reads a slot of the chunk, clamped: lanes past
                // their line's end take no part
                const float4 *cq = sh.cp - q0;
                const int qlast = q1 - 1;
                for (int qa = base;; qa += 2 * gsz) {
                    const int qb = qa + gsz;
                    const bool ona = qa < end, onb = qb < end;
                    if (__ballot(ona) == 0ull) break;
                    const float4 ca = cq[qa < qlast ? qa : qlast];
                    const float4 cb = cq[qb < qlast ? qb : qlast];
                    const float dxa = ca.x - xt.x, dya = ca.y - xt.y, dza = ca.z - xt.z;
                    const float dxb = cb.x - xt.x, dyb = cb.y - xt.y, dzb = cb.z - xt.z;
                    const float r2a = dxa * dxa + dya * dya + dza * dza;
                    const float r2b = dxb * dxb + dyb * dyb + dzb * dzb;
                    bool ha = ona && r2a < lo_f && __float_as_int(ca.w) != it;
                    bool hb = onb && r2b < lo_f && __float_as_int(cb.w) != it;
                    const bool ba = ona && r2a >= lo_f && r2a <= hi_f;
                    const bool bb = onb && r2b >= lo_f && r2b <= hi_f;
                    if (__builtin_expect(__ballot(ba || bb) != 0ull, 0)) {
                        if (ba) ha = exact(ca);
                        if (bb) hb = exact(cb);
                    }
                    ha = excluded(ha, ca);
                    hb = excluded(hb, cb);
                    const uint64_t ma = __ballot(ha), mb = __ballot(hb);
                    append(ha, ma, qa);
                    append(hb, mb, qb);
                }
                if (lane == 0) sh.rown[t] = ntot;
            }
        }
        lds_barrier();
        // ---- 6. halo numbering, rows out ------------------------------------------
        // writers: every wave but the loader
        const int wid = wv == 0 ? tid : tid - kWave;
        constexpr int kWriters = NT - kWave;
        const bool act0 = tid < kTile && r0 + tid < n_local;
        const int64_t i0 = row0 + r0 + tid;
        if (wv == 0) {
            // longest row of the tile: a wave reduction
            int n = act0 ? sh.rown[tid] : 0;
            n = wave_max_full(n < cap ? n : cap);
            if (tid == 0) sh.info[2] = n;
        }
        const int nwords = (nslot + 31) / 32;
        for (int q = tid; q < nwords; q += NT) sh.wpre[q] = __popc(sh.used[q]);
        lds_barrier();
        const int nhalo = uni(block_scan_w<NT>(sh.wpre, nwords, sh.scan));
        if (nhalo > halo_cap) {
            if (tid == 0) latch(st, 11 /*HALO_OVERFLOW*/, nhalo);
            if (act0) nn[i0] = 0;
            if (tid == 0) halo_n[tile] = 0;
            continue;
        }
        int32_t *hl = halo + (int64_t)tile * halo_cap;
        for (int q = loader ? nslot : wid; q < nslot; q += kWriters) {
            const uint32_t word = sh.used[q >> 5];
            if (word & (1u << (q & 31))) {
                const int h = sh.wpre[q >> 5] + __popc(word & ((1u << (q & 31)) - 1u));
                int32_t j;
                if (one_chunk) {
                    j = __float_as_int(sh.cp[q].w);
                } else {
                    const int u = upper_idx(sh.ustart, nu, q);
                    j = cell_idx[(int64_t)sh.ucell[u] * cell_cap + (q - sh.ustart[u])];
                }
                hl[h] = j;
            }
        }
        const int kmax = uni(sh.info[2]);
        if (tid == 0) {
            halo_n[tile] = (int32_t)((uint32_t)nhalo | ((uint32_t)kmax << 16) | (sh.info[1] ? 0x80000000u : 0u));
            // per-pair images or a halo beyond the force pass's LDS staging
            if (sh.info[1] || nhalo > halo_lds) rare_list[atomicAdd(rare_n, 1)] = tile;
        }
        uint16_t *out = nlist + nl0 + (int64_t)(r0 >> 6) * cap * kTile;
        // four entries of a thread at a time, their LDS reads issued together
        constexpr int kOut = 4;
        for (int e0 = loader ? kmax * kTile : wid; e0 < kmax * kTile; e0 += kOut * kWriters) {
            int q[kOut];
#pragma unroll
            for (int b = 0; b < kOut; ++b) {
                const int e = e0 + b * kWriters;
                const int k = e >> 6, t = e & 63;
                const int n = sh.rown[t];
                q[b] = e < kmax * kTile && k < n && k < cap ? (int)srows[t * rstride + k] : -1;
            }
#pragma unroll
            for (int b = 0; b < kOut; ++b) {
                const int e = e0 + b * kWriters;
                if (e < kmax * kTile) {
                    uint16_t v = 0;
                    if (q[b] >= 0) {
                        const uint32_t word = sh.used[q[b] >> 5];
                        v = (uint16_t)(sh.wpre[q[b] >> 5] + __popc(word & ((1u << (q[b] & 31)) - 1u)));
                    }
                    out[e] = v;
                }
            }
        }
        if (act0) {
            const int n = sh.rown[tid];
            nn[i0] = n < cap ? n : cap;
            if (n > cap) latch(st, 5 /*NLIST_OVERFLOW*/, n);
        }
    }
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------

size_t line_plan_bytes(int64_t tiles)
{
    // the carving of line_plan, with every part rounded to 256 bytes
    auto r = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t t = (size_t)(tiles > 0 ? tiles : 1);
    return r(sizeof(int4) * t) + r(sizeof(int2) * t * kUMax) + r(sizeof(float4) * t * kUMax) +
           r(sizeof(float4) * t * kTile) + r(sizeof(uint32_t) * t * kTile * kRuns) +
           r(sizeof(float) * t * kTile * kRuns);
}

static int line_dyn(int cap)
{
    return std::max(kLineBytes + kTile * nlist_row_stride(cap) * 2, (int)sizeof(GeneralShared<kChunk>));
}

hipError_t prepare_lines(int cap)
{
    auto attr = [&](auto k) {
        return hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   line_dyn(cap));
    };
    const hipError_t es[4] = {attr(&k_build_lines<false, 512>), attr(&k_build_lines<false, 256>),
                              attr(&k_build_lines<true, 512>), attr(&k_build_lines<true, 256>)};
    for (hipError_t e : es)
        if (e != hipSuccess) return e;
    return hipSuccess;
}

void launch_cells_and_lines(const LaunchCtx &L, const double4 *pos, int n_sort, int n_plan)
{
    const LinePlan plan = line_plan(L.plan, L.tiles_local);
    const dim3 grid((unsigned)(n_sort + n_plan));
    auto go = [&](auto k) {
        hipLaunchKernelGGL(k, grid, dim3(kWave), 0, L.stream, n_sort, L.sys, L.cprefix, L.n_sys, L.tprefix_local,
                           L.tiles_local, pos, L.n_cells, L.cell_count, L.cell_size, L.cell_idx, L.cell_xf, L.cell_cap,
                           L.xbuild, L.slow_list, L.slow_n, plan, L.flag, L.sflag, L.halo_n, L.halo_lds, L.rare_list,
                           L.rare_n);
    };
    if (L.cell_cap <= 64) go(k_cells_and_lines<1>);
    else go(k_cells_and_lines<2>);
}

void launch_build_lines(const LaunchCtx &L, const double4 *pos, const int32_t *tag, int block)
{
    const int blocks = capped(L.tiles_local);
    const LinePlan plan = line_plan(L.plan, L.tiles_local);
    auto go = [&](auto k, int nt) {
        hipLaunchKernelGGL(k, dim3(blocks), dim3(nt), line_dyn(L.nlist_cap), L.stream, L.sys, L.tprefix_local, L.n_sys,
                           L.tiles_local, pos, tag, L.ptag, L.cell_size, L.cell_idx, L.cell_xf, L.cell_cap,
                           cell_xf_stride(L.cell_cap), L.nlist, L.nn, L.nlist_cap, nlist_row_stride(L.nlist_cap),
                           L.halo, L.halo_n, L.halo_cap, plan, L.halo_lds, L.rare_list, L.rare_n, L.tile_ctr,
                           L.cell_count, L.n_cells, L.xbuild, L.tref, L.slow_list, L.slow_n, L.flag, L.sflag, L.build_count,
                           L.status);
    };
    if (L.has_bonds) {
        if (block == 256) go(k_build_lines<true, 256>, 256);
        else go(k_build_lines<true, 512>, 512);
    } else {
        if (block == 256) go(k_build_lines<false, 256>, 256);
        else go(k_build_lines<false, 512>, 512);
    }
}

}  // namespace md
