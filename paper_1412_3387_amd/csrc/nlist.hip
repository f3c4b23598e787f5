// nlist.hip -- cell list and tile-halo Verlet neighbour list (Sec. 5.1,
// Fig. 4, rebuilt for LDS-staged tiles on CDNA).
//
// Cell list: fixed-capacity bins.  A binning pass assigns every row to the
// cell floor((x - lo) * bins / L); lanes of a wave that hit the same cell
// claim their slots with one integer atomic per distinct cell.  A per-cell
// pass then sorts the members of each cell by x coordinate, ties by row
// index (rank sort inside one wave), so the list is deterministic although
// the slots were claimed in arbitrary order, and writes each member's FP32
// position from the cell's corner beside it.  The list build clears the
// counters for the next binning.
//
// Neighbour list, a tile of 64 consecutive rows (Morton ordered rows make a
// tile one or a few compact clusters) at a time:
//   * Most tiles fit one frame, unwrapped across periodic faces, and are built
//     in k_build_fast on the matrix cores (further down), from a plan of the
//     tile's cells.
//   * The others go through the general build (nlist_general.h): it sorts out
//     the distinct stencil cells of all rows (a bitmap or a sort in LDS), so
//     any tile shape works, and each row's lanes test the members of the row's
//     own 27 stencil cells.  Here they read the FP32 copies, and the FP64 test
//     on the stored positions (nearest image) decides beside r_list; beside
//     the line-ordered build of mixed-precision DPD (nlist_lines.hip) members
//     are staged and tested in FP64.
//   * Either way the list is exactly { j : |x_j - x_i|^2 < r_list^2 in FP64 }.
//     Every member that some row uses is numbered -- the tile's halo -- and
//     the rows hold 16-bit halo indices.
// The force pass then loads each halo position once per tile into LDS
// instead of once per neighbour from L2.
//
// Row layout (uint16): entry k of row r of a system lives at
// nl0 + (r / 64) * cap * 64 + k * 64 + r % 64.
// Tile header halo_n[tile]: bits 0-15 halo size, bits 16-30 the longest row
// of the tile, bit 31 set when the tile is too wide for one periodic image
// per halo entry.
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <type_traits>

#include "nlist_dev.h"
#include "nlist_general.h"

namespace md {

// ---------------------------------------------------------------------------
// binning
// ---------------------------------------------------------------------------
// Writes the list of the systems whose flag is set (a workgroup of 256).
__device__ __forceinline__ void write_flagged(int64_t *fl, int n_sys, const int32_t *__restrict__ sflag,
                                              const int32_t *__restrict__ tprefix, const int64_t *__restrict__ cprefix,
                                              int32_t *scan)
{
    const Flagged F = flagged_at(fl, n_sys);
    int64_t *cell = fl;
    int32_t *tile = const_cast<int32_t *>(F.tile), *id = const_cast<int32_t *>(F.sys);
    int nf = 0, nt = 0;
    int64_t nc = 0;
    for (int s0 = 0; s0 < n_sys; s0 += 256) {
        const int s = s0 + (int)threadIdx.x;
        const bool on = s < n_sys && sflag[s] != 0;
        int f, t, c;
        const int k = nf + block_rank<256>(on ? 1 : 0, scan, f);
        const int kt = nt + block_rank<256>(on ? tprefix[s + 1] - tprefix[s] : 0, scan, t);
        const int64_t kc = nc + block_rank<256>(on ? (int)(cprefix[s + 1] - cprefix[s]) : 0, scan, c);
        if (on) {
            id[k] = s;
            tile[k] = kt;
            cell[k] = kc;
        }
        nf += f;
        nt += t;
        nc += c;
    }
    if (threadIdx.x == 0) {
        tile[nf] = nt;
        cell[nf] = nc;
        *const_cast<int32_t *>(F.n) = nf;
    }
}
__global__ __launch_bounds__(256) void k_flagged(int64_t *fl, int n_sys, const int32_t *__restrict__ sflag,
                                                 const int32_t *__restrict__ tprefix,
                                                 const int64_t *__restrict__ cprefix)
{
    __shared__ int32_t scan[4];
    write_flagged(fl, n_sys, sflag, tprefix, cprefix, scan);
}

__global__ __launch_bounds__(256) void k_bin(const SysDev *__restrict__ sys,
                                             const int32_t *__restrict__ tprefix, int n_sys, int tiles,
                                             const double4 *__restrict__ pos,
                                             int32_t *__restrict__ cell_count,
                                             int32_t *__restrict__ cell_idx, int cell_cap,
                                             const int32_t *__restrict__ flag,
                                             const int32_t *__restrict__ sflag, Status *st,
                                             uint32_t *step_counter, int32_t *slow_n, int32_t *rare_n,
                                             int32_t *tile_ctr, int32_t *since, int since_inc,
                                             const int32_t *__restrict__ tprefix_local, int nvt_w,
                                             const double *__restrict__ khalf, double *__restrict__ thermostat,
                                             int64_t *fl, const int64_t *__restrict__ cprefix)
{
    // The Nose-Hoover update of the force launch just before (its half-step
    // partials are complete at that launch's end), folded into this launch,
    // which follows every step's force launch: a workgroup per thermostat
    // group.  The next force launch reads the new state.
    if (khalf) {
        __shared__ double red[kNvtSums];
        for (int q = blockIdx.x; q < n_sys; q += gridDim.x)
            if (sys[q].nvt_slot == q)
                nvt_group_update(sys, tprefix_local, n_sys, nvt_w, khalf, thermostat, q, red, blockDim.x, threadIdx.x);
    }
    // the binning launch follows every fused step launch: it also advances
    // the device step counter read by graph-replayed steps, and each system's
    // count of steps since its last build read by the displacement check
    if (blockIdx.x == 0) {
        if (step_counter && threadIdx.x == 0) *step_counter += 1u;
        if (since)
            for (int s = threadIdx.x; s < n_sys; s += blockDim.x) since[s] = sflag[s] ? 0 : since[s] + since_inc;
    }
    if (*flag == 0) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *slow_n = 0;
        *rare_n = 0;
    }
    // the framed build's per-die tile counters
    if (blockIdx.x == 0 && threadIdx.x < kDies) tile_ctr[threadIdx.x * kTileCtrStride] = 0;
    const int lane = lane_id();
    if (fl && n_sys > 1 && blockIdx.x == 0) {
        __shared__ int32_t scan[4];
        write_flagged(fl, n_sys, sflag, tprefix_local, cprefix, scan);
    }
    const uint64_t lt = lanemask_lt();
    const int waves = (int)(gridDim.x * blockDim.x) >> 6;
    for (int g = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6); g < tiles; g += waves) {
        const int s = find_sys(tprefix, n_sys, g);
        if (!sflag[s]) continue;  // this system keeps its list
        const SysDev &S = sys[s];
        const int r = (g - S.tile0_all) * kTile + lane;
        const bool valid = r < S.n_total;
        const int64_t i = S.row0 + r;
        int c = -1;
        if (valid) {
            const double4 x = pos[i];
            const int cx = cell_coord(x.x, S.lo[0], S.scale[0], S.bins[0]);
            const int cy = cell_coord(x.y, S.lo[1], S.scale[1], S.bins[1]);
            const int cz = cell_coord(x.z, S.lo[2], S.scale[2], S.bins[2]);
            c = (cz * S.bins[1] + cy) * S.bins[0] + cx;
        }
        // one atomic per distinct cell of the wave, all of them in flight
        // together (waited for one by one, 60 us for 2,000,000 LJ rows; 31)
        int leader = lane, rank = 0, members = 0;
        uint64_t todo = __ballot(valid);
        while (todo) {
            const int l = __ffsll((unsigned long long)todo) - 1;
            const int lc = __builtin_amdgcn_readlane(c, l);
            const uint64_t same = __ballot(c == lc);
            if (c == lc) {
                leader = l;
                rank = __popcll(same & lt);
                members = __popcll(same);
            }
            todo &= ~same;
        }
        int base = 0;
        if (valid && lane == leader) base = atomicAdd(&cell_count[S.cell0 + c], members);
        base = __shfl(base, leader, kWave);
        if (valid) {
            const int slot = base + rank;
            if (slot < cell_cap) cell_idx[(S.cell0 + c) * cell_cap + slot] = (int32_t)i;
            else latch(st, 6 /*CELL_OVERFLOW*/, slot + 1);
        }
    }
}

// ---------------------------------------------------------------------------
// tile-halo neighbour list
// ---------------------------------------------------------------------------

// The general build as a launch of its own, behind the line-ordered build in
// workgroups of 256.
template <bool EXCL>
__global__ __launch_bounds__(kBuildThreads) void k_build_tile(
    const SysDev *__restrict__ sys, const int32_t *__restrict__ tprefix, int n_sys,
    const double4 *__restrict__ pos, const int32_t *__restrict__ tag, const int32_t *__restrict__ ptag,
    const int32_t *__restrict__ cell_size, const int32_t *__restrict__ cell_idx, int cell_cap,
    uint16_t *__restrict__ nlist, int32_t *__restrict__ nn, int cap, int32_t *__restrict__ halo,
    int32_t *__restrict__ halo_n, int halo_cap, double4 *__restrict__ xbuild, double4 *__restrict__ tref,
    const int32_t *__restrict__ list, const int32_t *__restrict__ list_n, int halo_lds,
    int32_t *__restrict__ rare_list, int32_t *__restrict__ rare_n, const int32_t *__restrict__ flag, Status *st)
{
    if (*flag == 0) return;
    const int ntiles = *list_n;
    if ((int)blockIdx.x >= ntiles) return;
    __shared__ GeneralShared<kChunk> sh;
    for (int it = blockIdx.x; it < ntiles; it += gridDim.x)
        general_tile<EXCL, kBuildThreads, kChunk>(sh, list[it], sys, tprefix, n_sys, pos, tag, ptag, cell_size,
                                                  cell_idx, nullptr, cell_cap, nlist, nn, cap, halo, halo_n, halo_cap, xbuild,
                                                  tref, halo_lds, rare_list, rare_n, st);
}

// ---------------------------------------------------------------------------
// framed tile build
// ---------------------------------------------------------------------------
//
// The common case of the build above, with the distances of a whole tile
// taken on the matrix cores:
//   * The tile's cells are placed in one frame: cell coordinates relative to
//     the first row's cell, unwrapped across periodic faces, positions
//     relative to the centre of the rows' bounding box.  Cells of the frame's
//     box within r_list of the bounding box of some 16 rows are taken; where
//     the box is large, only those that some row's stencil meets (a bitmap).
//   * Members are staged as FP32 positions in the frame: the cell list keeps
//     each member's position from its cell's corner in FP32, and staging adds
//     the corner's frame position (one coalesced read per member, a segment
//     of up to 8 members of a cell per 8 lanes).  Members farther than
//     r_list from the bounding box are dropped, the others packed in order.
//   * |x_j - x_i|^2 - r_list^2 of 16 members x 16 rows is one
//     v_mfma_f32_16x16x4_f32: (x_j, |x_j|^2) against (-2 x_i, 1), accumulated
//     onto |x_i|^2 - r_list^2.  A wave takes 16 members at a time against all
//     64 rows; the sign bits of the results, shifted into one mask word per
//     lane and row, are the hits.  A result within the tile's band of zero
//     (a bound on its FP32 error) is decided by the exact FP64 test
//     (difference of the stored positions, then the periodic shift), so the
//     list is exactly the FP64 one.
//   * Two register swaps turn the masks so that lane t holds row t's words;
//     the members that some row uses (an OR over the rows) are numbered, that
//     is the tile's halo, and every row's hits are expanded into halo indices
//     in LDS and written out coalesced.
// Tiles that do not fit (a frame wider than a periodic box, fewer than three
// cells on a periodic axis, more segments than a plan holds) are appended to a
// device list and built in general, first in the same launch.

constexpr int kFastThreads = 256;    // threads per workgroup by default (4 waves)
constexpr int kFastThreadsMax = 512;
constexpr int kBoxDense = 160;       // cells of a frame box looked at without marking the stencils first
constexpr int kSegMin = 256;         // segments of a tile's plan there is always room for

// Per-tile plan of the framed build, written by k_cells_and_plan and read by
// k_build_fast: the header, the rows' frame positions and the segments of up
// to 8 members of its cells.
struct PlanTile {
    int32_t nu, nseg, pp;                // distinct cells (-1: passed on), segments, per-pair image flag
    float band;                          // accumulated values nearer zero do not decide
    float half[3], keep2;                // half widths of the rows' bounding box, bound on its distance^2
    int32_t row, nrows;                  // first row, rows
    float lo, hi;                        // FP32 differences squared below are inside, above outside
    double ref[3], pad;                  // the frame's origin
    float4 xrow[kTile];                  // row position in the frame, |x|^2 - r_list^2
    float4 seg[1];                       // corner of the cell in the frame, first member / 8 (bits) in w
};                                       // (as many as the context has room for)
constexpr int kPlanHead = 80 + 16 * kTile;
static_assert(offsetof(PlanTile, seg) == kPlanHead, "one packed block");

// Rounds of segments that k_build_fast reads ahead of those it needs, whether
// a plan has them or not: the plans are padded by as many.
constexpr int kRounds = 5;
constexpr int64_t kPlanOverRead = (int64_t)sizeof(float4) * kRounds * (kFastThreadsMax / kSeg);

// Bytes of a plan block with room for seg_cap segments.
__host__ __device__ inline int64_t plan_stride(int seg_cap) { return kPlanHead + (int64_t)sizeof(float4) * seg_cap; }

// Members staged at once, each wave's in its own part: eight of a wave's
// blocks of 16 fill a mask word of 32 bits per row and result group.  1,536
// hold the kept members of most tiles of a liquid in one pass (an LJ liquid
// at 0.8442 keeps 1,140 on average), whose rows are put together in the LDS
// of the staged positions, and leave room for four workgroups of 256 threads
// per CU.  (With 768 most tiles take two passes: 256 / 512 threads, us, 1,116
// / 2,074 against 902 / 1,384 for 2,000,000 LJ rows, 85 / 93 against 72 / 62
// for 32,000, and no faster in any context measured.  The passes decide the
// order of a row's entries, so they are the same with and without bonds.)
constexpr int kBuildChunk = 1536;
constexpr int kExSlots = 512;        // slots of a tile's partner-tag table (64 rows x 4 partners)

template <int NT>
struct FastShared {
    static constexpr int kC = kBuildChunk;
    static constexpr int kWaves = NT / kWave;
    static constexpr int kCw = kC / kWaves;              // members of a wave
    static constexpr int kWords = (kCw / 16 + 7) / 8;
    static_assert(kCw % 16 == 0 && kCw >= kWave && kCw <= 384, "whole blocks, at least a round");
    int32_t cj[kC];                      // particle rows of the staged members
    uint32_t used[kWords * kWaves * 4];  // hits of any row, per wave and result group
    uint16_t cnt[kWaves][kTile];         // hits of each row in each wave's members
    uint16_t selfq[kWaves][kTile];       // the row's own staged place, 0xFFFF: not this wave's
    int32_t left[kWaves];                // the wave has members left for another pass
    int32_t grab[3];                     // tile indices taken from the die's counter: the next of
                                         // the loop, the first two
};

// Exclusions of a tile of bonded rows: the rows' partner tags in an open-
// addressed table, and per wave the first staged places found for them (n
// counts all).
template <int NT>
struct ExShared {
    int32_t tag[kExSlots];
    uint8_t row[kExSlots];
    int32_t n[NT / kWave][kTile];
    uint16_t q[NT / kWave][kTile][2 * kMaxBondCap];
};

// x, y, z and |x|^2 of the staged members: the four components' rows start
// 16 banks apart, so that one read of 16 members' four components meets every
// bank once.
constexpr int build_astride(int kc) { return kc + 16 + (64 - kc % 64) % 64; }
template <int NT>
constexpr int kExShared = (int)((sizeof(ExShared<NT>) + 15) / 16 * 16);
template <int NT>
constexpr int kFastShared = (int)((sizeof(FastShared<NT>) + 15) / 16 * 16);


// The plan of one tile per wave (workgroups of one wave: no block barriers
// wait on other waves, so many tiles are in flight per CU).  Lane t takes
// row t: its home cell in the frame (cell coordinates relative to the first
// row's cell, unwrapped across periodic faces with the cut opposite the first
// row or, where that does not fit, through it).  Then a lane takes a cell of
// the frame's box (home cells +-1) at a time: those within r_list of the
// bounding box of some 16 rows are the tile's cells, their members its
// segments, in box order.  A large box (rows that jump, where the Morton curve
// leaves a region) holds many cells that no row's stencil meets: there the
// stencils are marked in a bitmap first.  The rows' build positions are
// written here.  Tiles that do not fit (a frame wider than a periodic box,
// fewer than three cells on a periodic axis, too many cells or members) go to
// the general build.
// Vector instructions bound it: with the cells of every tile found from the
// bitmap and a division per coordinate it took 2,250 of them per tile, and
// the launch 222 us for 2,000,000 LJ rows; now
// 174 us.
__device__ __forceinline__ void plan_tiles(
    int pb, int npb, const SysDev *__restrict__ sys, const int32_t *__restrict__ tprefix, int n_sys, int tiles,
    const double4 *__restrict__ pos, const int32_t *__restrict__ cell_count, int cell_cap,
    double4 *__restrict__ xbuild, double4 *__restrict__ tref, int32_t *__restrict__ slow_list, int32_t *__restrict__ slow_n,
    char *__restrict__ plan, int64_t stride, const int32_t *__restrict__ sflag,
    int32_t *__restrict__ halo_n, int halo_lds, int32_t *__restrict__ rare_list, int32_t *__restrict__ rare_n,
    int64_t *fl)
{
    __shared__ uint32_t box[kBoxMax / 32];
    const int lane = lane_id();
    const Flagged F = flagged_at(fl, n_sys);
    const int nf = n_sys > 1 ? *F.n : 1;
    if (n_sys > 1) {
        // a system that keeps its list: its tiles go back on the list of tiles
        // that the force pass takes first if its last build put them there
        // (the binning launch before this one emptied that list)
        for (int t0 = pb * kWave; t0 < tiles; t0 += npb * kWave) {
            const int t = t0 + lane < tiles ? t0 + lane : tiles - 1;
            const int32_t hn = halo_n[t];
            if (t == t0 + lane && !sflag[find_sys(tprefix, n_sys, t)] && (hn < 0 || (hn & 0xFFFF) > halo_lds))
                rare_list[atomicAdd(rare_n, 1)] = t;
        }
    }
    int64_t tfirst, tend;
    int tstep;
    die_range(pb, npb, n_sys > 1 ? F.tile[nf] : tiles, tfirst, tend, tstep);
    for (int x = (int)tfirst; x < tend; x += tstep) {
        int s;
        const int tile = flagged_tile(F, nf, tprefix, n_sys, x, s);
        const SysDev &S = sys[s];
        const double Ls[3] = {S.L[0], S.L[1], S.L[2]};
        const int bins[3] = {S.bins[0], S.bins[1], S.bins[2]};
        const int per[3] = {S.per[0], S.per[1], S.per[2]};
        const int64_t row0 = S.row0, cell0 = S.cell0;
        // (each system's own room, whatever the other systems of the context
        // have: it decides which build a tile gets)
        const int n_local = S.n_local, seg_cap = S.seg_cap;
        const double rl2 = S.rl2;
        const int r0 = (tile - S.tile0) * kTile;
        PlanTile *pt = reinterpret_cast<PlanTile *>(plan + tile * stride);
        // an empty plan: nu = 0 for a tile past the local rows (room for
        // particles that may arrive), -1 for one passed on
        auto empty = [&](int nu) {
            if (lane == 0) {
                pt->nu = nu;
                pt->nseg = 0;
                pt->pp = 0;
                pt->nrows = 0;
            }
        };
        if (r0 >= n_local) {
            empty(0);
            if (lane == 0) halo_n[tile] = 0;
            continue;
        }
        const double wide[3] = {Ls[0] / bins[0], Ls[1] / bins[1], Ls[2] / bins[2]};
        const float cw[3] = {(float)wide[0], (float)wide[1], (float)wide[2]};
        auto pass_on = [&]() {
            if (lane == 0) slow_list[atomicAdd(slow_n, 1)] = tile;
            empty(-1);
        };

        // ---- rows: home cell in the frame, frame position, build position ----
        const int r = r0 + lane;
        const bool act = r < n_local;
        const double4 xi = pos[row0 + (act ? r : r0)];
        if (act) xbuild[row0 + r] = make_double4(xi.x, xi.y, xi.z, 0.0);
        const double xr[3] = {uni(xi.x), uni(xi.y), uni(xi.z)};  // row 0 of the tile
        const double xa[3] = {xi.x, xi.y, xi.z};
        int c0[3], h[3], blo[3], X[3];
        double xd[3];
        float xf[3];
        bool pass = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int ci = cell_coord(xa[a], S.lo[a], S.scale[a], bins[a]);
            c0[a] = uni(ci);
            const int hd = ci - c0[a];
            // image of the row in the frame: the home cell at c0 + h
            int kimg = 0;
            if (per[a]) {
                const int sft = bins[a] / 2;
                kimg = hd >= bins[a] - sft ? -1 : (hd < -sft ? 1 : 0);
            }
            int elo = wave_min_full(act ? hd + kimg * bins[a] : INT32_MAX);
            int ehi = wave_max_full(act ? hd + kimg * bins[a] : INT32_MIN);
            if (per[a] && ehi - elo + 3 > bins[a]) {
                kimg = hd < 0 ? 1 : 0;
                elo = wave_min_full(act ? hd + kimg * bins[a] : INT32_MAX);
                ehi = wave_max_full(act ? hd + kimg * bins[a] : INT32_MIN);
            }
            h[a] = hd + kimg * bins[a];
            xd[a] = (xa[a] + (double)kimg * Ls[a]) - xr[a];
            xf[a] = (float)xd[a];
            // the frame's box
            int lo_ = elo - 1, hi_ = ehi + 1;
            if (!per[a]) {
                lo_ = lo_ > -c0[a] ? lo_ : -c0[a];
                hi_ = hi_ < bins[a] - 1 - c0[a] ? hi_ : bins[a] - 1 - c0[a];
            } else if (bins[a] < 3 || hi_ - lo_ + 1 > bins[a]) {
                pass = true;
            }
            blo[a] = lo_;
            X[a] = hi_ - lo_ + 1;
            pass = pass || (double)X[a] * wide[a] > 512.0 * sqrt(rl2);
        }
        if (pass || X[0] * X[1] * X[2] > kBoxMax) {
            pass_on();
            continue;
        }
        const int vol = X[0] * X[1] * X[2];

        // the frame's origin: the centre of the rows' bounding box (inactive
        // rows, and rows that are no numbers, find nothing); and the bounding
        // boxes of each 16 rows
        const bool found = act && fabsf(xf[0]) < 1e15f && fabsf(xf[1]) < 1e15f && fabsf(xf[2]) < 1e15f;
        const bool any = __ballot(found) != 0ull;
        float half[3], xc[3], gmid[4][3], ghalf[4][3];
        double ref[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int o = float_order(xf[a]);
            const int mnr = row_min_full(found ? o : INT32_MAX), mxr = row_max_full(found ? o : INT32_MIN);
            int mn[4], mx[4];
#pragma unroll
            for (int R = 0; R < 4; ++R) {
                mn[R] = __builtin_amdgcn_readlane(mnr, 16 * R);
                mx[R] = __builtin_amdgcn_readlane(mxr, 16 * R);
            }
            const float lo_ = any ? float_unorder(min(min(mn[0], mn[1]), min(mn[2], mn[3]))) : 0.f;
            const float hi_ = any ? float_unorder(max(max(mx[0], mx[1]), max(mx[2], mx[3]))) : 0.f;
            const float ctr = 0.5f * (lo_ + hi_);
            // (xf and its differences round: a little more than half the extent)
            half[a] = 0.5000005f * (hi_ - lo_) + 0x1p-22f * fmaxf(fabsf(lo_), fabsf(hi_));
#pragma unroll
            for (int R = 0; R < 4; ++R) {
                const bool none = mn[R] > mx[R];
                const float l = float_unorder(mn[R]), h2 = float_unorder(mx[R]);
                gmid[R][a] = none ? 0.f : 0.5f * (l + h2) - ctr;
                ghalf[R][a] = none ? -1e30f : 0.5f * (h2 - l);
            }
            ref[a] = xr[a] + (double)ctr;
            xc[a] = (float)(xd[a] - (double)ctr);
        }
        const double n2 = (double)xc[0] * xc[0] + (double)xc[1] * xc[1] + (double)xc[2] * xc[2];
        pt->xrow[lane] = found ? make_float4(xc[0], xc[1], xc[2], (float)(n2 - rl2)) : make_float4(0.f, 0.f, 0.f, 1e30f);
        // Band around zero inside which the FP32 value of |x_j - x_i|^2 -
        // r_list^2 cannot decide the test, with u = 2^-24 and the candidate
        // within about r_list of a row (farther ones come out far above it):
        // each separation is off by at most eta = 4 u (largest coordinate +
        // r_list + cell: the cell-relative position, the corner, their sum
        // and the row's position round once each), which moves r^2 by
        // 2 sqrt(3) r_list eta + 3 eta^2; |x_j|^2, the accumulator's start and
        // the four products and sums round to at most 12 u of the sum of the
        // magnitudes, (|x_i| + |x_j|)^2 + r_list^2.  Doubled.
        const float rmax = sqrtf(__int_as_float(wave_max_full(found ? __float_as_int((float)n2) : 0)));
        const float amax = fmaxf(half[0], fmaxf(half[1], half[2]));
        float band, keep2, near_lo, near_hi;
        const double rl = sqrt(rl2);
        {
            const double u = 0x1p-24;
            const double eta = 4.0 * u * ((double)amax + 1.02 * rl + (double)fmaxf(cw[0], fmaxf(cw[1], cw[2])));
            const double mag = 2.0 * rmax * 1.0001 + 1.02 * rl;
            const double moved = 2.0 * sqrt(3.0) * 1.02 * rl * eta + 3.0 * eta * eta;
            const double dr2 = moved + 12.0 * u * (mag * mag + rl2);
            band = (float)(2.0 * dr2);
            // the differences themselves, squared in FP32: moved, and five
            // more roundings of about r_list^2
            const double dd = 2.0 * (moved + 6.0 * u * rl2);
            near_lo = (float)(rl2 - dd);
            near_hi = (float)(rl2 + dd);
            // bound on the squared distance from the bounding box of anything
            // within r_list of a row
            keep2 = (float)(rl2 * 1.0001 + 1e-3 + 2.0 * dr2);
        }

        // ---- the cells within r_list of some 16 rows, their segments ----------
        // (a quotient of cell numbers by high product: exact while the product
        // of dividend and divisor stays below 2^32; kBoxMax^2 does)
        const bool marked = vol > kBoxDense;
        if (marked) {
            // a row's stencil as nine x-lines of (up to) three adjacent cells:
            // consecutive bits of one box row
            __syncthreads();  // (an earlier tile's marks are read)
            for (int q = lane; q < (vol + 31) / 32; q += kWave) box[q] = 0u;
            __syncthreads();
            if (found)
                for (int rr = 0; rr < 9; ++rr) {
                    const int fy = h[1] + rr % 3 - 1 - blo[1], fz = h[2] + rr / 3 - 1 - blo[2];
                    if (fy < 0 || fy >= X[1] || fz < 0 || fz >= X[2]) continue;  // beyond an open face
                    const int xa_ = h[0] - 1 > blo[0] ? h[0] - 1 : blo[0];
                    const int xb_ = h[0] + 1 < blo[0] + X[0] - 1 ? h[0] + 1 : blo[0] + X[0] - 1;
                    const int b = (fz * X[1] + fy) * X[0] + (xa_ - blo[0]);
                    const uint64_t bits = ((1ull << (xb_ - xa_ + 1)) - 1ull) << (b & 31);
                    atomicOr(&box[b >> 5], (uint32_t)bits);
                    if (bits >> 32) atomicOr(&box[(b >> 5) + 1], (uint32_t)(bits >> 32));
                }
            __syncthreads();
        }
        const uint32_t inv0 = 0xFFFFFFFFu / (uint32_t)X[0] + 1u, inv01 = 0xFFFFFFFFu / (uint32_t)(X[0] * X[1]) + 1u;
        const bool flat0 = X[0] == 1, flat01 = X[0] * X[1] == 1;
        const int xs = cell_xf_stride(cell_cap) / kSeg;
        int nu = 0, nseg = 0;
        for (int b0 = 0; b0 < vol; b0 += kWave) {
            const int b = b0 + lane < vol ? b0 + lane : vol - 1;
            const int fz = flat01 ? b : (int)__umulhi((uint32_t)b, inv01);
            const int t = b - fz * (X[0] * X[1]);
            const int fy = flat0 ? t : (int)__umulhi((uint32_t)t, inv0);
            const int f[3] = {t - fy * X[0] + blo[0], fy + blo[1], fz + blo[2]};
            int pc[3];
            float off[3], mid[3], wid[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                pc[a] = c0[a] + f[a];
                const int ki = pc[a] >= bins[a] ? 1 : (pc[a] < 0 ? -1 : 0);
                pc[a] -= ki * bins[a];
                // the cell's lower corner in the frame
                off[a] = (float)((S.lo[a] + (double)pc[a] * wide[a] + (double)ki * Ls[a]) - ref[a]);
                // its middle and half width; an open axis's outermost cells
                // hold whatever lies beyond them
                mid[a] = off[a] + 0.5f * cw[a];
                wid[a] = !per[a] && (pc[a] == 0 || pc[a] == bins[a] - 1) ? 1e30f : 0.501f * cw[a];
            }
            bool near = false;
#pragma unroll
            for (int R = 0; R < 4; ++R) {
                float d2 = 0.f;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float gap = fmaxf(fabsf(mid[a] - gmid[R][a]) - (ghalf[R][a] + wid[a]), 0.f);
                    d2 += gap * gap;
                }
                near = near || d2 <= keep2;
            }
            near = near && b0 + lane < vol && (!marked || ((box[b >> 5] >> (b & 31)) & 1u));
            const int64_t cell = cell0 + ((int64_t)pc[2] * bins[1] + pc[1]) * bins[0] + pc[0];
            int size = near ? cell_count[cell] : 0;
            size = size < cell_cap ? size : cell_cap;
            const int own = (size + kSeg - 1) / kSeg;
            const int incl = wave_scan_incl(own);
            const int s0 = nseg + incl - own;
            for (int q = 0; q < own; ++q)
                if (s0 + q < seg_cap)
                    pt->seg[s0 + q] = make_float4(off[0], off[1], off[2], __int_as_float((int)cell * xs + q));
            nseg += __builtin_amdgcn_readlane(incl, kWave - 1);
            nu += __popcll(__ballot(size > 0));
        }
        if (nseg > seg_cap) {
            pass_on();
            continue;
        }

        // One image per halo entry (the one nearest the centre of the rows'
        // bounding box, taken by the force pass at every step) is every row's
        // minimum image while, per periodic axis, half the box + r_list +
        // 2 r_buff < L/2: until the next build each particle moves at most
        // r_buff/2, so a row stays within half the box + r_buff/2 of the
        // centre and a listed pair within r_list + r_buff, and the partner
        // image nearest the row is within L/2 of the centre (the rows' FP32
        // offsets get a margin of 1e-5 L).  Otherwise the force pass takes the
        // minimum image per pair: around row 0 in place of the centre that
        // was 51 of the 63 tiles of a 4,000-particle LJ liquid and 1,810 of
        // 9,709 of 64 small systems.
        const double rbuff = 2.0 * sqrt(S.disp2);
        int pp = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a)
            if (per[a] && (double)half[a] + rl + 2.0 * rbuff + 1e-5 * Ls[a] >= 0.5 * Ls[a]) pp = 1;
        if (lane == 0) {
            pt->nu = nu;
            pt->nseg = nseg;
            pt->pp = pp;
            tref[tile] = make_double4(ref[0], ref[1], ref[2], 0.0);
            pt->band = band;
            pt->lo = near_lo;
            pt->hi = near_hi;
            pt->row = (int32_t)(row0 + r0);
            pt->nrows = n_local - r0 < kTile ? n_local - r0 : kTile;
            pt->keep2 = keep2;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                pt->half[a] = half[a];
                pt->ref[a] = ref[a];
            }
        }
    }
}

// The cell sort and the plans of the framed build in one launch of one-wave
// workgroups: both read only the binning results, so the first n_sort
// workgroups sort cells while the others plan tiles.
template <int CPL>
__global__ __launch_bounds__(kWave) void k_cells_and_plan(
    int n_sort, const SysDev *__restrict__ sys, const int64_t *__restrict__ cprefix, int n_sys,
    const int32_t *__restrict__ tprefix, int tiles,
    const double4 *__restrict__ pos, int64_t n_cells, const int32_t *__restrict__ cell_count,
    int32_t *__restrict__ cell_size, int32_t *__restrict__ cell_idx, float4 *__restrict__ cell_xf, int cell_cap,
    double4 *__restrict__ xbuild, double4 *__restrict__ tref, int32_t *__restrict__ slow_list, int32_t *__restrict__ slow_n,
    char *__restrict__ plan, int64_t stride, const int32_t *__restrict__ flag, const int32_t *__restrict__ sflag, int32_t *__restrict__ halo_n,
    int halo_lds, int32_t *__restrict__ rare_list, int32_t *__restrict__ rare_n, int64_t *fl)
{
    if (*flag == 0) return;
    if ((int)blockIdx.x < n_sort) {
        cell_sort_waves<CPL>(blockIdx.x, n_sort, sys, cprefix, n_sys, pos, n_cells, cell_count, cell_size, cell_idx,
                             cell_xf, cell_cap, sflag, fl);
    } else {
        plan_tiles((int)blockIdx.x - n_sort, (int)gridDim.x - n_sort, sys, tprefix, n_sys, tiles, pos,
                   cell_count, cell_cap, xbuild, tref, slow_list, slow_n, plan, stride, sflag, halo_n, halo_lds, rare_list,
                   rare_n, fl);
    }
}

// Counts back to zero for the next binning (systems without local tiles,
// whose builds have no framed scan).
__global__ void k_zero_counts(int32_t *__restrict__ cell_count, int64_t n_cells, const int32_t *__restrict__ flag)
{
    if (*flag == 0) return;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n_cells; c += (int64_t)gridDim.x * blockDim.x)
        cell_count[c] = 0;
}

typedef float v4f __attribute__((ext_vector_type(4)));

// The masks of the four row groups (16 rows each), one word per group and
// lane, turned so that lane t holds row t's words, one per result group:
// register index and group of 16 lanes change places.
__device__ __forceinline__ void turn_masks(uint32_t (&m)[4])
{
    auto p = __builtin_amdgcn_permlane32_swap(m[0], m[2], false, false);
    auto q = __builtin_amdgcn_permlane32_swap(m[1], m[3], false, false);
    auto r = __builtin_amdgcn_permlane16_swap(p[0], q[0], false, false);
    auto s = __builtin_amdgcn_permlane16_swap(p[1], q[1], false, false);
    m[0] = r[0];
    m[1] = r[1];
    m[2] = s[0];
    m[3] = s[1];
}

__device__ __forceinline__ uint32_t wave_or(uint32_t v)
{
    v |= (uint32_t)dpp_mov<0xB1>((int)v);
    v |= (uint32_t)dpp_mov<0x4E>((int)v);
    v |= (uint32_t)dpp_mov<0x141>((int)v);
    v |= (uint32_t)dpp_mov<0x140>((int)v);
    return (uint32_t)(__builtin_amdgcn_readlane((int)v, 0) | __builtin_amdgcn_readlane((int)v, 16) |
                      __builtin_amdgcn_readlane((int)v, 32) | __builtin_amdgcn_readlane((int)v, 48));
}

// Slot of a partner tag in a tile's table (kExSlots of them).
__device__ __forceinline__ uint32_t ex_slot(int32_t t) { return ((uint32_t)t * 2654435761u) >> 23; }
static_assert(kExSlots == 1 << 9, "ex_slot");

// NT threads per workgroup: its waves share a tile, each with members of its
// own, which it reads, packs and takes the distances of without waiting for
// the others; up to 1,536 / kWaves of them at a time.  The waves meet three
// times per tile: when the hits are known (halo numbering needs all of them),
// when the rows are together in LDS, and when they have been read out.
//
// Vector instructions bound it: about 9,400 per tile for an LJ liquid (1,140
// members kept, 628 of them in the halo), a fifth of them the 75 blocks of
// matrix results (30 each beside four matrix instructions), the others
// staging (45 per 64 places), the expansion of the masks and the fixed work
// of each wave; the matrix units are 13 % busy, the vector units 57 %.  LJ
// liquid of 2,000,000 rows: 0.86 ms on the sorted start, 1.02 to 1.07 in a melt
// (scan of x-cut lines, a wave per row: 1.70 ms; 17,900 instructions per
// tile).  Four waves a tile and 36 KB leave four tiles per CU; eight waves a
// tile, two per CU, took 0.5 ms more with the same code, because the fixed
// work is done twice as often and two tiles hide less of the reads' latency
// (where a tile's latency counts eight can win, 56 against 76 us for 4,000 LJ
// rows: the autotuner times both).
template <bool EXCL, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_build_fast(
    const SysDev *__restrict__ sys, const int32_t *__restrict__ tprefix, int n_sys, int tiles,
    const double4 *__restrict__ pos, const int32_t *__restrict__ tag, const int32_t *__restrict__ ptag,
    int bond_stride, const float4 *__restrict__ cell_xf,
    uint16_t *__restrict__ nlist, int32_t *__restrict__ nn, int cap, int rstride,
    int32_t *__restrict__ halo, int32_t *__restrict__ halo_n, int halo_cap, const char *__restrict__ plan,
    int64_t plan_stride, int halo_lds, int32_t *__restrict__ rare_list, int32_t *__restrict__ rare_n,
    int32_t *__restrict__ tile_ctr, int32_t *__restrict__ cell_count, int64_t n_cells,
    const int32_t *__restrict__ cell_size, const int32_t *__restrict__ cell_idx, int cell_cap,
    double4 *__restrict__ xbuild, double4 *__restrict__ tref, const int32_t *__restrict__ slow_list, const int32_t *__restrict__ slow_n,
    const int32_t *__restrict__ flag, int64_t *fl, int32_t *build_count, Status *st)
{
    if (*flag == 0) return;
    // the binning counts, read by the cell sort and the plans, back to zero
    // for the next build
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n_cells; c += (int64_t)gridDim.x * blockDim.x)
        cell_count[c] = 0;
    using Sh = FastShared<NT>;
    constexpr int kWaves = Sh::kWaves, kC = Sh::kC, kCw = Sh::kCw, kWords = Sh::kWords, kA = build_astride(kC);
    constexpr int kSegWave = kWave / kSeg;         // segments a wave stages at once
    static_assert(kWords * kWaves * 4 <= kWave, "one-wave scan of the marks");
    static_assert(NT <= kFastThreadsMax, "pad of the plans");
    // LDS: this structure and the exclusions', then the staged positions in
    // whose place (all distances taken) the rows' halo indices [kTile][rstride]
    // are put together
    extern __shared__ float4 lds_all[];
    Sh &sh = *reinterpret_cast<Sh *>(lds_all);
    using Ex = ExShared<NT>;
    Ex &ex = *reinterpret_cast<Ex *>(reinterpret_cast<char *>(lds_all) + kFastShared<NT>);
    float *const lds_a =
        reinterpret_cast<float *>(reinterpret_cast<char *>(lds_all) + kFastShared<NT> + (EXCL ? kExShared<NT> : 0));
    uint16_t *const srows = reinterpret_cast<uint16_t *>(lds_a);
    int tid = threadIdx.x;
    const int wv = uni(tid >> 6);
    if (blockIdx.x == 0 && tid == 0) atomicAdd(build_count, 1);

    // The tiles that the plan passed on, first: they take longest, and beside
    // the framed ones their time hides (as a launch of their own after these
    // they added it to most builds, and an empty launch to every step).
    for (int it = blockIdx.x; it < *slow_n; it += gridDim.x)
        general_tile<EXCL, NT, 0>(*reinterpret_cast<GeneralShared<0> *>(lds_all), slow_list[it],
                                              sys, tprefix, n_sys, pos, tag, ptag, cell_size, cell_idx, cell_xf, cell_cap,
                                              nlist, nn, cap, halo, halo_n, halo_cap, xbuild, tref, halo_lds, rare_list,
                                              rare_n, st);

    // Each die's workgroups walk one contiguous run of the rebuilt systems'
    // tiles, handed out one at a time from the die's counter (cleared by the
    // binning launch): a workgroup that meets costly tiles takes fewer, so the
    // launch ends with its run.  One lane takes the tile after next as a tile
    // starts.
    const Flagged F = flagged_at(fl, n_sys);
    const int nf = n_sys > 1 ? *F.n : 1;
    if (n_sys > 1) tiles = F.tile[nf];
    const int D = (int)gridDim.x < kDies ? (int)gridDim.x : kDies;
    const int die = (int)blockIdx.x % D;
    const int dfirst = (int)((int64_t)tiles * die / D), tend = (int)((int64_t)tiles * (die + 1) / D);
    int32_t *ctr = tile_ctr + die * kTileCtrStride;
    auto tile_of = [&](int x) {
        int s;
        return flagged_tile(F, nf, tprefix, n_sys, x, s);
    };
    int grabbed = 0;
    // (words of their own: no barrier lies between their reads here and the
    // first write of the loop's)
    if (tid == kWave) {
        sh.grab[1] = take_tile(ctr);
        sh.grab[2] = take_tile(ctr);
    }
    lds_barrier();
    int x_next = dfirst + uni(sh.grab[2]);
    int t_cur = dfirst + uni(sh.grab[1]);
    if (t_cur >= tend) return;
    t_cur = tile_of(t_cur);
    int t_next = x_next < tend ? tile_of(x_next) : t_cur;

    // a tile's plan: the header's first words, and this lane's segments of
    // kRounds rounds from r0 on (read whether they are there or not, up to
    // kPlanOverRead past the last; as many staging reads are in flight)
    float4 head[3], sg[kRounds];
    auto plan_of = [&](int t) { return reinterpret_cast<const PlanTile *>(plan + t * plan_stride); };
    auto read_segments = [&](int t, int r0) {
        const float4 *p = plan_of(t)->seg + (r0 * kWaves + wv) * kSegWave + (tid & (kWave - 1)) / kSeg;
#pragma unroll
        for (int k = 0; k < kRounds; ++k) sg[k] = p[k * kWaves * kSegWave];
    };
    auto read_head = [&](int t) {
        const float4 *p = reinterpret_cast<const float4 *>(plan_of(t));
#pragma unroll
        for (int k = 0; k < 3; ++k) head[k] = p[k];
    };
    // the partner tags of a tile's rows into its table (free slots hold -1;
    // half of the slots at most are ever taken), by one wave
    auto insert_partners = [&](int t) {
        if constexpr (EXCL) {
            if (wv != 0) return;
            for (int k = tid; k < kExSlots; k += kWave) ex.tag[k] = -1;
            const PlanTile *P = plan_of(t);
            if (tid >= P->nrows) return;
            const int64_t pr = (int64_t)(P->row + tid) * bond_stride;
            for (int b = 0; b < bond_stride; ++b) {
                const int32_t v = ptag[pr + b];
                if (v < 0) continue;
                uint32_t k = ex_slot(v);
                while (atomicCAS(&ex.tag[k], -1, v) != -1) k = (k + 1) & (kExSlots - 1);
                ex.row[k] = (uint8_t)tid;
            }
        }
    };
    read_head(t_cur);
    read_segments(t_cur, 0);
    if constexpr (EXCL) {
        insert_partners(t_cur);
        lds_barrier();
    }

    for (;;) {
        // what follows from the thread's number is worked out anew for each
        // tile: kept across the loop, its many addresses would take the
        // registers of resident waves
        asm volatile("" : "+v"(tid));
        const int lane = tid & (kWave - 1);
        const int tile = t_cur;
        const bool more = x_next < tend;
        if (tid == kWave) grabbed = take_tile(ctr);  // the tile after next
        const int nu = uni(__float_as_int(head[0].x)), nseg = uni(__float_as_int(head[0].y)),
                  pp = uni(__float_as_int(head[0].z));
        const float band = uni(head[0].w);
        const float hx = uni(head[1].x), hy = uni(head[1].y), hz = uni(head[1].z), keep2 = uni(head[1].w);
        const int rbase = uni(__float_as_int(head[2].x)), nrows = uni(__float_as_int(head[2].y));
        const int rounds = (nseg + kWaves * kSegWave - 1) / (kWaves * kSegWave);
        const int base = wv * kCw;  // this wave's staged members

        int ntot = 0;   // this lane's row: hits so far (the same in every wave)
        int hbase = 0;  // halo entries so far
        bool whole;     // one pass takes all members: the rows are put together in LDS
        int r = 0;      // rounds staged
        for (int pass = 0;; ++pass) {
            // ---- 1. stage: read, keep what is near the rows, pack ---------------
            sh.selfq[wv][lane] = 0xFFFF;
            if constexpr (EXCL) ex.n[wv][lane] = 0;
            int n = 0;
            bool full = false;
            while (r < rounds && !full) {
                if (r > 0) read_segments(tile, r);
                float4 mem[kRounds];
#pragma unroll
                for (int k = 0; k < kRounds; ++k) {
                    const bool in = ((r + k) * kWaves + wv) * kSegWave + lane / kSeg < nseg;
                    mem[k] = cell_xf[(int64_t)(in ? __float_as_int(sg[k].w) : 0) * kSeg + (lane & (kSeg - 1))];
                }
                const int r1 = r;
#pragma unroll
                for (int k = 0; k < kRounds; ++k) {
                    full = full || n + kWave > kCw;
                    if (full || r1 + k >= rounds) continue;
                    ++r;
                    const bool in = ((r1 + k) * kWaves + wv) * kSegWave + lane / kSeg < nseg;
                    const float x = mem[k].x + sg[k].x, y = mem[k].y + sg[k].y, z = mem[k].z + sg[k].z;
                    // distance from the rows' box; what is no number (a place
                    // without a member) stays so and is not kept
                    float gx = fabsf(x) - hx, gy = fabsf(y) - hy, gz = fabsf(z) - hz;
                    gx = gx <= 0.f ? 0.f : gx;
                    gy = gy <= 0.f ? 0.f : gy;
                    gz = gz <= 0.f ? 0.f : gz;
                    const bool keep = in && gx * gx + gy * gy + gz * gz <= keep2;
                    const uint64_t kb = __ballot(keep);
                    if (keep) {
                        const int q = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(kb >> 32),
                                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)kb, 0u));
                        const int32_t j = __float_as_int(mem[k].w);
                        float *w = lds_a + base + q;
                        w[0] = x;
                        w[kA] = y;
                        w[2 * kA] = z;
                        w[3 * kA] = x * x + y * y + z * z;
                        sh.cj[base + q] = j;
                        const uint32_t t = (uint32_t)(j - rbase);
                        if (t < (uint32_t)kTile) sh.selfq[wv][t] = (uint16_t)q;
                        if constexpr (EXCL) {
                            // rows that this member is a partner of
                            const int32_t tj = tag[j];
                            uint32_t h = ex_slot(tj);
                            for (int32_t v = ex.tag[h]; v != -1; v = ex.tag[h]) {
                                if (v == tj) {
                                    const int er = ex.row[h];
                                    const int slot = atomicAdd(&ex.n[wv][er], 1);
                                    if (slot < 2 * kMaxBondCap) ex.q[wv][er][slot] = (uint16_t)q;
                                }
                                h = (h + 1) & (kExSlots - 1);
                            }
                        }
                    }
                    n += __popcll(kb);
                }
            }
            // the last block's free places: far from every row
            if (lane < 16 && n + lane < ((n + 15) & ~15)) {
                float *w = lds_a + base + n + lane;
                w[0] = 0.f;
                w[kA] = 0.f;
                w[2 * kA] = 0.f;
                w[3 * kA] = 1e30f;
            }

            // ---- 2. distances, hit masks -------------------------------------------
            // the matrix operands of the rows: component lane / 16 of row
            // 16 R + lane % 16, and the accumulator's start
            int lane_ = lane;
            asm volatile("" : "+v"(lane_));  // (read anew for each pass, not kept)
            const int grp = lane_ >> 4, col = lane_ & 15;
            const float4 *xrow = plan_of(tile)->xrow;
            float bq[4];
            v4f cq[4];
#pragma unroll
            for (int R = 0; R < 4; ++R) {
                const float4 x = xrow[16 * R + col];
                bq[R] = grp == 0 ? -2.f * x.x : (grp == 1 ? -2.f * x.y : (grp == 2 ? -2.f * x.z : 1.f));
                cq[R] = v4f{x.w, x.w, x.w, x.w};
            }
            uint32_t m[kWords][4];
            uint32_t banded = 0u;  // blocks with a result in the band
            const float *ap = lds_a + grp * kA + base + col;
#pragma unroll
            for (int wd = 0; wd < kWords; ++wd) {
#pragma unroll
                for (int R = 0; R < 4; ++R) m[wd][R] = 0u;
                const int nb = (n + 15) / 16 - 8 * wd;
                if (nb <= 0) continue;
                // (each block's operand is read one block ahead)
                float an = ap[128 * wd];
#pragma unroll 1
                for (int i = 0; i < 8 && i < nb; ++i) {
                    const float av = an;
                    an = ap[128 * wd + 16 * (i < 7 ? i + 1 : 7)];
                    float mn = INFINITY;
                    v4f d[4];
#pragma unroll
                    for (int R = 0; R < 4; ++R)
                        d[R] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bq[R], cq[R], 0, 0, 0);
#pragma unroll
                    for (int R = 0; R < 4; ++R)
#pragma unroll
                        for (int r_ = 0; r_ < 4; r_ += 2)
                            mn = fminf(fminf(fabsf(d[R][r_]), fabsf(d[R][r_ + 1])), mn);
                    banded |= __ballot(mn <= band) != 0ull ? 1u << (8 * wd + i) : 0u;
#pragma unroll
                    for (int R = 0; R < 4; ++R)
#pragma unroll
                        for (int r_ = 0; r_ < 4; ++r_)
                            m[wd][R] = __builtin_amdgcn_alignbit(m[wd][R], __float_as_uint(d[R][r_]), 31);
                }
            }
            // blocks in word wd of this wave
            auto blocks = [&](int wd) -> int {
                const int nb = (n + 15) / 16 - 8 * wd;
                return nb < 8 ? nb : 8;
            };
            if (__builtin_expect(banded != 0u, 0)) {
                // the blocks with a result in the band once more: there the
                // FP32 difference decides what it can, else the FP64 test
                const PlanTile *P = plan_of(tile);
                const float lo = P->lo, hi = P->hi;
                for (; banded; banded &= banded - 1u) {
                    const int i = __ffs((int)banded) - 1;
                    const float av = ap[16 * i];
#pragma unroll
                    for (int R = 0; R < 4; ++R) {
                        const v4f d = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bq[R], cq[R], 0, 0, 0);
                        uint32_t open = 0u;
#pragma unroll
                        for (int r_ = 0; r_ < 4; ++r_) open |= fabsf(d[r_]) <= band ? 8u >> r_ : 0u;
                        if (__ballot(open != 0u) == 0ull) continue;
                        uint32_t hit = 0u;
#pragma unroll 1
                        for (uint32_t w = open; w; w &= w - 1u) {
                            const int q = 16 * i + 4 * grp + 4 - __ffs((int)w);
                            const float4 xt = xrow[16 * R + col];
                            const float *ac = lds_a + base + q;
                            const float ax = ac[0], ay = ac[kA], az = ac[2 * kA];
                            const float ex_ = ax - xt.x, ey_ = ay - xt.y, ez_ = az - xt.z;
                            const float r2 = ex_ * ex_ + ey_ * ey_ + ez_ * ez_;
                            bool in = r2 < lo;
                            if (!in && r2 <= hi) {
                                const SysDev &Q = sys[find_sys(tprefix, n_sys, tile)];
                                const double4 xa = pos[rbase + 16 * R + col], xb = pos[sh.cj[base + q]];
                                const double fj[3] = {(double)ax, (double)ay, (double)az};
                                const double fi[3] = {(double)xt.x, (double)xt.y, (double)xt.z};
                                const double pa[3] = {xa.x, xa.y, xa.z}, pb[3] = {xb.x, xb.y, xb.z};
                                double dd[3];
#pragma unroll
                                for (int c = 0; c < 3; ++c) {
                                    // frame images of both: k = round((frame - stored) / L)
                                    const double kj = rint((fj[c] + P->ref[c] - pb[c]) * Q.invL[c]);
                                    const double ki = rint((fi[c] + P->ref[c] - pa[c]) * Q.invL[c]);
                                    dd[c] = pb[c] - pa[c];
                                    if (kj != ki) dd[c] = dd[c] + (kj - ki) * Q.L[c];
                                }
                                in = norm2_exact(dd[0], dd[1], dd[2]) < Q.rl2;
                            }
                            if (in) hit |= w & (0u - w);
                        }
#pragma unroll
                        for (int wd = 0; wd < kWords; ++wd) {
                            const int sft = 4 * (blocks(wd) - 1 - (i & 7));
                            if (i >> 3 == wd) m[wd][R] = (m[wd][R] & ~(open << sft)) | (hit << sft);
                        }
                    }
                }
            }
            // word g of lane t: row t against the members 4 g + c of the
            // wave's blocks, block i result c at bit 4 (blocks - 1 - i) + 3 - c
#pragma unroll
            for (int wd = 0; wd < kWords; ++wd) turn_masks(m[wd]);
            auto drop = [&](int q) {
                const int i = q >> 4, g = (q >> 2) & 3;
#pragma unroll
                for (int wd = 0; wd < kWords; ++wd) {
                    const uint32_t bit = 1u << ((4 * (blocks(wd) - 1 - (i & 7)) + 3 - (q & 3)) & 31);
#pragma unroll
                    for (int v = 0; v < 4; ++v) m[wd][v] &= g == v && i >> 3 == wd ? ~bit : ~0u;
                }
            };
            const int sq = sh.selfq[wv][lane];
            if (sq != 0xFFFF) drop(sq);
            if constexpr (EXCL) {
                const int en = ex.n[wv][lane];
                const bool more_ex = en > 2 * kMaxBondCap;
                for (int b = 0; b < en && !more_ex; ++b) drop(ex.q[wv][lane][b]);
                if (__builtin_expect(__ballot(more_ex) != 0ull, 0)) {
                    // more copies of a row's partners than places are kept
                    // (ghosts that reach a small frame from several sides):
                    // every member's tag against the row's partners
                    const int32_t *pr = ptag + (int64_t)(rbase + (more_ex ? lane : 0)) * bond_stride;
#pragma unroll 1
                    for (int q = 0; q < n; ++q) {
                        const int32_t tj = tag[sh.cj[base + q]];
                        bool match = false;
                        for (int b = 0; b < bond_stride; ++b) match = match || (pr[b] >= 0 && pr[b] == tj);
                        if (more_ex && match) drop(q);
                    }
                }
            }
            int c = 0;
#pragma unroll
            for (int wd = 0; wd < kWords; ++wd)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    uint32_t used = 0u;
                    if (8 * 16 * wd < n) used = wave_or(m[wd][g]);
                    c += __popc(m[wd][g]);
                    if (lane == 0) sh.used[(wd * kWaves + wv) * 4 + g] = used;
                }
            sh.cnt[wv][lane] = (uint16_t)c;
            if (lane == 0) sh.left[wv] = r < rounds;
            if (tid == kWave) sh.grab[0] = grabbed;
            lds_barrier();

            // ---- 3. halo numbering, this pass's part of every row --------------------
            bool left = false;
            int p = ntot;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const int cw_ = sh.cnt[w][lane];
                p += w < wv ? cw_ : 0;
                ntot += cw_;
                left = left || sh.left[w] != 0;
            }
            left = uni((int)left) != 0;
            whole = pass == 0 && !left;
            const uint32_t uw = lane < kWords * kWaves * 4 ? sh.used[lane] : 0u;
            const int hown = __popc(uw);
            const int hi_ = wave_scan_incl(hown);
            const int hv = hbase + hi_ - hown;  // halo index before each word
            if constexpr (EXCL)
                if (!left && more) insert_partners(t_next);
            uint16_t *myrow = srows + lane * rstride;
            uint16_t *out = nlist + (int64_t)tile * cap * kTile;
            int32_t *hl = halo + (int64_t)tile * halo_cap;
#pragma unroll
            for (int wd = 0; wd < kWords; ++wd) {
                if (8 * 16 * wd >= n) continue;
                const int nb = blocks(wd);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const uint32_t used = (uint32_t)__builtin_amdgcn_readlane((int)uw, (wd * kWaves + wv) * 4 + g);
                    const int first = __builtin_amdgcn_readlane(hv, (wd * kWaves + wv) * 4 + g);
                    if (lane < 32 && ((used >> lane) & 1u)) {
                        const int h = first + __popc(used & ((1u << lane) - 1u));
                        const int q = 16 * (8 * wd + nb - 1 - (lane >> 2)) + 4 * g + 3 - (lane & 3);
                        if (h < halo_cap) hl[h] = sh.cj[base + q];
                    }
#pragma unroll 1
                    for (uint32_t w = m[wd][g]; w; w &= w - 1u) {
                        const uint32_t low = (w & (0u - w)) - 1u;
                        const uint16_t h = (uint16_t)(first + __popc(used & low));
                        // entries past the capacity land on the row's spare slot
                        if (whole) myrow[p < cap ? p : cap] = h;
                        else if (p < cap) out[p * kTile + lane] = h;
                        ++p;
                    }
                }
            }
            hbase += __builtin_amdgcn_readlane(hi_, kWave - 1);
            lds_barrier();
            if (!left) break;
        }
        if (more) {
            read_head(t_next);
            read_segments(t_next, 0);
        }

        // ---- 4. rows out --------------------------------------------------------
        if (nu >= 0) {  // (else built by the general kernel)
            const bool act = lane < nrows;
            const int n = ntot < cap ? ntot : cap;
            const int kmax = wave_max_full(act ? n : 0);
            const bool fits = hbase <= halo_cap;
            if (tid == 0) {
                halo_n[tile] = fits ? (int32_t)((uint32_t)hbase | ((uint32_t)kmax << 16) | (pp ? 0x80000000u : 0u)) : 0;
                // per-pair images or a halo beyond the force pass's LDS staging
                if (fits && (pp || hbase > halo_lds)) rare_list[atomicAdd(rare_n, 1)] = tile;
                if (!fits) latch(st, 11 /*HALO_OVERFLOW*/, hbase);
            }
            if (wv == 0 && act) {
                nn[rbase + lane] = fits ? n : 0;
                if (fits && ntot > cap) latch(st, 5 /*NLIST_OVERFLOW*/, ntot);
            }
            if (fits && whole) {
                // two rows' entries per lane, two entries of all rows per wave
                uint32_t *out = reinterpret_cast<uint32_t *>(nlist + (int64_t)tile * cap * kTile);
                const int ta = 2 * (lane & 31);
                const int na = __shfl(n, ta, kWave), nb2 = __shfl(n, ta + 1, kWave);
                const uint16_t *ra = srows + ta * rstride, *rb = ra + rstride;
                for (int k = 2 * wv + (lane >> 5); k < kmax; k += 2 * kWaves) {
                    const uint32_t va = k < na ? ra[k] : 0u, vb = k < nb2 ? rb[k] : 0u;
                    out[k * 32 + (lane & 31)] = va | (vb << 16);
                }
            }
        }
        if (!more) break;
        t_cur = t_next;
        x_next = dfirst + uni(sh.grab[0]);
        t_next = x_next < tend ? tile_of(x_next) : t_cur;
        lds_barrier();  // the rows are read, and the next index
    }
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------

void launch_bin(const LaunchCtx &L, const double4 *pos, int nvt_w)
{
    if (L.tiles_all == 0) return;
    const int blocks = capped(((int64_t)L.tiles_all * kWave + 255) / 256);
    hipLaunchKernelGGL(k_bin, dim3(blocks), dim3(256), 0, L.stream, L.sys, L.tprefix_all, L.n_sys,
                       L.tiles_all, pos, L.cell_count, L.cell_idx, L.cell_cap, L.flag, L.sflag, L.status,
                       L.step_counter, L.slow_n, L.rare_n, L.tile_ctr, L.since, L.since_inc, L.tprefix_local, nvt_w,
                       nvt_w > 0 && L.nvt ? L.khalf : nullptr, L.thermostat, L.line_rows ? nullptr : L.flagged, L.cprefix);
}

void launch_flagged(const LaunchCtx &L)
{
    if (L.n_sys > 1)
        hipLaunchKernelGGL(k_flagged, dim3(1), dim3(256), 0, L.stream, L.flagged, L.n_sys, L.sflag, L.tprefix_local,
                           L.cprefix);
}

void launch_cell_sort(const LaunchCtx &L, const double4 *pos)
{
    if (L.n_cells == 0) return;
    // one-wave workgroups: the cell sort (a multiple of the die count, so
    // that the plan workgroups keep their die mapping), then the plans
    int64_t n_sort = L.n_cells < 8192 ? L.n_cells : 8192;
    n_sort = (n_sort + kDies - 1) / kDies * kDies;
    const int n_plan = L.tiles_local < kPlanGrid ? L.tiles_local : kPlanGrid;
    if (L.line_rows) {
        launch_cells_and_lines(L, pos, (int)n_sort, n_plan);
        return;
    }
    const dim3 grid((unsigned)(n_sort + n_plan));
    if (L.cell_cap <= 64)
        hipLaunchKernelGGL(k_cells_and_plan<1>, grid, dim3(kWave), 0, L.stream, (int)n_sort, L.sys, L.cprefix, L.n_sys,
                           L.tprefix_local, L.tiles_local, pos, L.n_cells, L.cell_count, L.cell_size, L.cell_idx,
                           L.cell_xf, L.cell_cap, L.xbuild, L.tref, L.slow_list, L.slow_n, L.plan,
                           plan_stride(L.seg_cap), L.flag, L.sflag,
                           L.halo_n, L.halo_lds, L.rare_list, L.rare_n, L.flagged);
    else
        hipLaunchKernelGGL(k_cells_and_plan<2>, grid, dim3(kWave), 0, L.stream, (int)n_sort, L.sys, L.cprefix, L.n_sys,
                           L.tprefix_local, L.tiles_local, pos, L.n_cells, L.cell_count, L.cell_size, L.cell_idx,
                           L.cell_xf, L.cell_cap, L.xbuild, L.tref, L.slow_list, L.slow_n, L.plan,
                           plan_stride(L.seg_cap), L.flag, L.sflag,
                           L.halo_n, L.halo_lds, L.rare_list, L.rare_n, L.flagged);
}

int nlist_chunk() { return kWave; }
int nlist_block(bool line_rows) { return line_rows ? 512 : kFastThreads; }
bool nlist_shape_ok(int chunk, int block)
{
    return (chunk == 32 || chunk == 64) && (block == 256 || block == 512);
}

// Room for the segments of a tile's cells in its plan: 150 cells (a compact
// tile of 64 rows touches 40 to 100 once the far ones are dropped) of the
// densest occupancy to expect; tiles with more go to the general build.
int build_seg_cap(double cell_mean)
{
    const int per_cell = (int)std::ceil((cell_mean + 3.0 * std::sqrt(cell_mean)) / kSeg);
    return std::min(std::max(150 * per_cell, kSegMin), 2040);
}

size_t flagged_list_bytes(int n_sys) { return flagged_bytes(n_sys); }

size_t build_plan_bytes(int64_t tiles, int seg_cap, bool line_rows)
{
    return line_rows ? line_plan_bytes(tiles)
                     : (size_t)(tiles > 0 ? tiles : 1) * (size_t)plan_stride(seg_cap) + (size_t)kPlanOverRead;
}

int cell_xf_slots(int cell_cap) { return cell_xf_stride(cell_cap); }

// LDS of the framed launch: the shared structures, the staged positions (in
// their place the rows), or a tile of the general build.
template <bool EXCL, int NT>
static int fast_dyn(int cap)
{
    const int rows = kTile * nlist_row_stride(cap) * 2;
    const int framed = kFastShared<NT> + (EXCL ? kExShared<NT> : 0) +
                       std::max(rows, 4 * build_astride(kBuildChunk) * (int)sizeof(float));
    return std::max(framed, (int)sizeof(GeneralShared<0>));
}

template <bool EXCL, int NT>
static hipError_t fast_attr(int cap)
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&k_build_fast<EXCL, NT>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, fast_dyn<EXCL, NT>(cap));
}

hipError_t prepare_nlist(int cap)
{
    const hipError_t es[4] = {fast_attr<false, 512>(cap), fast_attr<false, 256>(cap), fast_attr<true, 512>(cap),
                              fast_attr<true, 256>(cap)};
    for (hipError_t e : es)
        if (e != hipSuccess) return e;
    return prepare_lines(cap);
}

template <bool EXCL, int NT>
static void fast_inst(const LaunchCtx &L, const double4 *pos, const int32_t *tag, int blocks, int rs)
{
    const int dyn = fast_dyn<EXCL, NT>(L.nlist_cap);
    hipLaunchKernelGGL((k_build_fast<EXCL, NT>), dim3(blocks), dim3(NT), dyn, L.stream, L.sys, L.tprefix_local,
                       L.n_sys, L.tiles_local, pos, tag, L.ptag, L.bond_stride, L.cell_xf, L.nlist, L.nn, L.nlist_cap, rs, L.halo,
                       L.halo_n, L.halo_cap, L.plan, plan_stride(L.seg_cap), L.halo_lds, L.rare_list, L.rare_n,
                       L.tile_ctr, L.cell_count, L.n_cells, L.cell_size, L.cell_idx, L.cell_cap, L.xbuild, L.tref, L.slow_list,
                       L.slow_n, L.flag, L.flagged, L.build_count, L.status);
}

// block: threads per workgroup of the framed build (512 or 256).  The
// general build's shape is fixed.
void launch_nlist(const LaunchCtx &L, const double4 *pos, const int32_t *tag, int block)
{
    if (L.tiles_local == 0) {
        // no framed scan to clear the cell counts
        if (L.n_cells > 0)
            hipLaunchKernelGGL(k_zero_counts, dim3(256), dim3(256), 0, L.stream, L.cell_count, L.n_cells, L.flag);
        return;
    }
    const int blocks = capped(L.tiles_local);
    const int rs = nlist_row_stride(L.nlist_cap);
    if (!L.line_rows) {
        if (L.has_bonds) {
            if (block == 256) fast_inst<true, 256>(L, pos, tag, blocks, rs);
            else fast_inst<true, 512>(L, pos, tag, blocks, rs);
        } else {
            if (block == 256) fast_inst<false, 256>(L, pos, tag, blocks, rs);
            else fast_inst<false, 512>(L, pos, tag, blocks, rs);
        }
        return;
    }
    launch_build_lines(L, pos, tag, block);
    if (block != 256) return;
    auto general = [&](auto k) {
        hipLaunchKernelGGL(k, dim3(blocks), dim3(kBuildThreads), 0, L.stream, L.sys, L.tprefix_local, L.n_sys, pos, tag,
                           L.ptag, L.cell_size, L.cell_idx, L.cell_cap, L.nlist, L.nn, L.nlist_cap, L.halo, L.halo_n,
                           L.halo_cap, L.xbuild, L.tref, L.slow_list, L.slow_n, L.halo_lds, L.rare_list, L.rare_n, L.flag,
                           L.status);
    };
    if (L.has_bonds) general(k_build_tile<true>);
    else general(k_build_tile<false>);
}

}  // namespace md
