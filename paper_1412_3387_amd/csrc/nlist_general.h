// nlist_general.h -- the list build of a tile of any shape, run ahead of the
// framed tiles by the launches of nlist.hip and nlist_lines.hip.
#pragma once
#include "nlist_dev.h"

namespace md {

constexpr int kBuildThreads = 512;   // threads per tile of the general build's own launch
constexpr int kChunk = 2048;         // members it stages at once
constexpr int kSlotMax = 16384;      // members of a tile's stencil cells
constexpr int kKeys = 2048;          // 64 rows x 27 stencil cells, padded
constexpr int kCellBits = 1 << 17;   // cells of a system whose stencil cells are marked in a bitmap
constexpr int kStencil = 27;

// LDS of a tile of the general build; CH members staged at once (0: none, and
// the rows' first kRowStage entries put together in their place).
constexpr int kRowStage = 128;
template <int CH>
struct GeneralStage {
    double cx[CH], cy[CH], cz[CH];
    int32_t cj[CH];
};
template <>
struct GeneralStage<0> {
    uint16_t rows[kTile][kRowStage + 2];  // (the stride keeps the rows of a wave on different banks)
};
template <int CH>
struct GeneralShared {
    union {
        GeneralStage<CH> stage;
        uint32_t bits[kCellBits / 32];    // stencil cells met, where the system has few enough cells
        int32_t tmp[kKeys];               // stencil cells to sort
    };
    int32_t keys[kTile * kStencil + 1];   // distinct stencil cells, ascending
    uint16_t ustart[kTile * kStencil + 1];  // first slot of each distinct cell
    uint32_t used[kSlotMax / 32];
    uint16_t ranks[kSlotMax / 32];        // used slots before each word
    int16_t su[kTile][kStencil];          // distinct-cell index of each row's stencil cell (-1: none)
    int8_t sm[kTile][kStencil];           // image code (mx+1) + 3 (my+1) + 9 (mz+1)
    int32_t scan[kBuildThreads / kWave];
    int32_t ext[6];                       // min / max cell offset from the first row
    int32_t info[2];                      // per-pair image flag, longest row
    int32_t st[3][3];                     // the stencil's offsets
};
static_assert(kSlotMax < 65536, "slots of a tile in 16 bits");

// Index of the largest entry <= x[v] in the ascending array a[0..n), a[0] <=
// x[v], for N values at once (a step's reads are in flight together).
template <int N, typename T>
__device__ __forceinline__ void upper_many(const T *a, int n, const int (&x)[N], int (&out)[N])
{
#pragma unroll
    for (int v = 0; v < N; ++v) out[v] = 0;
    for (int step = n > 1 ? 1 << (31 - __clz(n - 1)) : 0; step > 0; step >>= 1) {
#pragma unroll
        for (int v = 0; v < N; ++v) {
            const int c = out[v] + step;
            if ((int)a[c < n ? c : 0] <= x[v] && c < n) out[v] = c;
        }
    }
}

// The general build of one tile by NT threads.  A launch has few such tiles, so
// one tile's latency bounds it.  The distinct stencil cells come out of a
// bitmap of the system's cells where it has at most kCellBits: a sort of the
// 1,728 keys is 66 passes with a barrier each and stays for larger systems.
// Rows of these tiles lie far apart and share few cells, so (CH = 0) each row
// reads its own stencil from memory rather than all rows every staged chunk
// (CH > 0, which keeps the entries of a row in the order of the chunks: the
// bits of mixed-precision DPD sums).  Sort, chunks of 2,048 and a launch of its
// own took 70 - 127 us; inside the framed launch, staged 512 at a time, that
// launch took 147 us (DPD, 100,000 particles), 265 us (64 small systems) and
// 189 us (LJ, 255,000); reading directly, in FP32 with the exact test beside
// r_list, it takes 57, 104 and 156 us.
template <bool EXCL, int NT, int CH>
__device__ __forceinline__ void general_tile(
    GeneralShared<CH> &sh, int tile, const SysDev *__restrict__ sys, const int32_t *__restrict__ tprefix, int n_sys,
    const double4 *__restrict__ pos, const int32_t *__restrict__ tag, const int32_t *__restrict__ ptag,
    const int32_t *__restrict__ cell_size, const int32_t *__restrict__ cell_idx,
    const float4 *__restrict__ cell_xf, int cell_cap,
    uint16_t *__restrict__ nlist, int32_t *__restrict__ nn, int cap, int32_t *__restrict__ halo,
    int32_t *__restrict__ halo_n, int halo_cap, double4 *__restrict__ xbuild, double4 *__restrict__ tref, int halo_lds,
    int32_t *__restrict__ rare_list, int32_t *__restrict__ rare_n, Status *st)
{
    constexpr int W = NT / kTile;
    constexpr int P = kWave / W;
    constexpr int kKpt = kKeys / NT;  // stencil keys per thread
    static_assert(kKeys % NT == 0 && kKeys <= 8 * NT, "key split");
    // (worked out anew for each tile: kept across them, what follows from it
    // would take the registers)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & (kWave - 1);
    const int w = tid >> 6;
    const int pl = lane % P;
    const int sl = lane / P;
    const int t = w * P + pl;  // particle slot in the tile
    const uint64_t seg = segment_bits(pl, P);
    const uint64_t below = lanemask_lt();

    const int s = find_sys(tprefix, n_sys, tile);
    const SysDev &S = sys[s];
    // per-system constants, held in registers for the whole tile
    const double Lx = S.L[0], Ly = S.L[1], Lz = S.L[2];
    const double iLx = S.invL[0], iLy = S.invL[1], iLz = S.invL[2];
    const int bx = S.bins[0], by = S.bins[1], bz = S.bins[2];
    const int px = S.per[0], py = S.per[1], pz = S.per[2];
    const int64_t row0 = S.row0, cell0 = S.cell0, nl0 = S.nl0;
    const int n_local = S.n_local;
    const double rl2 = S.rl2;
    const int64_t ncell = (int64_t)bx * by * bz;
    const bool marks = ncell <= kCellBits;
    const int r0 = (tile - S.tile0) * kTile;
    const int r = r0 + t;
    const bool active = r < n_local;
    const int64_t i = row0 + (active ? r : r0);
    const double4 xi = pos[i];
    int ci[3];
    ci[0] = cell_coord(xi.x, S.lo[0], S.scale[0], bx);
    ci[1] = cell_coord(xi.y, S.lo[1], S.scale[1], by);
    ci[2] = cell_coord(xi.z, S.lo[2], S.scale[2], bz);
    const double4 x0 = pos[row0 + r0];
    const int c0[3] = {cell_coord(x0.x, S.lo[0], S.scale[0], bx), cell_coord(x0.y, S.lo[1], S.scale[1], by),
                       cell_coord(x0.z, S.lo[2], S.scale[2], bz)};

    // ---- 1. distinct stencil cells of the tile -------------------------------
    // stencil k = (oz * 3 + oy) * 3 + ox over the de-duplicated offsets
    if (tid < 3) {
        sh.ext[tid] = INT32_MAX;
        sh.ext[3 + tid] = INT32_MIN;
    }
    if (tid == 0) sh.info[1] = 0;
    if (tid < 9) sh.st[tid / 3][tid % 3] = S.st[tid / 3][tid % 3];
    const int nst[3] = {S.nst[0], S.nst[1], S.nst[2]};
    const int nbits = marks ? ((int)ncell + 31) / 32 : 0;
    for (int k = tid; k < nbits; k += NT) sh.bits[k] = 0u;
    __syncthreads();
    // the key of every row's stencil cell, kept for the lookup below
    int mykeys[(kStencil + W - 1) / W];
#pragma unroll
    for (int q = 0; q < (kStencil + W - 1) / W; ++q) {
        const int k = sl + q * W;
        int key = INT32_MAX;
        int code = 0;
        if (k < kStencil) {
            const int ox = k % 3, oy = (k / 3) % 3, oz = k / 9;
            if (active && ox < nst[0] && oy < nst[1] && oz < nst[2]) {
                const int off[3] = {sh.st[0][ox], sh.st[1][oy], sh.st[2][oz]};
                const int bins[3] = {bx, by, bz};
                const int per[3] = {px, py, pz};
                int cc[3];
                bool inside = true;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    cc[a] = ci[a] + off[a];
                    int m = 0;
                    if (per[a]) {
                        // image of the neighbour cell across a periodic face
                        if (cc[a] < 0) {
                            cc[a] += bins[a];
                            m = 1;
                        } else if (cc[a] >= bins[a]) {
                            cc[a] -= bins[a];
                            m = -1;
                        }
                    } else {
                        inside = inside && cc[a] >= 0 && cc[a] < bins[a];
                    }
                    code += (m + 1) * (a == 0 ? 1 : (a == 1 ? 3 : 9));
                }
                if (inside) key = (cc[2] * by + cc[1]) * bx + cc[0];
            }
            sh.sm[t][k] = (int8_t)code;
            if (marks) {
                if (key != INT32_MAX) atomicOr(&sh.bits[key >> 5], 1u << (key & 31));
            } else {
                sh.tmp[t * kStencil + k] = key;
            }
        }
        mykeys[q] = key;
    }
    if (active && sl == 0) {
        const int bins[3] = {bx, by, bz};
        const int per[3] = {px, py, pz};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int d = ci[a] - c0[a];
            const int rel = per[a] ? wrap_rel(d, bins[a]) : d;
            atomicMin(&sh.ext[a], rel);
            atomicMax(&sh.ext[3 + a], rel);
        }
    }
    if (!marks)
        for (int k = kTile * kStencil + tid; k < kKeys; k += NT) sh.tmp[k] = INT32_MAX;
    __syncthreads();
    int nu;
    if (marks) {
        // the marked cells in order: each thread's share of the words
        const int per_thread = (nbits + NT - 1) / NT;
        const int k0 = tid * per_thread, k1 = k0 + per_thread < nbits ? k0 + per_thread : nbits;
        int c = 0;
        for (int k = k0; k < k1; ++k) c += __popc(sh.bits[k]);
        int p = block_rank<NT>(c, sh.scan, nu);
        for (int k = k0; k < k1; ++k)
            for (uint32_t m = sh.bits[k]; m; m &= m - 1u) sh.keys[p++] = 32 * k + __ffs((int)m) - 1;
    } else {
        // bitonic sort, then the first of each run of equal keys
        for (int k = 2; k <= kKeys; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int e = tid; e < kKeys / 2; e += NT) {
                    const int a = ((e & ~(j - 1)) << 1) | (e & (j - 1));
                    const int b = a | j;
                    const int32_t ka = sh.tmp[a], kb = sh.tmp[b];
                    if ((ka > kb) == ((a & k) == 0)) {
                        sh.tmp[a] = kb;
                        sh.tmp[b] = ka;
                    }
                }
                __syncthreads();
            }
        }
        int c = 0;
        for (int k = 0; k < kKpt; ++k) {
            const int q = kKpt * tid + k;
            c += sh.tmp[q] != INT32_MAX && (q == 0 || sh.tmp[q] != sh.tmp[q - 1]) ? 1 : 0;
        }
        int p = block_rank<NT>(c, sh.scan, nu);
        for (int k = 0; k < kKpt; ++k) {
            const int q = kKpt * tid + k;
            if (sh.tmp[q] != INT32_MAX && (q == 0 || sh.tmp[q] != sh.tmp[q - 1])) sh.keys[p++] = sh.tmp[q];
        }
    }
    if (tid == 0) {
        int pp = 0;
        const double Ls[3] = {Lx, Ly, Lz};
        const int bins[3] = {bx, by, bz};
        const int per[3] = {px, py, pz};
        for (int a = 0; a < 3; ++a)
            if (per[a] && (double)(sh.ext[3 + a] - sh.ext[a] + 3) * (Ls[a] / bins[a]) >= 0.5 * Ls[a]) pp = 1;
        sh.info[0] = pp;
    }
    __syncthreads();
    // member counts of the distinct cells and their prefix
    int nslot;
    {
        constexpr int kPer = (kTile * kStencil + NT - 1) / NT;
        int n[kPer], c = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int u = kPer * tid + k;
            n[k] = u < nu ? cell_size[cell0 + sh.keys[u]] : 0;
            c += n[k];
        }
        int p = block_rank<NT>(c, sh.scan, nslot);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int u = kPer * tid + k;
            if (u < nu) sh.ustart[u] = (uint16_t)(p < 65535 ? p : 65535);
            p += n[k];
        }
        if (tid == 0) sh.ustart[nu] = (uint16_t)(nslot < 65535 ? nslot : 65535);
    }
    // each row's stencil cells as distinct-cell indices
    {
        int u[(kStencil + W - 1) / W];
        upper_many(sh.keys, nu, mykeys, u);
#pragma unroll
        for (int q = 0; q < (kStencil + W - 1) / W; ++q) {
            const int k = sl + q * W;
            if (k < kStencil) sh.su[t][k] = mykeys[q] == INT32_MAX ? (int16_t)-1 : (int16_t)u[q];
        }
    }
    if (nslot > kSlotMax) {
        if (tid == 0) latch(st, 11 /*HALO_OVERFLOW*/, nslot);
        if (active && sl == 0) nn[i] = 0;
        if (tid == 0) halo_n[tile] = 0;
        __syncthreads();
        return;
    }
    for (int q = tid; q < (nslot + 31) / 32; q += NT) sh.used[q] = 0u;

    // ---- 2./3. stage chunks, scan each row's stencil --------------------------
    int32_t part[kMaxBondCap];
    if constexpr (EXCL) {
#pragma unroll
        for (int b = 0; b < kMaxBondCap; ++b) part[b] = -1;
        if (active) {
            const int64_t prow = i * S.bond_stride;
            for (int b = 0; b < S.bond_cap && b < kMaxBondCap; ++b) part[b] = ptag[prow + b];
        }
    }
    const int64_t rowbase = nl0 + (int64_t)(r >> 6) * cap * kTile + (r & 63);
    const bool fx_ = px && bx < 3, fy_ = py && by < 3, fz_ = pz && bz < 3;
    const bool few = fx_ || fy_ || fz_;
    const bool few_axis[3] = {fx_, fy_, fz_};
    // offset of the particle inside its cell and the cell widths (FP32),
    // for the conservative per-cell distance test
    const float cellw[3] = {(float)(Lx / bx), (float)(Ly / by), (float)(Lz / bz)};
    const float frel[3] = {(float)(xi.x - (S.lo[0] + ci[0] * (Lx / bx))), (float)(xi.y - (S.lo[1] + ci[1] * (Ly / by))),
                           (float)(xi.z - (S.lo[2] + ci[2] * (Lz / bz)))};
    const float rl2f = (float)rl2 * 1.0001f + 1e-3f;
    // whether a stencil cell's nearest face lies beyond r_list of the row (FP32
    // with a relative margin: it never drops a cell that can hold a neighbour)
    auto out_of_reach = [&](int k) {
        const int ox = k % 3, oy = (k / 3) % 3, oz = k / 9;
        const int offs[3] = {sh.st[0][ox < nst[0] ? ox : 0], sh.st[1][oy < nst[1] ? oy : 0],
                             sh.st[2][oz < nst[2] ? oz : 0]};
        float g2 = 0.f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (offs[a] == 0 || few_axis[a]) continue;
            const float g = offs[a] < 0 ? frel[a] : cellw[a] - frel[a];
            g2 += g > 0.f ? g * g : 0.f;
        }
        return g2 > rl2f;
    };
    int ntot = 0;
    if constexpr (CH > 0) {
        for (int q0 = 0; q0 < nslot; q0 += CH) {
            const int q1 = q0 + CH < nslot ? q0 + CH : nslot;
            __syncthreads();
            for (int q = q0 + tid; q < q1; q += NT) {
                int us[1];
                upper_many(sh.ustart, nu, {q}, us);
                const int u = us[0];
                const int32_t j = cell_idx[(cell0 + sh.keys[u]) * cell_cap + (q - sh.ustart[u])];
                const double4 xj = pos[j];
                sh.stage.cx[q - q0] = xj.x;
                sh.stage.cy[q - q0] = xj.y;
                sh.stage.cz[q - q0] = xj.z;
                sh.stage.cj[q - q0] = j;
            }
            __syncthreads();
            if (!active) continue;
            for (int k = 0; k < kStencil; ++k) {
                const int u = sh.su[t][k];
                if (u < 0) continue;
                if (out_of_reach(k)) continue;
                const int code = sh.sm[t][k];
                const double sx = Lx * (double)(code % 3 - 1);
                const double sy = Ly * (double)((code / 3) % 3 - 1);
                const double sz = Lz * (double)(code / 9 - 1);
                const bool shifted = code != 13;
                int a0 = sh.ustart[u], a1 = sh.ustart[u + 1];
                a0 = a0 > q0 ? a0 : q0;
                a1 = a1 < q1 ? a1 : q1;
                for (int k0 = a0; k0 < a1; k0 += 2 * W) {
                    bool hit[2];
                    int qq[2];
                    int32_t jj[2];
                    double ddx[2], ddy[2], ddz[2];
    #pragma unroll
                    for (int v = 0; v < 2; ++v) {
                        qq[v] = k0 + sl + v * W;
                        const int qs = (qq[v] < a1 ? qq[v] : a0) - q0;
                        jj[v] = sh.stage.cj[qs];
                        ddx[v] = sh.stage.cx[qs] - xi.x;
                        ddy[v] = sh.stage.cy[qs] - xi.y;
                        ddz[v] = sh.stage.cz[qs] - xi.z;
                    }
    #pragma unroll
                    for (int v = 0; v < 2; ++v) {
                        if (few) {
                            // fewer than 3 cells: several images share a cell, take the nearest
                            ddx[v] = fx_ ? min_image(ddx[v], Lx, iLx) : ddx[v] - sx;
                            ddy[v] = fy_ ? min_image(ddy[v], Ly, iLy) : ddy[v] - sy;
                            ddz[v] = fz_ ? min_image(ddz[v], Lz, iLz) : ddz[v] - sz;
                        } else if (shifted) {
                            ddx[v] -= sx;
                            ddy[v] -= sy;
                            ddz[v] -= sz;
                        }
                        hit[v] = qq[v] < a1 && jj[v] != (int32_t)i && norm2_exact(ddx[v], ddy[v], ddz[v]) < rl2;
                        if constexpr (EXCL) {
                            if (hit[v]) {
                                const int32_t tj = tag[jj[v]];
    #pragma unroll
                                for (int b = 0; b < kMaxBondCap; ++b) hit[v] = hit[v] && (part[b] != tj);
                            }
                        }
                    }
    #pragma unroll
                    for (int v = 0; v < 2; ++v) {
                        const uint64_t mask = __ballot(hit[v]) & seg;
                        if (hit[v]) {
                            const int p = ntot + __popcll(mask & below);
                            if (p < cap) nlist[rowbase + (int64_t)p * kTile] = (uint16_t)qq[v];
                            atomicOr(&sh.used[qq[v] >> 5], 1u << (qq[v] & 31));
                        }
                        ntot += __popcll(mask);
                    }
                }
            }
        }
    } else {
        // Rows far apart share few cells: each of a row's W lanes reads the
        // members of stencil cells of its own from the cells' FP32 copies, V
        // at a time (a batch's loads are in flight together).  The latency of
        // reads and instructions bounds it: with FP64 positions behind the row
        // numbers, two reads one after the other, a launch with 23 such tiles
        // took 93 us, now 72 (4,000 LJ particles); 16 at a time 72 and more
        // registers, the lanes of a row side by side in one cell 85.
        constexpr int V = 8;
        const int xstride = cell_xf_stride(cell_cap);
        const float Lf[3] = {(float)Lx, (float)Ly, (float)Lz}, iLf[3] = {(float)iLx, (float)iLy, (float)iLz};
        const float rlf = (float)sqrt(rl2), rl2s = (float)rl2;
        __syncthreads();
        for (int k = sl; __ballot(k < kStencil); k += W) {
            const int u = k < kStencil && !out_of_reach(k) ? sh.su[t][k] : -1;
            const int start = u < 0 ? 0 : sh.ustart[u];
            const int m = u < 0 ? 0 : sh.ustart[u + 1] - start;
            const float4 *p = cell_xf + (u < 0 ? 0 : (cell0 + sh.keys[u]) * xstride);
            // the row in the cell's frame, at the image beside the cell
            const int o[3] = {k % 3, (k / 3) % 3, k / 9};
            float xr[3], amax = 0.f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                xr[a] = frel[a] - (u < 0 ? 0.f : (float)sh.st[a][o[a]]) * cellw[a];
                amax = fmaxf(amax, fmaxf(fabsf(xr[a]), cellw[a]));
            }
            // where |x_j - x_i|^2 - r_list^2 in FP32 does not decide: with u =
            // 2^-24, each separation of a pair within about r_list is off by at
            // most eta = 4 u (row + r_list + cell), which moves r^2 by 2 sqrt(3)
            // r_list eta + 3 eta^2; its three squares, their sums and r_list^2
            // round to 6 u r^2 more.  Doubled.
            const float eta = 0x1p-22f * (amax + rlf + amax);
            const float band = 2.f * (3.4642f * rlf * eta + 3.f * eta * eta + 0x1p-21f * rl2s);
            for (int m0 = 0; __ballot(m0 < m); m0 += V) {
                float4 f[V];
#pragma unroll
                for (int v = 0; v < V; ++v) f[v] = p[m0 + v < m ? m0 + v : 0];
                uint32_t hits = 0, near = 0;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    float d[3] = {f[v].x - xr[0], f[v].y - xr[1], f[v].z - xr[2]};
                    if (few) {
                        // fewer than 3 cells: several images share a cell, take the nearest
#pragma unroll
                        for (int a = 0; a < 3; ++a)
                            if (few_axis[a]) d[a] = __builtin_fmaf(-Lf[a], rintf(d[a] * iLf[a]), d[a]);
                    }
                    const float e = __builtin_fmaf(d[0], d[0], __builtin_fmaf(d[1], d[1], d[2] * d[2])) - rl2s;
                    const bool ok = m0 + v < m && __float_as_int(f[v].w) != (int32_t)i;
                    hits |= ok && e < -band ? 1u << v : 0u;
                    near |= ok && fabsf(e) <= band ? 1u << v : 0u;
                }
                while (near) {
                    // (the minimum image: for a pair inside r_list the shift of
                    // its cell, and the nearest where a cell has several)
                    const uint32_t bit = near & (0u - near);
                    near &= near - 1u;
                    const double4 xj = pos[__float_as_int(p[m0 + __ffs((int)bit) - 1].w)];
                    double dx = xj.x - xi.x, dy = xj.y - xi.y, dz = xj.z - xi.z;
                    dx = px ? min_image(dx, Lx, iLx) : dx;
                    dy = py ? min_image(dy, Ly, iLy) : dy;
                    dz = pz ? min_image(dz, Lz, iLz) : dz;
                    hits |= norm2_exact(dx, dy, dz) < rl2 ? bit : 0u;
                }
                if constexpr (EXCL) {
                    int32_t tj[V];
#pragma unroll
                    for (int v = 0; v < V; ++v) tj[v] = tag[hits >> v & 1u ? __float_as_int(f[v].w) : (int32_t)i];
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        bool keep = true;
#pragma unroll
                        for (int b = 0; b < kMaxBondCap; ++b) keep = keep && part[b] != tj[v];
                        hits &= keep ? ~0u : ~(1u << v);
                    }
                }
                // the lanes of a row append one after the other
                int p2 = ntot;
                const int c = __popc(hits);
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    const int cq = __shfl(c, q * P + pl, kWave);
                    p2 += q < sl ? cq : 0;
                    ntot += cq;
                }
                for (; hits; hits &= hits - 1u, ++p2) {
                    const int q = start + m0 + __ffs((int)hits) - 1;
                    atomicOr(&sh.used[q >> 5], 1u << (q & 31));
                    if (p2 < kRowStage) sh.stage.rows[t][p2] = (uint16_t)q;
                    else if (p2 < cap) nlist[rowbase + (int64_t)p2 * kTile] = (uint16_t)q;
                }
            }
        }
    }
    if (active && sl == 0) atomicMax(&sh.info[1], ntot < cap ? ntot : cap);
    __syncthreads();
    // ---- 4. halo numbering and row rewrite -------------------------------------
    const int nwords = (nslot + 31) / 32;
    int nhalo;
    {
        constexpr int kPer = (kSlotMax / 32 + NT - 1) / NT;
        int n[kPer], c = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int q = kPer * tid + k;
            n[k] = q < nwords ? __popc(sh.used[q]) : 0;
            c += n[k];
        }
        int p = block_rank<NT>(c, sh.scan, nhalo);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int q = kPer * tid + k;
            if (q < nwords) sh.ranks[q] = (uint16_t)p;
            p += n[k];
        }
    }
    __syncthreads();
    if (nhalo > halo_cap) {
        if (tid == 0) latch(st, 11 /*HALO_OVERFLOW*/, nhalo);
        if (active && sl == 0) nn[i] = 0;
        if (tid == 0) halo_n[tile] = 0;
        __syncthreads();
        return;
    }
    // halo list: row number of every used member, in staging order
    int32_t *hl = halo + (int64_t)tile * halo_cap;
    for (int q0 = tid; q0 < nslot; q0 += 4 * NT) {
        int64_t at[4];
        int32_t j[4];
        int h[4], q[4], u[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) q[v] = q0 + v * NT < nslot ? q0 + v * NT : nslot - 1;
        upper_many(sh.ustart, nu, q, u);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const uint32_t word = q0 + v * NT < nslot ? sh.used[q[v] >> 5] : 0u;
            const uint32_t bit = 1u << (q[v] & 31);
            h[v] = word & bit ? sh.ranks[q[v] >> 5] + __popc(word & (bit - 1u)) : -1;
            at[v] = (cell0 + sh.keys[u[v]]) * cell_cap + (q[v] - sh.ustart[u[v]]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) j[v] = cell_idx[at[v]];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (h[v] >= 0) hl[h[v]] = j[v];
    }
    if (tid == 0) {
        tref[tile] = x0;
        halo_n[tile] = (int32_t)((uint32_t)nhalo | ((uint32_t)sh.info[1] << 16) | (sh.info[0] ? 0x80000000u : 0u));
        // per-pair images or a halo beyond the force pass's LDS staging
        if (sh.info[0] || nhalo > halo_lds) rare_list[atomicAdd(rare_n, 1)] = tile;
    }
    __threadfence_block();
    __syncthreads();
    if (active) {
        const int n = ntot < cap ? ntot : cap;
        constexpr int V = 8;
        for (int k0 = sl; k0 < n; k0 += V * W) {
            int q[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const int k = k0 + v * W;
                q[v] = 0;
                if constexpr (CH == 0) {
                    if (k < n && k < kRowStage) q[v] = sh.stage.rows[t][k];
                    else if (k < n) q[v] = nlist[rowbase + (int64_t)k * kTile];
                } else {
                    if (k < n) q[v] = nlist[rowbase + (int64_t)k * kTile];
                }
            }
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (k0 + v * W < n)
                    nlist[rowbase + (int64_t)(k0 + v * W) * kTile] =
                        (uint16_t)(sh.ranks[q[v] >> 5] + __popc(sh.used[q[v] >> 5] & ((1u << (q[v] & 31)) - 1u)));
        }
        if (sl == 0) {
            nn[i] = n;
            xbuild[i] = xi;
            if (ntot > cap) latch(st, 5 /*NLIST_OVERFLOW*/, ntot);
        }
    }
    __syncthreads();
}

}  // namespace md
