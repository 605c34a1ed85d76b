// warp_fwd.hip -- fused forward augmentation kernels for gfx950.
//
// One workgroup (256 threads, 4 wave64) per output tile; each thread owns
// runs of 4 consecutive output voxels along z, so that output stores are one
// 16-byte store of intensities plus one 4-byte store of labels, and the four
// Gaussians of a run come from one Philox call.  Per voxel: the pinned FP32
// coordinate, a trilinear gather of the image and a nearest-neighbour gather
// of the labels, then gain/offset, noise, window and gamma in registers.
//
// Each sub-tile is classified once (uniformly for the workgroup) from the
// bounds of its coordinates, widened by a bound on FP32 rounding:
//   outside  -- every sample fails the (-1, n) guard: fill / label_fill only;
//   interior -- every cell floor(q)..floor(q)+1 is inside the volume: no
//               bounds checks;
//   boundary -- the footprint staged with fill outside the volume, coordinates
//               clamped to it (guard_coord).
// Footprints that fit no reservation are gathered from memory, with
// per-sample guard and per-corner fill.  All paths compute identical values
// where they overlap.
//
// Workgroup-to-tile mapping is XCD-aware (xcd_tile): consecutive workgroup
// ids are dispatched round-robin over the 8 XCDs, and tiles are dealt to the
// XCDs in chunks of consecutive tiles, so that each XCD's L2 sees spatially
// coherent runs and every XCD gets a share of every job.
#include "device_common.h"
#include "launch.h"
#include "tile_geom.h"

#include <algorithm>
#include <cmath>

namespace ctaug {

enum : int { kPathOutside, kPathLdsInterior, kPathLdsBoundary, kPathDirectInterior,
             kPathDirectBoundary };

// Sample coordinates of one thread's run, computed once by a displacement
// tile (which needs them to bound its footprint) and reused for sampling;
// already through guard_coord.
struct RunQ {
    float q[3][4];
};

// A box of output voxels and its input footprint in LDS, uniform over the
// workgroup: voxels from (x0, y0, z0) up to (x1, y1, z1) inclusive; input cell
// (i, j, k) at byte c0 + i sx + j sy + k sizeof(cell) of the LDS (modulo 2^32).
struct Box {
    int x0, y0, z0, x1, y1, z1;
    int sx, sy, c0;
};

// All runs of one box along one sampling path (uniform).  Each thread owns runs
// of 4 consecutive output voxels along z.  With a displacement (DISP) the box
// has exactly one run per thread and its coordinates come precomputed in Q.
//
// What bounds the affine warps is shared between the vector memory path (lines of
// footprint and labels fetched through L1: without the staging loads the
// 16-volume batch took 170 us of 241, without the label gathers 198, without the
// stores 198) and VALU issue (72 % of the CUs' busy cycles there, 148 instructions
// per voxel; 76 % and 133 for a 512 x 512 x 320 scan), so the per-voxel chain is
// kept short: floor and fraction are one instruction each where q >= 0
// (v_cvt_flr_i32_f32, v_fract_f32 equals q - floor(q) there), the LDS byte address
// three (24-bit multiply-adds on strides that are the job's, one origin per box),
// and the samples of a boundary box cost the same as an interior one's plus the
// clamp above (fill cells are staged).
//
// INNER: tiles of a displacement inside the volume that are gathered sample without tests
// (1.3 to 1.5 times faster on maps that shrink to a third).  That path costs a warp whose
// tiles are staged 1 %, so a single call has it only where its affine part alone
// fills the reservation (disp_cells).
template <typename T, typename LT, bool ALIGNED, int DISP, bool INNER>
__device__ __forceinline__ void run_box(JobPtr Jp, const Box &B, int path, const Tiling &SL,
                                        const uint8_t *s_lds, const RunQ &Q)
{
    const FwdJob &J = *(const FwdJob *)reload(Jp);
    const Src S = make_src<T>(J);
    gmut<float> *out = gm<float>(J.out);
    gmut<int8_t> *lout = gm<int8_t>(J.lout);
    Photo P = photo_of(J);
    const int runs_z_log = SL.lz - 2;
    const int nruns = 1 << (SL.lx + SL.ly + runs_z_log);
    const int8_t lfill = (int8_t)J.label_fill;
    const bool labels = (J.flags & kFlagLabels) != 0;

    for (int r = threadIdx.x; r < nruns; r += kThreads) {
        if (DISP != kDispNone && r != (int)threadIdx.x)
            break;
        const int zr = r & ((1 << runs_z_log) - 1);
        const int rr = r >> runs_z_log;
        const int y = B.y0 + (rr & ((1 << SL.ly) - 1));
        const int x = B.x0 + (rr >> SL.ly);
        const int z = B.z0 + 4 * zr;
        if (x > B.x1 || y > B.y1 || z > B.z1)
            continue;
        const int nvalid = ALIGNED ? 4 : min(4, J.oz - z);
        const uint32_t v0 = (uint32_t)((x * J.oy + y) * J.oz + z);
        float V[4];
        int8_t L[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            V[k] = J.fill;
            L[k] = lfill;
        }
        float q[4][3];
        if (DISP == kDispNone) {
            float rb[3];
            row_base(J.M, (float)x, (float)y, rb);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    q[k][i] = coord(J.M, i, rb, (float)(z + k));
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    q[k][i] = Q.q[i][k];
        }
        // the 8 corners of a cell whose LDS byte address is a
        auto cell = [&](int32_t ix, int32_t iy, int32_t iz, float tx, float ty, float tz) {
            int32_t a = iz * (int)sizeof(LT) + B.c0;
            a = mad_i24(iy, B.sy, a);
            a = mad_i24(ix, B.sx, a);
            const LT *c00 = reinterpret_cast<const LT *>(s_lds + a);
            const LT *c01 = reinterpret_cast<const LT *>(s_lds + (a + B.sy));
            const LT *c10 = reinterpret_cast<const LT *>(s_lds + (a + B.sx));
            const LT *c11 = reinterpret_cast<const LT *>(s_lds + (a + B.sx + B.sy));
            const float kk[8] = {(float)c00[0], (float)c00[1], (float)c01[0], (float)c01[1],
                                 (float)c10[0], (float)c10[1], (float)c11[0], (float)c11[1]};
            return tri(kk, tx, ty, tz);
        };
        // Runs past the output's end sample all four voxels where the box is interior or
        // staged: its window covers the whole box, whatever part of it the output has.
        if (path == kPathLdsInterior) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                V[k] = cell(flr_i32(q[k][0]), flr_i32(q[k][1]), flr_i32(q[k][2]),
                            __builtin_amdgcn_fractf(q[k][0]), __builtin_amdgcn_fractf(q[k][1]),
                            __builtin_amdgcn_fractf(q[k][2]));
                if (k == 1)
                    __builtin_amdgcn_sched_barrier(0);     // two voxels' corners at a time
            }
            if (labels)                // an interior box's nearest voxels are inside
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    L[k] = label_interior(S, q[k][0], q[k][1], q[k][2]);
        } else if (path == kPathLdsBoundary) {
            if (DISP == kDispNone) {
                const float nf[3] = {(float)J.nx, (float)J.ny, (float)J.nz};
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        q[k][i] = guard_coord(q[k][i], nf[i]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float fx = floorf(q[k][0]), fy = floorf(q[k][1]), fz = floorf(q[k][2]);
                V[k] = cell((int)fx, (int)fy, (int)fz, q[k][0] - fx, q[k][1] - fy, q[k][2] - fz);
                if (k & 1)
                    __builtin_amdgcn_sched_barrier(0);
            }
            if (labels)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    L[k] = label_clamped(S, q[k][0], q[k][1], q[k][2], lfill);
                    if (k == 1)
                        __builtin_amdgcn_sched_barrier(0);
                }
        } else if (INNER && path == kPathDirectInterior) {
            // the run's loads together: its voxels share lines, which would else be
            // fetched again
#pragma unroll
            for (int k = 0; k < 4; ++k)
                V[k] = sample_interior<T>(S, q[k][0], q[k][1], q[k][2]);
            if (labels)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    L[k] = label_interior(S, q[k][0], q[k][1], q[k][2]);
        } else if (path == kPathDirectBoundary) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (ALIGNED || k < nvalid) {
                    V[k] = sample_checked<T>(S, q[k][0], q[k][1], q[k][2], J.fill);
                    if (labels)
                        L[k] = label_checked(S, q[k][0], q[k][1], q[k][2], lfill);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // The flags are re-read each iteration so that the compiler tests their
        // bits in SALU where they are used instead of keeping one 64-bit lane
        // mask per flag live across the loop (scalar register pressure).
        uint32_t fl = J.flags;
        asm volatile("" : "+s"(fl));
        P.flags = fl;
        if (fl & kFlagOcclude) {
            // I_occ: the occluded output slab is 0 in place of the warped image
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float zf = (float)(z + k);
                if (zf >= J.occ_lo && zf <= J.occ_hi)
                    V[k] = 0.0f;
            }
        }

        if (P.flags & kFlagPhoto) {
            float n[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (P.flags & kFlagNoise) {
                if (ALIGNED)
                    gauss_group((uint64_t)(v0 >> 2), J.vol_id, J.key0, J.key1, n);
                else
                    gauss_run((uint64_t)v0, J.vol_id, J.key0, J.key1, n);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                V[k] = photometric(P, V[k], n[k]);
        }

        if (ALIGNED && (fl & kFlagVec)) {
            *reinterpret_cast<gmut<f32x4> *>(out + v0) = f32x4{V[0], V[1], V[2], V[3]};
            if (labels) {
                const uint32_t packed = (uint32_t)(uint8_t)L[0] | ((uint32_t)(uint8_t)L[1] << 8) |
                                        ((uint32_t)(uint8_t)L[2] << 16) |
                                        ((uint32_t)(uint8_t)L[3] << 24);
                *reinterpret_cast<gmut<uint32_t> *>(lout + v0) = packed;
            }
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < nvalid) {
                    out[v0 + k] = V[k];
                    if (labels)
                        lout[v0 + k] = L[k];
                }
        }
    }
}

// Displacement tile (ALIGNED, LT: see fwd_tile_affine).  A displacement has no
// a-priori footprint bound: the tile (one run of 4 z voxels per thread)
// computes its coordinates once, reduces their cells, and stages that
// footprint when it fits the reservation, as affine windows are (bulk loads;
// row by row with tests the 256^3 B-spline warp took 160 us, so 139).
template <typename T, typename LT, bool ALIGNED, int DISP, bool INNER>
__device__ __forceinline__ void fwd_tile_disp(JobPtr Jp, const Box &B0, const Tiling &TL,
                                              int32_t lds_cells, uint8_t *s_lds)
{
    const FwdJob &J = *(const FwdJob *)reload(Jp);
    Box B = B0;
    __shared__ __attribute__((aligned(16))) int s_red[4][8];
    const int zr = threadIdx.x & ((1 << (TL.lz - 2)) - 1);
    const int rr = threadIdx.x >> (TL.lz - 2);
    const int x = B.x0 + (rr >> TL.ly), y = B.y0 + (rr & ((1 << TL.ly) - 1)), z = B.z0 + 4 * zr;
    const bool mine = x <= B.x1 && y <= B.y1 && z <= B.z1;
    const int nvalid = min(4, J.oz - z);
    float u[3][4];
    if (DISP == kDispSpline)
        spline_tile_u(J.ctrl, J.bs, B.x0, B.y0, B.z0, B.x1, B.y1, B.z1, x, y, z, 1, nvalid, mine,
                      (int)threadIdx.x, reinterpret_cast<float *>(s_lds), u);
    const float nf[3] = {(float)J.nx, (float)J.ny, (float)J.nz};
    RunQ Q;
    int fmn[3] = {INT_MAX, INT_MAX, INT_MAX}, fmx[3] = {INT_MIN, INT_MIN, INT_MIN};
    if (mine) {
        gconst<float> *disp = gc<float>(J.disp);
        const int32_t nvox = J.ox * J.oy * J.oz;
        const int32_t v0 = (x * J.oy + y) * J.oz + z;
        float rb[3];
        row_base(J.M, (float)x, (float)y, rb);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int c = ALIGNED ? k : min(k, nvalid - 1);
            const float zf = (float)(z + k);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const float q = guard_coord(
                    coord(J.M, i, rb, zf) +
                        (DISP == kDispField ? disp[i * nvox + v0 + c] : u[i][k]),
                    nf[i]);
                // past the output's end: the last voxel's
                Q.q[i][k] = ALIGNED || k < nvalid ? q : Q.q[i][max(k, 1) - 1];
            }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const float *q = Q.q[i];
            fmn[i] = flr_i32(fminf(fminf(q[0], q[1]), fminf(q[2], q[3])));
            fmx[i] = flr_i32(fmaxf(fmaxf(q[0], q[1]), fmaxf(q[2], q[3])));
        }
    }
    block_minmax3(fmn, fmx, s_red);
    // the footprint: cells fmn .. fmx + 1 per axis, within [-2, n + 2)
    const int n[3] = {J.nx, J.ny, J.nz};
    int lo[3], e[3];
    bool outside = J.nx == 0 || J.ny == 0 || J.nz == 0, inside = true;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        lo[i] = fmn[i];
        e[i] = fmx[i] - fmn[i] + 2;
        outside = outside || lo[i] >= n[i] || lo[i] + e[i] <= 0;
        inside = inside && lo[i] >= 0 && lo[i] + e[i] <= n[i];
    }
    const int quads = (e[2] + 3) >> 2, pitch = lds_pitch(e[2]);
    const bool fits = (int64_t)e[0] * e[1] <= lds_cells && pitch <= lds_cells &&
                      e[0] * e[1] * pitch <= lds_cells && window24(lo[0], e[0]) &&
                      window24(lo[1], e[1]);
    int path = outside           ? kPathOutside
               : INNER && inside ? kPathDirectInterior
                                 : kPathDirectBoundary;
    if (!outside && fits) {
        path = inside ? kPathLdsInterior : kPathLdsBoundary;
        const Src S = make_src<T>(J);
        // whole quads inside the volume: the window of an inside tile may start earlier
        const bool whole = inside && 4 * quads <= J.nz;
        lo[2] = whole ? min(lo[2], J.nz - 4 * quads) : lo[2];
        const StageWalk W = stage_walk<kThreads>(e[0] * e[1], e[1], quads, (int)threadIdx.x);
        if (W.passes > 0 && J.nz >= 4) {
            const float g[3] = {0.0f, 0.0f, 0.0f};
            stage_window<T, LT, false>(J, S, W, lo, g, e[1], pitch, whole, s_lds);
        } else {
            TileGeom G;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                G.lo[i] = lo[i];
                G.e[i] = e[i];
            }
            G.quads = quads;
            G.pitch = pitch;
            stage_footprint<T, LT>(J, S, G, reinterpret_cast<LT *>(s_lds));
        }
        B.sy = pitch * (int)sizeof(LT);
        B.sx = e[1] * B.sy;
        B.c0 = window_origin(lo, B.sx, B.sy, (int)sizeof(LT));
        __syncthreads();
    }
    run_box<T, LT, ALIGNED, DISP, INNER>(Jp, B, path, TL, s_lds, Q);
    __syncthreads();                   // LDS is reused by the next tile
}

// Affine tile, processed as sub-tiles of the job's sub-tile shape (the whole
// tile unless its footprint would not fit the LDS reservation).  LT: type of
// the LDS footprint cells (FP32, or int16 for int16 inputs).  ALIGNED: the
// output z extent is a multiple of 4, so every run is one noise group and (with
// 16-byte aligned outputs) one vector store.
//
// What a sub-tile costs besides its samples is kept small: the extents of its
// footprint are the job's (from the host), only its origin is computed (all
// sub-tiles at once, one per lane), and all loads of a footprint are in flight
// at once.
template <typename T, typename LT, bool ALIGNED>
__device__ __forceinline__ void fwd_tile_affine(JobPtr Jp, const Box &B0, const Tiling &TL,
                                                uint8_t *s_lds)
{
    const RunQ Q0{};
    int cls = kOutside, lo[3] = {0, 0, 0};
    float g[3] = {0.0f, 0.0f, 0.0f};
    StageWalk W;
    uint32_t todo;
    bool fast = false;
    {
        const FwdJob &J = *(const FwdJob *)reload(Jp);
        const Tiling SL = {J.sub[0], J.sub[1], J.sub[2]};
        const int e[3] = {J.box_e[0], J.box_e[1], J.box_e[2]};
        const int quads = (e[2] + 3) >> 2;
        // sub-tile i in lane i of each wave: its class and the window's first cell
        const int nz_log = TL.lz - SL.lz, ny_log = TL.ly - SL.ly, nx_log = TL.lx - SL.lx;
        const int lane = threadIdx.x & 63;
        const int bx = B0.x0 + ((lane >> (nz_log + ny_log)) << SL.lx);
        const int by = B0.y0 + (((lane >> nz_log) & ((1 << ny_log) - 1)) << SL.ly);
        const int bz = B0.z0 + ((lane & ((1 << nz_log) - 1)) << SL.lz);
        // A tile that is gathered (set_gather) is classed by voxels that the output has: one
        // that reaches past the end by the last whole tile before it.
        const bool gathers = e[0] == 0;
        const int cx = gathers ? min(bx, max(J.ox - (1 << SL.lx), 0)) : bx;
        const int cy = gathers ? min(by, max(J.oy - (1 << SL.ly), 0)) : by;
        const int cz = gathers ? min(bz, max(((J.oz - 1) | 3) - (1 << SL.lz) + 1, 0)) : bz;
        cls = box_window(J, (float)cx, (float)cy, (float)cz, lo, g);
        const int nsub = 1 << (nx_log + ny_log + nz_log);  // at most 32
        todo = (uint32_t)__ballot(lane < nsub && bx <= B0.x1 && by <= B0.y1 && bz <= B0.z1);
        W.passes = 0;
        if (e[0] != 0 && __any(cls != kOutside)) {
            W = stage_walk<kThreads>(e[0] * e[1], e[1], quads, (int)threadIdx.x);
            fast = W.passes > 0 && J.nz >= 4;
        }
    }
    bool used = false;                                     // LDS read by a sub-tile
    while (todo) {
        const int i = __builtin_ctz(todo);
        todo &= todo - 1;
        const int c = __builtin_amdgcn_readlane(cls, i);
        int path = c == kOutside ? kPathOutside
                                 : c == kInterior ? kPathDirectInterior : kPathDirectBoundary;
        Box B;
        const FwdJob &J = *(const FwdJob *)reload(Jp);
        const Tiling SL = {J.sub[0], J.sub[1], J.sub[2]};
        const int nz_log = TL.lz - SL.lz, ny_log = TL.ly - SL.ly;
        B.x0 = B0.x0 + ((i >> (nz_log + ny_log)) << SL.lx);
        B.y0 = B0.y0 + (((i >> nz_log) & ((1 << ny_log) - 1)) << SL.ly);
        B.z0 = B0.z0 + ((i & ((1 << nz_log) - 1)) << SL.lz);
        B.x1 = min(B.x0 + (1 << SL.lx) - 1, B0.x1);
        B.y1 = min(B.y0 + (1 << SL.ly) - 1, B0.y1);
        B.z1 = min(B.z0 + (1 << SL.lz) - 1, B0.z1);
        B.sx = B.sy = B.c0 = 0;
        if (c != kOutside && J.box_e[0] != 0 && (sizeof(LT) == 4 || (J.flags & kFlagFillInT))) {
            path = c == kInterior ? kPathLdsInterior : kPathLdsBoundary;
            const Src S = make_src<T>(J);
            const int e1 = J.box_e[1], pitch = J.box_pitch;
            const int l[3] = {__builtin_amdgcn_readlane(lo[0], i),
                              __builtin_amdgcn_readlane(lo[1], i),
                              __builtin_amdgcn_readlane(lo[2], i)};
            B.sy = pitch * (int)sizeof(LT);
            B.sx = e1 * B.sy;
            B.c0 = window_origin(l, B.sx, B.sy, (int)sizeof(LT));
            if (used)
                __syncthreads();       // the last sub-tile has been sampled
            if (fast) {
                const float gi[3] = {
                    __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g[0]), i)),
                    __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g[1]), i)),
                    __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g[2]), i))};
                stage_window<T, LT, true>(J, S, W, l, gi, e1, pitch, c == kInterior, s_lds);
            } else {
                TileGeom G;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    G.lo[a] = l[a];
                    G.e[a] = J.box_e[a];
                }
                G.quads = (G.e[2] + 3) >> 2;
                G.pitch = pitch;
                stage_footprint<T, LT>(J, S, G, reinterpret_cast<LT *>(s_lds));
            }
            __syncthreads();
            used = true;
        }
        run_box<T, LT, ALIGNED, kDispNone, true>(Jp, B, path, SL, s_lds, Q0);
    }
    if (used)
        __syncthreads();               // LDS is reused by the next tile
}

// One output tile t of job J.
template <typename T, typename LT, bool ALIGNED, int DISP, bool INNER = true>
__device__ __forceinline__ void fwd_tile_lt(JobPtr Jp, int t, const Tiling &TL,
                                            int32_t lds_cells, uint8_t *s_lds)
{
    const FwdJob &J = *(const FwdJob *)reload(Jp);
    const int rest = (int)div_rcp((uint32_t)t, (uint32_t)J.tiles_z, J.rcp_tz);
    const int tz = t - rest * J.tiles_z;
    const int tx = (int)div_rcp((uint32_t)rest, (uint32_t)J.tiles_y, J.rcp_ty);
    const int ty = rest - tx * J.tiles_y;
    Box B;
    B.x0 = tx << TL.lx;
    B.y0 = ty << TL.ly;
    B.z0 = tz << TL.lz;
    B.x1 = min(B.x0 + (1 << TL.lx), J.ox) - 1;
    B.y1 = min(B.y0 + (1 << TL.ly), J.oy) - 1;
    B.z1 = min(B.z0 + (1 << TL.lz), J.oz) - 1;
    B.sx = B.sy = B.c0 = 0;
    if constexpr (DISP != kDispNone)
        fwd_tile_disp<T, LT, ALIGNED, DISP, INNER>(Jp, B, TL, lds_cells, s_lds);
    else
        fwd_tile_affine<T, LT, ALIGNED>(Jp, B, TL, s_lds);
}

template <typename T, bool ALIGNED, int DISP>
__device__ __forceinline__ void fwd_tile(JobPtr Jp, int t, const Tiling &TL, int32_t lds_cells,
                                         uint8_t *s_lds)
{
    if (sizeof(T) == 2 && (Jp->flags & kFlagLds16))
        fwd_tile_lt<T, T, ALIGNED, DISP>(Jp, t, TL, lds_cells, s_lds);
    else
        fwd_tile_lt<T, float, ALIGNED, DISP>(Jp, t, TL, lds_cells, s_lds);
}

// Dynamic LDS: lds_cells input-type cells of image footprint (rounded up to
// 16 bytes); labels are gathered from global memory.
extern __shared__ __attribute__((aligned(16))) uint8_t s_footprint[];

// Single job, job in kernel arguments, one workgroup per tile.
template <typename T, bool ALIGNED, int DISP, bool INNER>
__global__ __launch_bounds__(kThreads) void k_warp_single(FwdJob J, Tiling TL, int32_t ntiles,
                                                          int32_t lds_cells)
{
    const int b = blockIdx.x;
    const int t = xcd_tile(b & 7, b >> 3);
    if (t >= ntiles)
        return;
    // J is the first kernel argument (a single call's footprints are FP32 cells)
    fwd_tile_lt<T, float, ALIGNED, DISP, INNER>((JobPtr)__builtin_amdgcn_kernarg_segment_ptr(), t,
                                                TL, lds_cells, s_footprint);
}

// Index of the job holding global tile t: the number of i in [1, njobs) with
// prefix[i] <= t (the prefix is nondecreasing), 64 entries per step with one
// vector load and a ballot, so that a workgroup finds its job in one memory
// round trip (for up to 64 jobs) rather than one per job passed over.  The
// count is the same on every lane; it is returned as a scalar.
__device__ __forceinline__ int job_of(const int32_t *__restrict__ prefix, int njobs, int t)
{
    int j = 0;
    const int lane = threadIdx.x & 63;
    for (int base = 1; base < njobs; base += 64) {
        const int i = base + lane;
        const bool le = i < njobs && prefix[i] <= t;
        j += __popcll(__ballot(le));
    }
    return __builtin_amdgcn_readfirstlane(j);
}

// Batch of jobs from a device table.  prefix[j] = first global tile of job j,
// prefix[njobs] = total.  Workgroups stride over the tiles of their XCD
// (xcd_tile): one tile each, or several when a tuning asks for a few workgroups per CU.  MODE fixes
// the input and LDS cell types when every job shares them (fewer code paths
// in the kernel, less register pressure); kBatchMixed dispatches per job.
template <bool ALIGNED, int MODE>
__global__ __launch_bounds__(kThreads) void k_warp_batch(const FwdJob *__restrict__ jobs,
                                                         const int32_t *__restrict__ prefix,
                                                         int32_t njobs, Tiling TL,
                                                         int32_t lds_cells)
{
    const int total = prefix[njobs];
    const int b = blockIdx.x;
    const int per_xcd_wg = gridDim.x >> 3;
    const int xcd = b & 7;
    for (int i = b >> 3;; i += per_xcd_wg) {
        const int t = xcd_tile(xcd, i);
        if (t >= total)
            break;
        const int j = job_of(prefix, njobs, t);
        const JobPtr J = (JobPtr)(jobs + j);
        const int lt = t - prefix[j];
        if constexpr (MODE == kBatchSplineI16) {
            fwd_tile_lt<int16_t, float, ALIGNED, kDispSpline>(J, lt, TL, lds_cells, s_footprint);
        } else if constexpr (MODE == kBatchSplineF32) {
            fwd_tile_lt<float, float, ALIGNED, kDispSpline>(J, lt, TL, lds_cells, s_footprint);
        } else if constexpr (MODE == kBatchSplineMixed) {
            if (J->dtype == kI16)
                fwd_tile_lt<int16_t, float, ALIGNED, kDispSpline>(J, lt, TL, lds_cells, s_footprint);
            else
                fwd_tile_lt<float, float, ALIGNED, kDispSpline>(J, lt, TL, lds_cells, s_footprint);
        } else if constexpr (MODE == kBatchI16F32) {
            fwd_tile_lt<int16_t, float, ALIGNED, kDispNone>(J, lt, TL, lds_cells, s_footprint);
        } else if constexpr (MODE == kBatchI16I16) {
            fwd_tile_lt<int16_t, int16_t, ALIGNED, kDispNone>(J, lt, TL, lds_cells, s_footprint);
        } else if constexpr (MODE == kBatchF32) {
            fwd_tile_lt<float, float, ALIGNED, kDispNone>(J, lt, TL, lds_cells, s_footprint);
        } else {
            if (J->dtype == kI16)
                fwd_tile<int16_t, ALIGNED, kDispNone>(J, lt, TL, lds_cells, s_footprint);
            else
                fwd_tile<float, ALIGNED, kDispNone>(J, lt, TL, lds_cells, s_footprint);
        }
    }
}

// Range (dn, up) of coordinate i over a box of t voxels about its first voxel's coordinate.
static void coord_range(const FwdJob &J, const int (&t)[3], int i, double &dn, double &up)
{
    dn = -(double)J.delta[i];
    up = (double)J.delta[i];
    for (int j = 0; j < 3; ++j) {
        const double d = (double)J.M[4 * i + j] * (double)(t[j] - 1);
        (d < 0.0 ? dn : up) += d;
    }
}

// The footprint window of sub-tile shape S of job J: the range (dn, up) of axis i about
// its first voxel's coordinate, its cells e[i], and the LDS cells of the whole.  The window
// of axis i holds the cells floor(l) .. floor(h) + 1 of any coordinate range [l, h] of width
// at most span (delta on either side included): floor(span) + 3, and no more than the n + 4
// cells [-2, n + 2) that clamped coordinates reach.
static int32_t window_cells(const FwdJob &J, const Tiling &S, double (&dn)[3], double (&up)[3],
                            int32_t (&e)[3])
{
    const int t[3] = {1 << S.lx, 1 << S.ly, 1 << S.lz};
    const int n[3] = {J.nx, J.ny, J.nz};
    int64_t cells = 1;
    for (int i = 0; i < 3; ++i) {
        coord_range(J, t, i, dn[i], up[i]);
        e[i] = (int32_t)std::min({std::floor(up[i] - dn[i]) + 3.0, (double)n[i] + 4.0, 0x1p30});
        cells = std::min<int64_t>(cells * (i == 2 ? lds_pitch(e[2]) : e[i]), (int64_t)1 << 30);
    }
    return (int32_t)cells;
}

// LDS cells that hold the window of any tile of job J.
int32_t footprint_cells_bound(const FwdJob &J, const Tiling &TL)
{
    double dn[3], up[3];
    int32_t e[3];
    return window_cells(J, TL, dn, up, e);
}

// The window of sub-tile shape S into FwdJob::box_*; its LDS cells.
static int32_t set_box(FwdJob &J, const Tiling &S)
{
    double dn[3], up[3];
    const int32_t cells = window_cells(J, S, dn, up, J.box_e);
    for (int i = 0; i < 3; ++i) {
        J.box_dn[i] = (float)dn[i];
        J.box_up[i] = (float)up[i];
    }
    J.box_pitch = lds_pitch(J.box_e[2]);
    return cells;
}

// Tiles TL that are gathered from memory: no window, and the range of coordinates over no
// more voxels than the output has (whole runs of 4 along z), as tiles inside the volume
// gather without tests.  With the padding counted, the tiles of thin outputs were none of
// these (200 x 200 x 12 voxels of a 512 x 512 x 160 int16 scan, tiles of 16 along z: 38 us,
// 16 without it; 130 x 130 x 48 of 400 x 400 x 300, its last tile half full: 24 and 15).
static void set_gather(FwdJob &J, const Tiling &TL)
{
    const int t[3] = {std::min(1 << TL.lx, std::max(J.ox, 1)),
                      std::min(1 << TL.ly, std::max(J.oy, 1)),
                      std::min((1 << TL.lz) - 1, std::max(J.oz - 1, 0) | 3) + 1};
    for (int i = 0; i < 3; ++i) {
        double dn, up;
        coord_range(J, t, i, dn, up);
        J.box_dn[i] = (float)dn;
        J.box_up[i] = (float)up;
        J.box_e[i] = 0;
    }
    J.box_pitch = 0;
}

// Which quads of the window the samples of sub-tile shape S can use
// (FwdJob::inv, reach): a sample p of the box uses cell c when q(p) = A p + b
// lies in (c - 1, c + 1) per axis, a quad c .. c + 3 along z when it lies in (c -
// 1, c + 4); so p lies in A^-1 of that block, along output axis k within sum_j
// |A^-1_kj| r_j of its centre (r = 1, 1, 2.5).  The slack takes the rounding of
// q and of the kernel's FP32 test: with |A^-1| <= 8 and windows of at most 30704 cells,
// no axis longer than 3412 of them, its terms stay under 2^14, and five roundings of
// them under 2^-7; other maps copy every quad.
static void set_reach(FwdJob &J, const Tiling &S)
{
    const int t[3] = {1 << S.lx, 1 << S.ly, 1 << S.lz};
    double a[3][3], c[3][3], inv[3][3];
    for (int i = 0; i < 3; ++i) {
        J.box_mid[i] = 0.0f;
        double mid = 0.0;
        for (int j = 0; j < 3; ++j) {
            a[i][j] = (double)J.M[4 * i + j];
            mid += a[i][j] * 0.5 * (double)(t[j] - 1);
        }
        J.box_mid[i] = (float)mid;
    }
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            const int i1 = (i + 1) % 3, i2 = (i + 2) % 3, j1 = (j + 1) % 3, j2 = (j + 2) % 3;
            c[i][j] = a[i1][j1] * a[i2][j2] - a[i1][j2] * a[i2][j1];
        }
    const double det = a[0][0] * c[0][0] + a[0][1] * c[0][1] + a[0][2] * c[0][2];
    bool ok = std::isfinite(det) && det != 0.0;
    for (int k = 0; k < 3 && ok; ++k)
        for (int j = 0; j < 3; ++j) {
            inv[k][j] = c[j][k] / det;
            ok = ok && std::fabs(inv[k][j]) <= 8.0;
        }
    for (int k = 0; k < 3; ++k) {
        double m = 0.5 * (double)(t[k] - 1) + 0.02;
        for (int j = 0; j < 3; ++j) {
            J.inv[3 * k + j] = ok ? (float)inv[k][j] : 0.0f;
            if (ok)
                m += std::fabs(inv[k][j]) * ((j == 2 ? 2.5 : 1.0) + 2.0 * (double)J.delta[j]);
        }
        J.reach[k] = (float)m;
    }
}

// Whether cell indices and coordinates of J stay where the LDS paths compute
// them exactly: 24-bit cell indices and coordinates that FP32 resolves to
// fractions (delta is 2^-20 of their bound).
static bool box_exact(const FwdJob &J)
{
    for (int i = 0; i < 3; ++i)
        if (!(J.delta[i] < 4.0f))
            return false;
    return J.nx < (1 << 22) && J.ny < (1 << 22) && J.nz < (1 << 22);
}

bool keeps_rows(const FwdJob &J)
{
    return 31.0 * (std::fabs((double)J.M[2]) + std::fabs((double)J.M[6])) < 0.25;
}

// Whether the windows (set in J) of sub-tiles S of tiles TL are worth staging.  A voxel
// reads 8 cells, so a window of many cells per voxel costs more than it shares.  Where z
// runs keep to an input row (keeps_rows), gathers read whole lines, and win from 10 cells
// per voxel on (512 x 512 x 320 int16 to 256 x 256 x 160: 81 us staged, 42 gathered; FP32 95 and 73; at 8
// cells and a factor of 1.8 they take 0.9 to 1.2 times as long); and always where only
// sub-tiles of 4 voxels along z fit (400 x 400 x 300 to 160 x 160 x 120 turned by 1 degree:
// int16 89 and 45 us, FP32 136 and 63).
static bool staging_pays(const FwdJob &J, const Tiling &S, const Tiling &TL)
{
    const double cells = (double)J.box_e[0] * J.box_e[1] * J.box_pitch;
    const double voxels = (double)(1 << (S.lx + S.ly + S.lz));
    const bool flat = S.lz == 2 && TL.lz > 2 && J.oz > 4;
    return !(keeps_rows(J) && cells >= 10.0 * voxels) && !flat;
}

int32_t set_window(FwdJob &J, const Tiling &S)
{
    const int32_t cells = set_box(J, S);
    set_reach(J, S);
    if (!box_exact(J))
        J.box_e[0] = 0;
    return cells;
}

// Sub-tile shape of job J for tile TL and an LDS reservation of lds_cells
// cells (into J.sub and J.box_*): the whole tile when its window fits;
// otherwise the sub-box of the tile with the most voxels (at least 2^9, or
// the tile's own count if smaller; z extent >= 4) whose window fits, fewest
// cells per voxel among equals; the whole tile and no window (direct gathers,
// 2.4 times slower on a 512 x 512 x 320 scan) when none fits or staging it
// does not pay: false.  As tiles hold at most 2^14 voxels, a tile has at most
// 32 sub-tiles (the kernels compute one sub-tile's geometry per lane of a wave).
bool choose_subtile(FwdJob &J, const Tiling &TL, int32_t lds_cells)
{
    bool fits = true;
    Tiling best = TL;
    if (!J.disp && !J.ctrl) {
        fits = lds_cells > 0 && box_exact(J);
        if (fits && set_box(J, TL) > lds_cells) {
            const int min_log = std::min(9, TL.lx + TL.ly + TL.lz);
            int best_log = -1;
            double best_ratio = 0.0;
            for (int a = 0; a <= TL.lx; ++a)
                for (int b = 0; b <= TL.ly; ++b)
                    for (int c = 2; c <= TL.lz; ++c) {
                        if (a + b + c < min_log)
                            continue;
                        const Tiling S = {a, b, c};
                        const int32_t cells = set_box(J, S);
                        if (cells > lds_cells)
                            continue;
                        const double ratio = (double)cells / (double)(1 << (a + b + c));
                        if (a + b + c > best_log || (a + b + c == best_log && ratio < best_ratio)) {
                            best = S;
                            best_log = a + b + c;
                            best_ratio = ratio;
                        }
                    }
            fits = best_log >= 0;
        }
        (void)set_box(J, best);
        if (fits && !staging_pays(J, best, TL)) {
            fits = false;
            best = TL;
        }
        set_reach(J, best);
        if (!fits)
            set_gather(J, best);
    }
    J.sub[0] = best.lx;
    J.sub[1] = best.ly;
    J.sub[2] = best.lz;
    return fits;
}

int32_t lds_cells_cap(int32_t elem_bytes)
{
    return (kMaxLdsBytes - 16) / elem_bytes & ~15;
}

int32_t lds_cells_for(int32_t bound, int32_t elem_bytes)
{
    return std::min(bound, lds_cells_cap(elem_bytes));
}

size_t lds_bytes_for(int32_t cells, int32_t elem_bytes)
{
    return ((size_t)cells * (size_t)elem_bytes + 15) & ~(size_t)15;
}

template <int DISP, bool INNER>
static void launch_single_t(const FwdJob &J, const Tiling &TL, int ntiles, int32_t cells, int grid,
                            size_t lds, hipStream_t s)
{
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, J, TL, ntiles, cells);
    };
    const bool aligned = J.oz % 4 == 0;
    if (J.dtype == kI16)
        launch(aligned ? &k_warp_single<int16_t, true, DISP, INNER>
                       : &k_warp_single<int16_t, false, DISP, INNER>);
    else
        launch(aligned ? &k_warp_single<float, true, DISP, INNER>
                       : &k_warp_single<float, false, DISP, INNER>);
}

static_assert(1 << (3 + 3 + 4 - 2) == kThreads, "one run of a displacement tile per thread");
static_assert(kDispTiling.lx == 3 && kDispTiling.ly == 3 && kDispTiling.lz == 4 && kThreads == 256,
              "the tile of spline_tile_u");
static_assert(kDispLdsCells >= kSplineTileLdsFloats,
              "the B-spline scratch of a tile fits its footprint reservation");

// Labels alone: one thread per run of 4 output voxels along z (one packed
// 4-byte store with kFlagVec), the coordinate and the nearest-neighbour gather
// of the fused warps (row_base, coord, label_checked), so the labels equal
// theirs bit for bit.  Block row blockIdx.y is the x-slab x = x0 + blockIdx.y;
// within it run r covers z = 4 (r mod runs_z) .. + 3 of y = r / runs_z.
__global__ __launch_bounds__(kThreads) void k_warp_labels(FwdJob J, int32_t runs_z, int32_t x0)
{
    const int r = blockIdx.x * kThreads + threadIdx.x;
    if (r >= J.oy * runs_z)
        return;
    const int x = x0 + (int)blockIdx.y;
    const int y = r / runs_z;
    const int z = 4 * (r - y * runs_z);
    const int32_t row = x * J.oy + y;
    Src S;
    S.lbl = make_rsrc(J.lbl, (uint32_t)J.in_extent);
    S.img = S.lbl;                     // not read
    S.nx = J.nx;
    S.ny = J.ny;
    S.nz = J.nz;
    S.ry = J.in_ry;
    S.rsy = J.in_sy;
    S.sy = S.sx = S.sxy = 0;
    const int8_t lfill = (int8_t)J.label_fill;
    const bool any_in = J.nx > 0 && J.ny > 0 && J.nz > 0;
    float rb[3];
    row_base(J.M, (float)x, (float)y, rb);
    int8_t L[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        L[k] = lfill;
        if (!any_in || z + k >= J.oz)
            continue;
        const float zf = (float)(z + k);
        L[k] = label_checked(S, coord(J.M, 0, rb, zf), coord(J.M, 1, rb, zf),
                             coord(J.M, 2, rb, zf), lfill);
    }
    gmut<int8_t> *lout = gm<int8_t>(J.lout);
    const uint32_t v0 = (uint32_t)row * (uint32_t)J.oz + (uint32_t)z;
    if (J.flags & kFlagVec) {
        *reinterpret_cast<gmut<uint32_t> *>(lout + v0) =
            (uint32_t)(uint8_t)L[0] | ((uint32_t)(uint8_t)L[1] << 8) |
            ((uint32_t)(uint8_t)L[2] << 16) | ((uint32_t)(uint8_t)L[3] << 24);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (z + k < J.oz)
                lout[v0 + k] = L[k];
    }
}

// Labels alone under a diagonal map, what resampling a label map to another grid
// is: the x and y cells are a plane's and a row's, and the z cells are the same
// for every row.  A wave takes rows of one plane, L = ceil(oz / V) lanes a row with
// V voxels each, 64 / L rows at once (SUB: two or more; rows past 64 V voxels in
// segments).  A row costs one store per lane, and V byte gathers, which a wave
// with one row at a time skips where its input row is the last one's; four rows'
// gathers are in flight together (one at a time a small map waits for each: 31 us
// where the general kernel took 24).  What is left is the output's own traffic:
// 512 x 512 x 320 from 160 x 160 x 100 takes 30 us, 103 with the general kernel.
// Coordinates are those of row_base and coord (the products with 0 add nothing),
// nearest voxels and the guard those of label_checked.
template <int V, bool SUB>
__global__ __launch_bounds__(kThreads) void k_warp_labels_diag(FwdJob J, int32_t x0, int32_t rows,
                                                               int32_t L)
{
    constexpr int kAhead = 4;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x = x0 + (int)blockIdx.y;
    const int sub = SUB ? div_small(lane, L, rcp_small(L)) : 0;
    const int nsub = SUB ? div_small(64, L, rcp_small(L)) : 1;      // rows at once
    const int y0 = ((int)blockIdx.x * (kThreads / 64) + wave) * rows;
    const int y1 = min(y0 + rows, J.oy);
    const rsrc_t src = make_rsrc(J.lbl, (uint32_t)J.in_extent);
    const uint32_t fill = (uint32_t)(uint8_t)(int8_t)J.label_fill;
    // nearest voxel of coordinate q on an axis of n voxels, or -1
    auto nearest = [](float q, int n) {
        const int j = nn_index(q);
        return q > -1.0f && q < (float)n && (uint32_t)j < (uint32_t)n ? j : -1;
    };
    const int jx = J.nz == 0 ? -1 : nearest(__builtin_fmaf(J.M[0], (float)x, J.M[3]), J.nx);
    for (int z0 = 0; z0 < J.oz; z0 += 64 * V) {    // (SUB: one segment)
        const int z = z0 + (lane - sub * L) * V;
        uint32_t jz[V], in = 0;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const int j = nearest(__builtin_fmaf(J.M[10], (float)(z + k), J.M[11]), J.nz);
            jz[k] = (uint32_t)max(j, 0);
            in |= (j >= 0 ? 1u : 0u) << k;
        }
        uint32_t w[V / 4];
#pragma unroll
        for (int i = 0; i < V / 4; ++i)
            w[i] = 0x01010101u * fill;
        int last = -1;                 // the input row in w (-1: fill)
        for (int yb = y0; yb < y1; yb += kAhead * nsub) {
            int row[kAhead];
            uint32_t c[kAhead][V];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int y = yb + u * nsub + sub;
                const int jy = nearest(__builtin_fmaf(J.M[5], (float)y, J.M[7]), J.ny);
                row[u] = jx < 0 || jy < 0 ? -1 : jx * J.in_ry + jy;
                if (!SUB)
                    row[u] = __builtin_amdgcn_readfirstlane(row[u]);
                if (SUB || row[u] != (u ? row[u - 1] : last)) {
                    const uint32_t base = (uint32_t)max(row[u], 0) * (uint32_t)J.in_sy;
#pragma unroll
                    for (int k = 0; k < V; ++k)
                        c[u][k] = row[u] < 0 ? fill
                                  : SUB      ? (uint8_t)load_i8(src, base + jz[k])
                                             : (uint8_t)load_i8_at(src, jz[k], base);
                }
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int y = yb + u * nsub + sub;
                if (SUB || row[u] != (u ? row[u - 1] : last))
#pragma unroll
                    for (int i = 0; i < V / 4; ++i) {
                        w[i] = 0;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            w[i] |= ((in >> (4 * i + k)) & 1 ? c[u][4 * i + k] : fill) << (8 * k);
                    }
                int8_t *out = J.lout + (((uint32_t)x * (uint32_t)J.oy + (uint32_t)y) *
                                            (uint32_t)J.oz + (uint32_t)z);
                if (y < y1 && (!SUB || sub < nsub)) {
                    if (z + V <= J.oz)
                        __builtin_memcpy(gm<int8_t>(out), w, V);
                    else
                        for (int k = 0; k < V && z + k < J.oz; ++k)
                            out[k] = (int8_t)(w[k >> 2] >> (8 * (k & 3)));
                }
            }
            last = row[kAhead - 1];
        }
    }
}

template <int V, bool SUB> static void launch_labels_diag(const FwdJob &J, hipStream_t s)
{
    // rows per wave: a multiple of the four steps in flight, more once that still
    // leaves 16384 waves (two per resident slot)
    const int32_t L = (J.oz + V - 1) / V, nsub = SUB ? 64 / L : 1;
    const int64_t steps = (int64_t)J.ox * ((J.oy + nsub - 1) / nsub);
    const int32_t rows = 4 * nsub * (int32_t)std::min<int64_t>(4, std::max<int64_t>(1, steps / (4 * 16384)));
    const unsigned bx = (unsigned)((J.oy + 4 * (int64_t)rows - 1) / (4 * (int64_t)rows));
    for (int32_t x0 = 0; x0 < J.ox; x0 += 65535) {
        const unsigned nx = (unsigned)std::min<int32_t>(65535, J.ox - x0);
        hipLaunchKernelGGL((k_warp_labels_diag<V, SUB>), dim3(bx, nx), dim3(kThreads), 0, s, J, x0,
                           rows, L);
    }
}

hipError_t launch_warp_labels(const FwdJob &J, hipStream_t s)
{
    const bool diagonal = J.M[1] == 0.0f && J.M[2] == 0.0f && J.M[4] == 0.0f && J.M[6] == 0.0f &&
                          J.M[8] == 0.0f && J.M[9] == 0.0f;
    // Rows past 512 voxels go in segments of 256, one after the other, which takes waves
    // enough (four rows each): 30 x 30 x 4000 took 20 us, 7 with the general kernel, but 100 x
    // 100 x 1500 takes 13 where that takes 22.  16 voxels a lane instead (4 KB of LDS, three
    // waves per SIMD) took 27 us for 100 x 100 x 600, 9 in segments.
    const bool waves = J.oz <= 512 || (int64_t)J.ox * ((J.oy + 3) >> 2) >= 1024;
    if (diagonal && waves && J.ox > 0 && J.oy > 0 && J.oz > 0) {
        // the fewest voxels a lane that cover a row at once (short rows would leave
        // lanes idle)
        if (J.oz <= 128)
            launch_labels_diag<4, true>(J, s);
        else if (J.oz <= 256 || J.oz > 512)
            launch_labels_diag<4, false>(J, s);
        else
            launch_labels_diag<8, false>(J, s);
        return hipGetLastError();
    }
    const int32_t runs_z = (J.oz + 3) >> 2;
    const int64_t slab = (int64_t)J.oy * runs_z;     // runs per x-slab (< 2^31)
    if (slab == 0 || J.ox == 0)
        return hipSuccess;
    const unsigned bx = (unsigned)((slab + kThreads - 1) / kThreads);
    for (int32_t x0 = 0; x0 < J.ox; x0 += 65535) {   // grid y: at most 65535 slabs a launch
        const unsigned nx = (unsigned)std::min<int32_t>(65535, J.ox - x0);
        hipLaunchKernelGGL(k_warp_labels, dim3(bx, nx), dim3(kThreads), 0, s, J, runs_z, x0);
    }
    return hipGetLastError();
}

// LDS cells for a displacement warp: the window of a tile under the affine part
// alone with two more cells per axis for the field's own variation, between the
// B-spline scratch and kDispLdsCells.  Tiles past it gather from memory; a gentle
// map leaves room for more workgroups (256^3 B-spline warps: 106 to 137 us at
// 7152 cells by the draw, 137 to 140 at 10224).
static int32_t disp_cells(const FwdJob &J)
{
    const int t[3] = {1 << kDispTiling.lx, 1 << kDispTiling.ly, 1 << kDispTiling.lz};
    double cells = 1.0;
    for (int i = 0; i < 3; ++i) {
        double span = 2.0 * (double)J.delta[i];
        for (int j = 0; j < 3; ++j)
            span += std::fabs((double)J.M[4 * i + j]) * (double)(t[j] - 1);
        const double e = std::min(std::floor(span) + 5.0, 16384.0);
        cells *= i == 2 ? (double)lds_pitch((int32_t)e) : e;
    }
    const int32_t least = (kSplineTileLdsFloats + 15) & ~15;
    return (int32_t)std::min(std::max(cells, (double)least), (double)kDispLdsCells);
}

// Tile of a single call whose windows fit no reservation and which gathers from memory
// (no LDS: the 60 KB that held nothing left two workgroups per CU): 4 x 8 x 32 voxels.
// Along z a tile reads whole lines of few rows where the map keeps to the rows (128 x 128 x
// 107 voxels of a 512 x 512 x 320 int16 scan: 20 us; 31 in 8 x 16 x 16, 28 in 8 x 8 x 16, 29 in
// 4 x 8 x 128); where it turns, a long tile spreads over as many rows as voxels (turned by
// 10 degrees 84 us; 91, 87, 143; 160 x 160 x 120 of 400 x 400 x 300 82; 100, 77, 251).
static Tiling gather_tiling(const FwdJob &J)
{
    return J.oz > 16 ? Tiling{2, 3, 5} : Tiling{3, 3, 4};
}

hipError_t launch_warp_single(const FwdJob &J0, const Tiling &TL0, hipStream_t s)
{
    FwdJob Js = J0;
    const bool displaced = J0.disp || J0.ctrl;
    const int32_t esz = (Js.flags & kFlagLds16) ? 2 : 4;
    Tiling TL = displaced ? kDispTiling : TL0;
    const int32_t bound = displaced ? disp_cells(Js) : footprint_cells_bound(Js, TL);
    int32_t cells = lds_cells_for(displaced ? bound : std::min(bound, kAffineLdsCells), esz);
    const bool fits = choose_subtile(Js, TL, cells);
    if (!fits && !displaced) {         // gathers from memory
        const Tiling G = gather_tiling(Js);
        const int64_t tiles = (((int64_t)Js.ox + (1 << G.lx) - 1) >> G.lx) *
                              (((int64_t)Js.oy + (1 << G.ly) - 1) >> G.ly) *
                              (((int64_t)Js.oz + (1 << G.lz) - 1) >> G.lz);
        if (tiles < (int64_t)1 << 23)  // (2^32 threads at most; thin outputs keep theirs)
            TL = G;
        cells = 0;
        (void)choose_subtile(Js, TL, cells);
    }
    Js.tiles_x = (Js.ox + (1 << TL.lx) - 1) >> TL.lx;
    Js.tiles_y = (Js.oy + (1 << TL.ly) - 1) >> TL.ly;
    Js.tiles_z = (Js.oz + (1 << TL.lz) - 1) >> TL.lz;
    Js.rcp_ty = rcp_u32((uint32_t)Js.tiles_y);
    Js.rcp_tz = rcp_u32((uint32_t)Js.tiles_z);
    const FwdJob &J = Js;
    const int ntiles = J.tiles_x * J.tiles_y * J.tiles_z;
    if (ntiles == 0)
        return hipSuccess;
    const int grid = 8 * xcd_slots(ntiles);
    const size_t lds = lds_bytes_for(cells, esz);
    auto launch = &launch_single_t<kDispNone, true>;
    if (displaced && bound == kDispLdsCells)
        launch = J.ctrl ? &launch_single_t<kDispSpline, true> : &launch_single_t<kDispField, true>;
    else if (displaced)
        launch = J.ctrl ? &launch_single_t<kDispSpline, false> : &launch_single_t<kDispField, false>;
    launch(Js, TL, ntiles, cells, grid, lds, s);
    return hipGetLastError();
}

template <bool ALIGNED>
static void launch_batch_mode(int mode, const FwdJob *jobs_dev, const int32_t *prefix_dev,
                              int32_t njobs, int32_t grid, const Tiling &TL, int32_t lds_cells,
                              size_t lds, hipStream_t s)
{
    switch (mode) {
    case kBatchI16F32:
        hipLaunchKernelGGL((k_warp_batch<ALIGNED, kBatchI16F32>), dim3(grid), dim3(kThreads), lds,
                           s, jobs_dev, prefix_dev, njobs, TL, lds_cells);
        break;
    case kBatchI16I16:
        hipLaunchKernelGGL((k_warp_batch<ALIGNED, kBatchI16I16>), dim3(grid), dim3(kThreads), lds,
                           s, jobs_dev, prefix_dev, njobs, TL, lds_cells);
        break;
    case kBatchF32:
        hipLaunchKernelGGL((k_warp_batch<ALIGNED, kBatchF32>), dim3(grid), dim3(kThreads), lds, s,
                           jobs_dev, prefix_dev, njobs, TL, lds_cells);
        break;
    case kBatchSplineI16:
        hipLaunchKernelGGL((k_warp_batch<ALIGNED, kBatchSplineI16>), dim3(grid), dim3(kThreads),
                           lds, s, jobs_dev, prefix_dev, njobs, TL, lds_cells);
        break;
    case kBatchSplineF32:
        hipLaunchKernelGGL((k_warp_batch<ALIGNED, kBatchSplineF32>), dim3(grid), dim3(kThreads),
                           lds, s, jobs_dev, prefix_dev, njobs, TL, lds_cells);
        break;
    case kBatchSplineMixed:
        hipLaunchKernelGGL((k_warp_batch<ALIGNED, kBatchSplineMixed>), dim3(grid), dim3(kThreads),
                           lds, s, jobs_dev, prefix_dev, njobs, TL, lds_cells);
        break;
    default:
        hipLaunchKernelGGL((k_warp_batch<ALIGNED, kBatchMixed>), dim3(grid), dim3(kThreads), lds,
                           s, jobs_dev, prefix_dev, njobs, TL, lds_cells);
    }
}

hipError_t launch_warp_batch(const FwdJob *jobs_dev, const int32_t *prefix_dev, int32_t njobs,
                             int32_t total_tiles, int32_t grid, const Tiling &TL,
                             int32_t lds_cells, int32_t elem_bytes, int mode, bool aligned,
                             hipStream_t s)
{
    if (total_tiles == 0 || njobs == 0)
        return hipSuccess;
    const size_t lds = lds_bytes_for(lds_cells, elem_bytes);
    if (aligned)
        launch_batch_mode<true>(mode, jobs_dev, prefix_dev, njobs, grid, TL, lds_cells, lds, s);
    else
        launch_batch_mode<false>(mode, jobs_dev, prefix_dev, njobs, grid, TL, lds_cells, lds, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Standalone photometric pass (in place) and raw noise generator.
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kThreads) void k_photometric(float *data, int64_t n, int64_t nz,
                                                          Photo P, float occ_lo, float occ_hi,
                                                          uint32_t vol, uint32_t k0, uint32_t k1,
                                                          int vec)
{
    const int64_t ngroups = (n + 3) >> 2;
    for (int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x; g < ngroups;
         g += (int64_t)gridDim.x * kThreads) {
        const int64_t v0 = g << 2;
        float nzs[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (P.flags & kFlagNoise)
            gauss_group((uint64_t)g, vol, k0, k1, nzs);
        float x[4];
        if (vec) {
            const f32x4 w = *reinterpret_cast<const f32x4 *>(data + v0);
            x[0] = w.x;
            x[1] = w.y;
            x[2] = w.z;
            x[3] = w.w;
        } else {
            for (int k = 0; k < 4; ++k)
                x[k] = v0 + k < n ? data[v0 + k] : 0.0f;
        }
        if (P.flags & kFlagOcclude) {
            const int64_t z0 = v0 % nz;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float zf = (float)((z0 + k) % nz);
                if (zf >= occ_lo && zf <= occ_hi)
                    x[k] = 0.0f;
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            x[k] = photometric(P, x[k], nzs[k]);
        if (vec) {
            *reinterpret_cast<f32x4 *>(data + v0) = f32x4{x[0], x[1], x[2], x[3]};
        } else {
            for (int k = 0; k < 4; ++k)
                if (v0 + k < n)
                    data[v0 + k] = x[k];
        }
    }
}

hipError_t launch_photometric(float *data, int64_t n, int64_t nz, const Photo &P, float occ_lo,
                              float occ_hi, uint32_t vol, uint32_t k0, uint32_t k1, bool vec,
                              hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    const int64_t ngroups = (n + 3) >> 2;
    const int64_t blocks = std::min<int64_t>((ngroups + kThreads - 1) / kThreads, 256 * 64);
    hipLaunchKernelGGL(k_photometric, dim3((unsigned)blocks), dim3(kThreads), 0, s, data, n, nz, P,
                       occ_lo, occ_hi, vol, k0, k1, vec ? 1 : 0);
    return hipGetLastError();
}

__global__ __launch_bounds__(kThreads) void k_noise(uint64_t v0, int64_t n, uint32_t vol,
                                                    uint32_t k0, uint32_t k1, float *gauss,
                                                    uint32_t *words)
{
    const uint64_t g0 = v0 >> 2;
    const uint64_t g1 = (v0 + (uint64_t)n - 1) >> 2;
    const int64_t ng = (int64_t)(g1 - g0) + 1;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < ng;
         i += (int64_t)gridDim.x * kThreads) {
        const uint64_t g = g0 + (uint64_t)i;
        uint32_t c[4] = {(uint32_t)g, (uint32_t)(g >> 32), vol, 0u};
        philox4x32_10(c, k0, k1);
        if (words) {
            words[4 * i + 0] = c[0];
            words[4 * i + 1] = c[1];
            words[4 * i + 2] = c[2];
            words[4 * i + 3] = c[3];
        }
        if (gauss) {
            float z[4];
            box_muller(c[0], c[1], z[0], z[1]);
            box_muller(c[2], c[3], z[2], z[3]);
            for (int k = 0; k < 4; ++k) {
                const uint64_t v = 4 * g + k;
                if (v >= v0 && v < v0 + (uint64_t)n)
                    gauss[v - v0] = z[k];
            }
        }
    }
}

hipError_t launch_noise(uint64_t v0, int64_t n, uint32_t vol, uint32_t k0, uint32_t k1,
                        float *gauss, uint32_t *words, hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    const int64_t ng = (int64_t)(((v0 + (uint64_t)n - 1) >> 2) - (v0 >> 2)) + 1;
    const int64_t blocks = std::min<int64_t>((ng + kThreads - 1) / kThreads, 256 * 64);
    hipLaunchKernelGGL(k_noise, dim3((unsigned)blocks), dim3(kThreads), 0, s, v0, n, vol, k0, k1,
                       gauss, words);
    return hipGetLastError();
}

__global__ __launch_bounds__(kThreads) void k_box_muller(const uint32_t *__restrict__ w,
                                                         int64_t npairs, float *__restrict__ out)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < npairs;
         i += (int64_t)gridDim.x * kThreads) {
        float c, sn;
        box_muller(w[2 * i], w[2 * i + 1], c, sn);
        out[2 * i] = c;
        out[2 * i + 1] = sn;
    }
}

hipError_t launch_box_muller(const uint32_t *words, int64_t npairs, float *out, hipStream_t s)
{
    const int64_t blocks = std::min<int64_t>((npairs + kThreads - 1) / kThreads, 256 * 64);
    hipLaunchKernelGGL(k_box_muller, dim3((unsigned)blocks), dim3(kThreads), 0, s, words, npairs,
                       out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Plain streaming copy (measurement reference and cache eviction).
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kThreads) void k_copy16(const float4 *__restrict__ src,
                                                     float4 *__restrict__ dst, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads)
        dst[i] = src[i];
}

__global__ __launch_bounds__(kThreads) void k_copy1(const uint8_t *__restrict__ src,
                                                    uint8_t *__restrict__ dst, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads)
        dst[i] = src[i];
}

hipError_t launch_copy(const void *src, void *dst, size_t bytes, hipStream_t s)
{
    const bool aligned = ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst) |
                           bytes) & 15u) == 0;
    if (aligned) {
        const int64_t n = (int64_t)(bytes / 16);
        const int64_t blocks = std::min<int64_t>((n + kThreads - 1) / kThreads, 256 * 16);
        hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks), dim3(kThreads), 0, s,
                           static_cast<const float4 *>(src), static_cast<float4 *>(dst), n);
    } else {
        const int64_t n = (int64_t)bytes;
        const int64_t blocks = std::min<int64_t>((n + kThreads - 1) / kThreads, 256 * 16);
        hipLaunchKernelGGL(k_copy1, dim3((unsigned)blocks), dim3(kThreads), 0, s,
                           static_cast<const uint8_t *>(src), static_cast<uint8_t *>(dst), n);
    }
    return hipGetLastError();
}

}  // namespace ctaug
