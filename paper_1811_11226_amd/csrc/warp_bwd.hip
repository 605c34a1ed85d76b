// warp_bwd.hip -- adjoint kernels of the warp (gfx950).
//
// Workgroups take 8 x 8 x 16 output tiles, groups of consecutive ones (affine jobs) or
// one wave of persistent workgroups (displacements).  For every output voxel
// the upstream gradient is taken through the adjoint of the photometric chain
// (gain, zero on the occluded slab), the forward coordinate and cell are
// recomputed; the eight corner values
// (staged in LDS, fill substituted outside the volume) give the derivative of
// the trilinear interpolant on that cell, dV/dq.  Then
//   grad_img[c] += w_c * g          summed per tile in fixed point in LDS
//                                   (integer atomics, order-independent; 32
//                                   bits in one pass where the host bounds a
//                                   cell's samples, else 64 bits in x-plane
//                                   passes), then one global FP32 atomic per touched
//                                   cell; tiles whose footprint exceeds the
//                                   reservation, or with non-finite g, add
//                                   per corner with global FP32 atomics
//   grad_disp[i](p) = g * dV/dq_i   coalesced SoA stores
//   grad_ctrl                        B-spline warps evaluated from a control
//                                   grid: the tile's g dV/dq is contracted
//                                   with the spline weights along z, y and x
//                                   in LDS and added to the workgroup's LDS
//                                   accumulators of the control entries; one
//                                   row per workgroup, summed in a fixed order
//   grad_M[i][j] = sum g dV/dq_i [x,y,z,1]_j, FP64 per thread, reduced in the
//   workgroup and then across workgroups in a fixed order.
// grad_M and grad_ctrl are deterministic for a given device; grad_img is
// deterministic within a tile, and tiles meet in FP32 atomics.
#include "device_common.h"
#include "launch.h"
#include "tile_geom.h"

#include <algorithm>
#include <climits>
#include <cstring>
#include <cmath>
#include <mutex>
#include <vector>

namespace ctaug {

// Launch shape of the backward pass: 8 x 8 x 16 voxel tiles (one run of 4 z
// voxels per thread) in the XCD order (xcd_tile); for a displacement kBwdLdsCells
// FP32 cells of input footprint per workgroup (48 KB of LDS), for an affine job its
// windows' cells, used first for the staged image, then as the adjoint
// accumulators of the same cells.
constexpr Tiling kBwdTiling = {3, 3, 4};
constexpr int32_t kBwdLdsCells = 12288;
// An affine job whose windows need more takes up to this (60 KB, two workgroups
// per CU) before its tiles fall back to per-corner atomics.
constexpr int32_t kBwdLdsMax = 15360;
constexpr int64_t kBwdMaxGrid = kBwdMaxRows;

static int64_t bwd_tiles(int64_t ox, int64_t oy, int64_t oz)
{
    return ((ox + 7) >> 3) * ((oy + 7) >> 3) * ((oz + 15) >> 4);
}

static int64_t bwd_grid(int64_t ntiles)
{
    return std::min(((ntiles + 7) >> 3) << 3, kBwdMaxGrid);
}

int64_t bwd_partial_rows(int64_t ox, int64_t oy, int64_t oz)
{
    return bwd_grid(bwd_tiles(ox, oy, oz));
}

// Sum over the wave in a fixed order, in lane 63: DPP row shifts and broadcasts (a
// shuffle goes through LDS; twelve sums of six took about 7000 cycles).
__device__ __forceinline__ double wave_sum(double v)
{
#define CTAUG_DPP_ADD(ctrl, rows)                                                                 \
    v += __hiloint2double(                                                                        \
        __builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, rows, 0xF, true),                 \
        __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, rows, 0xF, true))
    CTAUG_DPP_ADD(0x111, 0xF);         // row_shr:1, 2, 4, 8: lane 15 of each row of 16
    CTAUG_DPP_ADD(0x112, 0xF);
    CTAUG_DPP_ADD(0x114, 0xF);
    CTAUG_DPP_ADD(0x118, 0xF);
    CTAUG_DPP_ADD(0x142, 0xA);         // row_bcast:15 into rows 1 and 3
    CTAUG_DPP_ADD(0x143, 0xC);         // row_bcast:31 into rows 2 and 3
#undef CTAUG_DPP_ADD
    return v;
}

extern __shared__ __attribute__((aligned(16))) float s_cells[];

// Derivative of the trilinear interpolant on the cell with corners K[a][b][c]
// (a: x, b: y, c: z) at fractions tt.
__device__ __forceinline__ void cell_gradient(const float K[8], const float tt[3], float dV[3])
{
    const float e00 = lerp(K[0], K[1], tt[2]), e01 = lerp(K[2], K[3], tt[2]);
    const float e10 = lerp(K[4], K[5], tt[2]), e11 = lerp(K[6], K[7], tt[2]);
    dV[0] = lerp(e10, e11, tt[1]) - lerp(e00, e01, tt[1]);
    dV[1] = lerp(e01 - e00, e11 - e10, tt[0]);
    dV[2] = lerp(lerp(K[1] - K[0], K[3] - K[2], tt[1]), lerp(K[5] - K[4], K[7] - K[6], tt[1]),
                 tt[0]);
}

// Largest control grid (3 Gx Gy Gz entries) whose gradient is fused into the
// adjoint kernel: FP32 accumulators in LDS beside a footprint reservation
// shrunk by as much, so that the workgroup's LDS stays at 48 KB; one FP64 row
// per workgroup in the workspace; rows summed in kCtrlRowGroups groups, then
// the groups (both in a fixed order).
constexpr int32_t kCtrlMaxEntries = 2048;
constexpr int32_t kSplineBwdCells = kBwdLdsCells - kCtrlMaxEntries;
constexpr int32_t kCtrlRowGroups = 64;
static_assert(kSplineTileLdsFloats <= kSplineBwdCells, "the B-spline scratch fits the reservation");
static_assert(kBwdTiling.lx == 3 && kBwdTiling.ly == 3 && kBwdTiling.lz == 4 && kThreads == 256,
              "the tile of spline_tile_u");

// v + (v of the lane at quad position q ^ 1), then ^ 2: sum over the 4 lanes
// of a quad, in the same order on every lane (DPP quad permutes, no LDS).
__device__ __forceinline__ float quad_sum(float v)
{
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true));
    return v;
}

// Fixed-point image adjoint.  A tile's contributions w_c * g are added into
// 64-bit integer LDS accumulators (integer LDS atomics run at full rate where
// FP32 ones do not, and integer sums do not depend on the order of the
// additions): with gmax the tile's largest |g| and gmax < 2^e, each FP32
// contribution v is scaled by S = 2^(50 - e) (exact) and rounded to the
// nearest integer (ties to even), so |v S| < 2^50 and, as the weights of a
// sample sum to 1, every cell's sum over the tile's 1024 samples stays below
// 2^60.  The rounding adds 1.5 * 2^52 in FP64, which leaves the integer in
// the low mantissa bits: two integer operations recover it.
__device__ __forceinline__ long long to_fixed(float v, double S)
{
    constexpr double kMagic = 0x1.8p52;
    const double d = __builtin_fma((double)v, S, kMagic);
    return __double_as_longlong(d) - __double_as_longlong(kMagic);
}

// The 32-bit variant for affine jobs, one pass over the whole footprint (the
// accumulators take the cells the staged image took).  The host bounds how
// many of a tile's samples can have one input cell among their corners: at
// most 2^b (fixed32_bits).  Each contribution is scaled by 2^sc, sc = 30 - b
// - e (exact: the voxel's gradient is multiplied by the power of two before
// the weights, which rounds as the unscaled product would), and rounded to
// the nearest integer: |v 2^sc| < 2^(30 - b), so a cell's sum of at most 2^b
// of them stays within 2^30.  The unit 2^-sc is at most 2^(b - 29) gmax, so
// for b <= kFixed32MaxBits the rounding stays within 2^-23 gmax, the order
// of the FP32 product's own.
constexpr int kFixed32MaxBits = 7;

// Spline weight matrix of one tile axis: Wt[p][c] = B_{c - (i(p) - i(p0))}(t(p))
// for the 2^lp voxels p0 + p <= p1 of the axis and the window of kSplineWindow
// controls starting at i(p0); 0 elsewhere.  One entry per calling thread.
__device__ __forceinline__ void spline_weight_entry(int e, int p0, int p1, float inv_h, int32_t G,
                                                    float *Wt)
{
    const int p = p0 + (e / kSplineWindow), c = e % kSplineWindow;
    float w = 0.0f;
    if (p <= p1) {
        int32_t i;
        float t, Bw[4];
        bs_cell(p, inv_h, G, i, t);
        bs_basis(t, Bw);
        const int j = c - (i - bs_index(p0, inv_h, G));
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
            if (j == jj)
                w = Bw[jj];
    }
    Wt[e] = w;
}

// Control-grid adjoint of one 8 x 8 x 16 displacement tile.  gu[k][i] is
// g dV/dq_i of voxel k of the thread's run (0 outside the tile or the guard).
// Contractions in LDS, each in a fixed order (FP32 inside the tile):
//   W[row][i][c]   = sum_z  Zw[z][c] gu_i(row, z)        (4 lanes of a row, butterfly)
//   H[x][i][b][c]  = sum_y  Yw[y][b] W[(x, y)][i][c]
//   R[i][a][b][c]  = sum_x  Xw[x][a] H[x][i][b][c]
// then R is added to the workgroup's FP32 accumulators acc (LDS, one per
// control entry; each entry is updated by one thread per tile and tiles come
// in a fixed order, so the sums are deterministic).  Every axis window must
// hold at most kSplineWindow controls (checked on the host).  The caller
// guarantees that no thread reads the scratch LDS on entry; ends with a
// barrier.
__device__ __forceinline__ void ctrl_adjoint_tile(const BsplineGeom &B, int x0, int y0, int z0,
                                                  int x1, int y1, int z1, int t,
                                                  const float (&gu)[4][3], float *lds, float *acc)
{
    constexpr int NW = kSplineWindow;
    static_assert(NW == 8, "window entries are indexed with 3-bit fields");
    float *Zw = lds;                           // [16][NW]
    float *Yw = Zw + 16 * NW;                  // [8][NW]
    float *Xw = Yw + 8 * NW;                   // [8][NW]
    float *W = Xw + 8 * NW;                    // [64][3][NW]
    float *H = W + 64 * 3 * NW;                // [8][3][NW][NW]
    float *R = H + 8 * 3 * NW * NW;            // [3][NW][NW][NW]
    static_assert(16 * NW + 16 * NW + 64 * 3 * NW + 8 * 3 * NW * NW + 3 * NW * NW * NW <=
                      kSplineBwdCells,
                  "the tile's contraction scratch fits the footprint reservation");
    const int rr = t >> 2, zr = t & 3;
    // controls of the tile's window per axis (at most NW): contractions stop
    // there, as every weight beyond is zero and no later stage reads beyond
    const int ixl = bs_index(x0, B.inv_hx, B.gx), iyl = bs_index(y0, B.inv_hy, B.gy),
              izl = bs_index(z0, B.inv_hz, B.gz);
    const int ncx = bs_index(x1, B.inv_hx, B.gx) - ixl + 4,
              ncy = bs_index(y1, B.inv_hy, B.gy) - iyl + 4,
              ncz = bs_index(z1, B.inv_hz, B.gz) - izl + 4;
    if (t < 16 * NW)
        spline_weight_entry(t, z0, z1, B.inv_hz, B.gz, Zw);
    else if (t < 24 * NW)
        spline_weight_entry(t - 16 * NW, y0, y1, B.inv_hy, B.gy, Yw);
    else if (t < 32 * NW)
        spline_weight_entry(t - 24 * NW, x0, x1, B.inv_hx, B.gx, Xw);
    __syncthreads();
    // z: the 4 lanes of a row hold its 16 voxels; butterfly sum over them
#pragma unroll 1
    for (int c = 0; c < ncz; ++c) {
        const float *zc = Zw + zr * NW + c;    // voxel k of the run sits at z offset zr + 4k
        const float w0 = zc[0], w1 = zc[4 * NW], w2 = zc[8 * NW], w3 = zc[12 * NW];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            float v = w0 * gu[0][i];
            v = __builtin_fmaf(w1, gu[1][i], v);
            v = __builtin_fmaf(w2, gu[2][i], v);
            v = __builtin_fmaf(w3, gu[3][i], v);
            v = quad_sum(v);
            if (zr == 0)
                W[(rr * 3 + i) * NW + c] = v;
        }
    }
    __syncthreads();
    if (t < 8 * 3 * NW && (t & (NW - 1)) < ncz) {   // (x, i, c) -> H[x][i][b][c], b < ncy
        const int xr = t / (3 * NW), ic = t - xr * 3 * NW;
        const int i = ic / NW, c = ic - i * NW;
        float wv[8];
#pragma unroll
        for (int yr = 0; yr < 8; ++yr)
            wv[yr] = W[((xr * 8 + yr) * 3 + i) * NW + c];
#pragma unroll 1
        for (int b = 0; b < ncy; ++b) {
            float h = 0.0f;
#pragma unroll
            for (int yr = 0; yr < 8; ++yr)
                h = __builtin_fmaf(Yw[yr * NW + b], wv[yr], h);
            H[((xr * 3 + i) * NW + b) * NW + c] = h;
        }
    }
    __syncthreads();
    if (t < 3 * NW * NW && (t & (NW - 1)) < ncz && ((t >> 3) & (NW - 1)) < ncy) {
        // (i, b, c) -> R[i][a][b][c], a < ncx
        const int i = t / (NW * NW), bc = t - i * NW * NW;
        float hv[8];
#pragma unroll
        for (int xr = 0; xr < 8; ++xr)
            hv[xr] = H[(xr * 3 + i) * NW * NW + bc];
#pragma unroll 1
        for (int a = 0; a < ncx; ++a) {
            float r = 0.0f;
#pragma unroll
            for (int xr = 0; xr < 8; ++xr)
                r = __builtin_fmaf(Xw[xr * NW + a], hv[xr], r);
            R[(i * NW + a) * NW * NW + bc] = r;
        }
    }
    __syncthreads();
    for (int e = t; e < 3 * NW * NW * NW; e += kThreads) {
        const int c = e & (NW - 1), b = (e >> 3) & (NW - 1), a = (e >> 6) & (NW - 1), i = e >> 9;
        if (a < ncx && b < ncy && c < ncz)
            acc[((i * B.gx + ixl + a) * B.gy + iyl + b) * B.gz + izl + c] += R[e];
    }
    __syncthreads();
}

// The workgroup's sum of acc[12] (fixed order: wave butterflies, then the
// four waves in order) written to row[0..11].  Every thread must call it;
// ends after a barrier.
__device__ __forceinline__ void write_partial_row(const double (&acc)[12],
                                                  double (*red)[12], double *row)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const double sum = wave_sum(acc[i]);
        if (lane == 63)
            red[wave][i] = sum;
    }
    __syncthreads();
    if (threadIdx.x < 12) {
        double sum = 0.0;
        for (int w = 0; w < kThreads / 64; ++w)
            sum += red[w][threadIdx.x];
        row[threadIdx.x] = sum;
    }
    __syncthreads();                   // red is reused by the next row
}

// Place of tile t in job J's grid of tiles.
__device__ __forceinline__ void tile_place(const FwdJob &J, int t, int &tx, int &ty, int &tz)
{
    const int rest = (int)div_rcp((uint32_t)t, (uint32_t)J.tiles_z, J.rcp_tz);
    tz = t - rest * J.tiles_z;
    tx = (int)div_rcp((uint32_t)rest, (uint32_t)J.tiles_y, J.rcp_ty);
    ty = rest - tx * J.tiles_y;
}

// The upstream gradient of the calling thread's run in tile t of job J
// (voxels z0 + zr + 4k of row (x0 + xr, y0 + yr)); 0 past the output.
__device__ __forceinline__ void load_run_g(JobPtr Jp, const float *__restrict__ g, int t, int tid,
                                           float (&gv)[4])
{
    const int zr = tid & 3, yr = (tid >> 2) & 7, xr = tid >> 5;
    const FwdJob &J = *(const FwdJob *)reload(Jp);
    const Tiling TL = kBwdTiling;
    int tx, ty, tz;
    tile_place(J, t, tx, ty, tz);
    const int x = (tx << TL.lx) + xr, y = (ty << TL.ly) + yr, z = (tz << TL.lz) + zr;
    const bool row_ok = x < J.ox && y < J.oy;
    const int32_t v0 = row_ok ? (x * J.oy + y) * J.oz + z : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        gv[k] = row_ok && z + 4 * k < J.oz ? g[v0 + 4 * k] : 0.0f;
}

// Largest of the wave's values, as a scalar (DPP, as in block_minmax3).
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
#define CTAUG_DPP_MAX(ctrl, rows)                                                                 \
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xF, false))
    CTAUG_DPP_MAX(0x111, 0xF);
    CTAUG_DPP_MAX(0x112, 0xF);
    CTAUG_DPP_MAX(0x114, 0xF);
    CTAUG_DPP_MAX(0x118, 0xF);
    CTAUG_DPP_MAX(0x142, 0xA);
    CTAUG_DPP_MAX(0x143, 0xC);
#undef CTAUG_DPP_MAX
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Adds the touched accumulators of `planes` window planes from lox (rows of ez
// cells, ey rows per plane, pitch cells apart in s_acc) to the in-volume cells of
// g_img, one FP32 global atomic each; conv converts an accumulator.  A row is
// taken by neighbouring lanes, one cell each (atomics of an instruction on
// consecutive cells coalesce; lanes 16 bytes apart took twice as long).  A wave
// takes planes, and of a plane as many rows at once as it has lanes for: its place
// is then scalar, a lane's offset from it fixed, and the loop a few additions.  The
// kernel is bound by the instructions its waves issue; rows handed to lanes across
// planes took 35 a cell where this takes 16 (8 x 128^3 228 -> 211 us, 256^3 B-spline
// adjoint 375 -> 356).
template <typename A, typename F>
__device__ __forceinline__ void flush_cells(const A *s_acc, int planes, int ey, int ez, int pitch,
                                            int lox, int loy, int loz, const FwdJob &J, int tid,
                                            float *__restrict__ g_img, F conv)
{
    constexpr int kWaves = kThreads / 64;
    const int xl = max(0, -lox), xh = min(planes, J.nx - lox);
    const int yl = max(0, -loy), ny = min(ey, J.ny - loy) - yl;
    const int lane = tid & 63, lpr = min(ez, 64);
    const float rcp_l = rcp_small(lpr);
    const int rpw = __builtin_amdgcn_readfirstlane(div_small(64, lpr, rcp_l));
    const int r = div_small(lane, lpr, rcp_l);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const char *s = reinterpret_cast<const char *>(s_acc);
    const int step = (int)sizeof(A) * rpw * pitch;         // bytes from pass to pass
    const int last = (int)sizeof(A) * (planes * ey * pitch - 1);
    constexpr int kAhead = 2;          // passes whose accumulators are read together
    for (int z0 = 0; z0 < ez; z0 += 64) {                  // (rarely more than once)
        const int z = z0 + lane - r * lpr;
        const int row = z < ez && (uint32_t)(loz + z) < (uint32_t)J.nz && r < rpw ? r : INT_MAX;
        const int in_plane = (int)sizeof(A) * (r * pitch + z);
        const uint32_t o = (uint32_t)(r * J.nz + (z - z0));
        for (int cx = xl + wave; cx < xh; cx += kWaves) {
            int at = (int)sizeof(A) * (cx * ey + yl) * pitch + in_plane;
            float *p = g_img + (((lox + cx) * J.ny + loy + yl) * J.nz + loz + z0);
            for (int left = ny; left > 0; left -= kAhead * rpw) {
                A v[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u)           // no branch: past the plane, unused
                    v[u] = *reinterpret_cast<const A *>(s + min(at + u * step, last));
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    if (row < left - u * rpw && v[u] != 0)
                        unsafeAtomicAdd(p + o, conv(v[u]));
                    p += rpw * J.nz;
                }
                at += kAhead * step;
            }
        }
    }
}

// The adjoint of one 8 x 8 x 16 output tile t of job J, for the calling
// thread's run (voxels z0 + zr + 4k, k = 0..3, of row (xr, yr): lanes next to each
// other take neighbouring z, so that the LDS accumulator updates of one
// instruction fall in different banks): coordinates, the
// staged footprint, dV/dq and its FP64 parameter sums (into acc), the image
// adjoint (fixed-point tile sums, flushed with FP32 atomics), the
// displacement gradient and the control-grid contraction.  gin holds the
// run's upstream gradient (load_run_g); the next tile's (tn of job Jn, when
// has_next) is loaded into gnext once the image scatter is done, so that its
// latency hides behind the flush.  Uniform over the workgroup; ends with
// every LDS read and write of the tile done.
//
// Footprints are the forward warps' windows (fill where outside the volume,
// coordinates through guard_coord): a sample outside the guard reads only fill,
// so its dV/dq is exactly 0, and voxels past the output take the coordinates of the
// last one inside it, so no sample branches.
template <typename T, int DISP, bool NARROW>
__device__ __forceinline__ void bwd_tile(JobPtr Jp, int t, bool want_ctrl, bool need_dv,
                                         const float (&gin)[4], bool has_next, JobPtr Jn,
                                         const float *__restrict__ gn, int tn, float (&gnext)[4],
                                         float *__restrict__ g_img, float *__restrict__ g_disp,
                                         float *s_ctrl, int32_t lds_cells, int fix_bits,
                                         double (&acc)[12],
                                         int (*s_red)[8], uint32_t *s_gmax)
{
    const Tiling TL = kBwdTiling;
    // the thread's index anew for each tile: what follows from it is then computed where
    // it is used, not kept (and spilled) across the tiles
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int zr = tid & 3, yr = (tid >> 2) & 7, xr = tid >> 5;
    bool fetched = false;              // gnext loaded (uniform)
    int x0, y0, z0, x1, y1, z1;
    float qv[4][3], gpk[4];
    uint32_t live = 0;                 // voxel k of the run is in the output and guarded
    int cls, lo[3], e[3], pitch;
    bool lds;
    {
        const FwdJob &J = *(const FwdJob *)reload(Jp);
        int tx, ty, tz;
        tile_place(J, t, tx, ty, tz);
        x0 = tx << TL.lx;
        y0 = ty << TL.ly;
        z0 = tz << TL.lz;
        x1 = min(x0 + (1 << TL.lx), J.ox) - 1;
        y1 = min(y0 + (1 << TL.ly), J.oy) - 1;
        z1 = min(z0 + (1 << TL.lz), J.oz) - 1;
        float gr[3] = {0.0f, 0.0f, 0.0f};
        if (DISP == kDispNone) {
            const int c = box_window(J, (float)x0, (float)y0, (float)z0, lo, gr);
            cls = __builtin_amdgcn_readfirstlane(c);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                lo[i] = __builtin_amdgcn_readfirstlane(lo[i]);
                e[i] = J.box_e[i];
            }
            if (cls == kInterior)      // whole quads, of which the last ones may be needed
                e[2] = (e[2] + 3) & ~3;
            pitch = J.box_pitch;
            lds = cls != kOutside && e[0] != 0;
        }
        const int x = x0 + xr, y = y0 + yr, z = z0 + zr;
        const bool row_ok = x <= x1 && y <= y1;
        const int xc = min(x, x1), yc = min(y, y1);
        const float nf[3] = {(float)J.nx, (float)J.ny, (float)J.nz};
        float u[3][4];
        if (DISP == kDispSpline)
            spline_tile_u<false>(J.ctrl, J.bs, x0, y0, z0, x1, y1, z1, x, y, z, 4, 4, true, tid,
                                 s_cells, u);
        float rb[3];
        row_base(J.M, (float)xc, (float)yc, rb);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int zc = min(z + 4 * k, z1);
            const bool valid = row_ok && z + 4 * k <= z1;
            const float zf = (float)zc;
            float q[3];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                q[i] = coord(J.M, i, rb, zf);
            if (DISP == kDispField) {
                gconst<float> *disp = gc<float>(J.disp);
                const int32_t nvox = J.ox * J.oy * J.oz;
                const int32_t v = (xc * J.oy + yc) * J.oz + zc;
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    q[i] = q[i] + disp[i * nvox + v];
            } else if (DISP == kDispSpline) {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    q[i] = q[i] + u[i][k];
            }
            const bool interior = DISP == kDispNone && cls == kInterior;
            const bool gd = valid && (interior || in_guard(q[0], q[1], q[2], J.nx, J.ny, J.nz));
            live |= (gd ? 1u : 0u) << k;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                qv[k][i] = interior ? q[i] : guard_coord(q[i], nf[i]);
            // adjoint of the photometric chain without window: the output
            // is gain * V + offset + sigma * n off the occluded slab and
            // does not depend on V on it
            float gv = gin[k];
            if (J.flags & kFlagPhoto) {
                gv = J.gain * gv;
                if ((J.flags & kFlagOcclude) && zf >= J.occ_lo && zf <= J.occ_hi)
                    gv = 0.0f;
            }
            gpk[k] = gv;
        }
        if (DISP != kDispNone) {
            // no a-priori bound with a displacement field: the footprint is the
            // range of the cells of the tile's samples (block reduction)
            int fmn[3], fmx[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                fmn[i] = flr_i32(fminf(fminf(qv[0][i], qv[1][i]), fminf(qv[2][i], qv[3][i])));
                fmx[i] = flr_i32(fmaxf(fmaxf(qv[0][i], qv[1][i]), fmaxf(qv[2][i], qv[3][i])));
            }
            block_minmax3(fmn, fmx, s_red);
            __syncthreads();           // a tile without a footprint passes no other
            const int n[3] = {J.nx, J.ny, J.nz};
            bool outside = J.nx == 0 || J.ny == 0 || J.nz == 0, inside = true;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                lo[i] = fmn[i];
                e[i] = fmx[i] - fmn[i] + 2;
                outside = outside || lo[i] >= n[i] || lo[i] + e[i] <= 0;
                inside = inside && lo[i] >= 0 && lo[i] + e[i] <= n[i];
            }
            // whole quads inside the volume: an inside window may start earlier
            inside = inside && ((e[2] + 3) & ~3) <= J.nz;
            if (inside) {
                const int zl = min(lo[2], J.nz - ((e[2] + 3) & ~3));
                e[2] += lo[2] - zl;
                lo[2] = zl;
            }
            pitch = lds_pitch(e[2]);
            cls = outside ? kOutside : inside ? kInterior : kBoundary;
            lds = !outside && (int64_t)e[0] * e[1] <= lds_cells && pitch <= lds_cells &&
                  e[0] * e[1] * pitch <= lds_cells && window24(lo[0], e[0]) &&
                  window24(lo[1], e[1]);
        }
        if (lds && g_img) {
            // the tile's largest |g| over its guarded samples, as bits: reduced
            // in each wave here, across the waves after the barrier that ends
            // the corner reads
            uint32_t gw = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                gw = max(gw, (live >> k) & 1 ? __float_as_uint(gpk[k]) & 0x7fffffffu : 0u);
            gw = wave_max(gw);
            if ((tid & 63) == 0)
                s_gmax[tid >> 6] = gw;
        }
        if (lds && need_dv) {          // the image adjoint alone needs no corner values
            const Src S = make_src<T>(J);
            const int quads = (e[2] + 3) >> 2;
            const StageWalk W = stage_walk<kThreads>(e[0] * e[1], e[1], quads, tid);
            if (W.passes > 0 && J.nz >= 4) {
                stage_window<T, float, DISP == kDispNone>(J, S, W, lo, gr, e[1], pitch,
                                                          cls == kInterior,
                                                          reinterpret_cast<uint8_t *>(s_cells));
            } else {
                TileGeom G;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    G.lo[i] = lo[i];
                    G.e[i] = e[i];
                }
                G.quads = quads;
                G.pitch = pitch;
                stage_footprint<T, float>(J, S, G, s_cells);
            }
            __syncthreads();
        }
    }
    const int ey = e[1], sxy = e[1] * pitch;
    // per voxel of the run: LDS cell of corner (0,0,0), fractions
    int base[4], cx0[4];
    float tw[4][3];
    float S[3] = {0.0f, 0.0f, 0.0f}, Sz[3] = {0.0f, 0.0f, 0.0f};
    float gu[4][3];
    const FwdJob &J = *(const FwdJob *)reload(Jp);
    const int x = x0 + xr, y = y0 + yr, z = z0 + zr;
    const bool row_ok = x <= x1 && y <= y1;
    const int sy = 4 * pitch, sx = 4 * sxy;                // bytes
    const int c0 = window_origin(lo, sx, sy, 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool valid = row_ok && z + 4 * k <= z1;
        float dV[3] = {0.0f, 0.0f, 0.0f};
        if (lds) {
            int ix, iy, iz;
            if (cls == kInterior) {
                ix = flr_i32(qv[k][0]);
                iy = flr_i32(qv[k][1]);
                iz = flr_i32(qv[k][2]);
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    tw[k][i] = __builtin_amdgcn_fractf(qv[k][i]);
            } else {
                const float fx = floorf(qv[k][0]), fy = floorf(qv[k][1]), fz = floorf(qv[k][2]);
                ix = (int)fx;
                iy = (int)fy;
                iz = (int)fz;
                tw[k][0] = qv[k][0] - fx;
                tw[k][1] = qv[k][1] - fy;
                tw[k][2] = qv[k][2] - fz;
            }
            const int a = mad_i24(ix, sx, mad_i24(iy, sy, iz * 4 + c0));
            base[k] = a;
            cx0[k] = ix - lo[0];
            if (need_dv) {
                const char *s = reinterpret_cast<const char *>(s_cells);
                const float *c00 = reinterpret_cast<const float *>(s + a);
                const float *c01 = reinterpret_cast<const float *>(s + (a + sy));
                const float *c10 = reinterpret_cast<const float *>(s + (a + sx));
                const float *c11 = reinterpret_cast<const float *>(s + (a + sx + sy));
                const float K[8] = {c00[0], c00[1], c01[0], c01[1], c10[0], c10[1], c11[0], c11[1]};
                cell_gradient(K, tw[k], dV);
            }
        } else if (cls != kOutside && (live >> k) & 1) {
            const Src src = make_src<T>(J);
            const float gp = gpk[k];
            float K[8], tt[3];
            int32_t i0[3];
            corners_checked<T>(src, qv[k][0], qv[k][1], qv[k][2], J.fill, K, tt, i0);
            cell_gradient(K, tt, dV);
            if (g_img && gp != 0.0f) {
                const float wx[2] = {1.0f - tt[0], tt[0]};
                const float wy[2] = {1.0f - tt[1], tt[1]};
                const float wz[2] = {1.0f - tt[2], tt[2]};
#pragma unroll 1
                for (int c = 0; c < 8; ++c) {
                    const int32_t cx = i0[0] + (c >> 2), cy = i0[1] + ((c >> 1) & 1),
                                  cz = i0[2] + (c & 1);
                    // zero contributions are skipped; a non-finite
                    // g reaches every in-volume corner (0 * inf and
                    // 0 * NaN are NaN), as in the per-corner path
                    const float cw = (c & 4 ? wx[1] : wx[0]) * (c & 2 ? wy[1] : wy[0]) *
                                     (c & 1 ? wz[1] : wz[0]) * gp;
                    const bool ok = cx >= 0 && cx < J.nx && cy >= 0 && cy < J.ny && cz >= 0 &&
                                    cz < J.nz && cw != 0.0f;
                    if (ok)
                        unsafeAtomicAdd(g_img + (cx * J.ny + cy) * J.nz + cz, cw);
                }
            }
        }
        if (DISP != kDispNone && g_disp && valid) {
            const int32_t nvox = J.ox * J.oy * J.oz;
            const int32_t v = (x * J.oy + y) * J.oz + z + 4 * k;
            g_disp[v] = gpk[k] * dV[0];
            g_disp[nvox + v] = gpk[k] * dV[1];
            g_disp[2 * nvox + v] = gpk[k] * dV[2];
        }
        const float zf = (float)(z + 4 * k);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const float c = valid ? gpk[k] * dV[i] : 0.0f;
            gu[k][i] = c;
            S[i] += c;
            Sz[i] = __builtin_fmaf(c, zf, Sz[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        acc[4 * i + 0] += (double)x * (double)S[i];
        acc[4 * i + 1] += (double)y * (double)S[i];
        acc[4 * i + 2] += (double)Sz[i];
        acc[4 * i + 3] += (double)S[i];
    }
    if (lds)                           // uniform: no barrier is skipped by part of the group
        __syncthreads();               // every corner read of the staged image is done
    if (want_ctrl)                     // before the image scatter: gu dies here
        ctrl_adjoint_tile(J.bs, x0, y0, z0, x1, y1, z1, tid, gu, s_cells, s_ctrl);
    if (lds && g_img) {
        // the tile's largest |g| (the waves' maxima, written before the
        // barrier that ended the corner reads); every wave reads it before
        // any wave goes on to the next tile, which writes s_gmax again:
        // each branch below passes a barrier before the tile ends
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        const u4 gw = *reinterpret_cast<const u4 *>(s_gmax);
        const float gm = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane(
            (int)max(max(gw.x, gw.y), max(gw.z, gw.w))));
        // x-planes of 64-bit accumulators that fit the footprint reservation
        const int planes = (lds_cells >> 1) / sxy;
        if (NARROW && gm >= 0x1p-96f && gm <= 3.40282347e38f) {
            // one pass, 32-bit accumulators (gmax >= 2^-96 keeps every
            // scaled value and every flushed sum in the normal range)
            const int sc = 30 - fix_bits - (ilogbf(gm) + 1);
            const float S32 = __builtin_ldexpf(1.0f, sc);    // normal: sc in [-105, 125]
            const float r32 = __builtin_ldexpf(1.0f, -sc);
            int *s_acc = reinterpret_cast<int *>(s_cells);
            const int n = e[0] * sxy;                        // a multiple of 4
            for (int c = 4 * tid; c < n; c += 4 * kThreads)
                *reinterpret_cast<f32x4 *>(s_acc + c) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (!((live >> k) & 1))
                    continue;
                const float wx[2] = {1.0f - tw[k][0], tw[k][0]};
                const float wy[2] = {1.0f - tw[k][1], tw[k][1]};
                const float gks = gpk[k] * S32;
                const float gz0 = (1.0f - tw[k][2]) * gks, gz1 = tw[k][2] * gks;
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int bb = 0; bb < 2; ++bb) {
                        const float wxy = wx[a] * wy[bb];
                        int *row = reinterpret_cast<int *>(reinterpret_cast<char *>(s_acc) +
                                                           (base[k] + a * sx + bb * sy));
                        atomicAdd(row, (int)__builtin_rintf(wxy * gz0));
                        atomicAdd(row + 1, (int)__builtin_rintf(wxy * gz1));
                    }
                __builtin_amdgcn_sched_barrier(0);       // one voxel at a time
            }
            __syncthreads();
            if (has_next) {            // waited for here: after the flush the wait would be
                                       // for its atomics too (memory operations return in order)
                load_run_g(Jn, gn, tn, tid, gnext);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    asm volatile("" : "+v"(gnext[k]));
                fetched = true;
            }
            flush_cells(s_acc, e[0], ey, e[2], pitch, lo[0], lo[1], lo[2], J, tid, g_img,
                        [=](int v) { return (float)v * r32; });
            __syncthreads();           // LDS is reused next
        } else if (!NARROW && gm > 0.0f && gm <= 3.40282347e38f && planes > 0) {
            const int ex = ilogbf(gm) + 1;         // gm < 2^ex
            const double S64 = ldexp(1.0, 50 - ex);
            const double rS = ldexp(1.0, ex - 50);
            long long *s_acc = reinterpret_cast<long long *>(s_cells);
            for (int sx0 = 0; sx0 < e[0]; sx0 += planes) {     // uniform
                const int np = min(planes, e[0] - sx0);
                const int n = np * sxy;                        // a multiple of 4
                for (int c = 2 * tid; c < n; c += 2 * kThreads)
                    *reinterpret_cast<f32x4 *>(s_acc + c) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                __syncthreads();
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (!((live >> k) & 1))
                        continue;
                    const float wx[2] = {1.0f - tw[k][0], tw[k][0]};
                    const float wy[2] = {1.0f - tw[k][1], tw[k][1]};
                    const float gz0 = (1.0f - tw[k][2]) * gpk[k], gz1 = tw[k][2] * gpk[k];
#pragma unroll
                    for (int a = 0; a < 2; ++a) {
                        const int px = cx0[k] + a - sx0;
                        if ((unsigned)px >= (unsigned)np)
                            continue;
#pragma unroll
                        for (int bb = 0; bb < 2; ++bb) {
                            const float wxy = wx[a] * wy[bb];
                            unsigned long long *row = reinterpret_cast<unsigned long long *>(
                                s_acc + (base[k] >> 2) + (a - sx0) * sxy + bb * pitch);
                            atomicAdd(row, (unsigned long long)to_fixed(wxy * gz0, S64));
                            atomicAdd(row + 1, (unsigned long long)to_fixed(wxy * gz1, S64));
                        }
                    }
                    // one voxel's conversions at a time (register pressure)
                    __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();
                flush_cells(s_acc, np, ey, e[2], pitch, lo[0] + sx0, lo[1], lo[2], J, tid, g_img,
                            [=](long long v) { return (float)((double)v * rS); });
                __syncthreads();       // LDS is reused next
            }
        } else {
            __syncthreads();           // every wave has read s_gmax
            // non-finite gradients, a footprint too large for one x-plane
            // of 64-bit accumulators, or a 32-bit tile with gmax < 2^-96:
            // FP32 global atomics per corner (none when gmax = 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (!((live >> k) & 1) || gm == 0.0f)
                    continue;
                const int rel = (base[k] >> 2) - cx0[k] * sxy;
                const int cy0 = rel / pitch, cz0 = rel - cy0 * pitch;
                const float wx[2] = {1.0f - tw[k][0], tw[k][0]};
                const float wy[2] = {1.0f - tw[k][1], tw[k][1]};
                const float gz[2] = {(1.0f - tw[k][2]) * gpk[k], tw[k][2] * gpk[k]};
#pragma unroll 1
                for (int c = 0; c < 8; ++c) {
                    const int gx = lo[0] + cx0[k] + (c >> 2), gy = lo[1] + cy0 + ((c >> 1) & 1),
                              gz2 = lo[2] + cz0 + (c & 1);
                    if ((unsigned)gx < (unsigned)J.nx && (unsigned)gy < (unsigned)J.ny &&
                        (unsigned)gz2 < (unsigned)J.nz)
                        unsafeAtomicAdd(g_img + (gx * J.ny + gy) * J.nz + gz2,
                                        (c & 4 ? wx[1] : wx[0]) * (c & 2 ? wy[1] : wy[0]) *
                                            (c & 1 ? gz[1] : gz[0]));
                }
            }
        }
    }
    if (!fetched) {
        if (has_next)
            load_run_g(Jn, gn, tn, tid, gnext);
        else
#pragma unroll
            for (int k = 0; k < 4; ++k)
                gnext[k] = 0.0f;
    }
}

// An affine adjoint's tiles come in groups of consecutive ones, a workgroup each,
// which the hardware hands out as workgroups end: tiles cost from nothing (outside
// the volume) to a full footprint, and with one wave of workgroups striding over
// all tiles the last ended 35 % after the mean on 8 x 128^3.  The group's FP64 sums
// of grad_M are one row, so they do not depend on who ran it when.  That took 8 x
// 128^3 from 257 to 229 us (2 tiles a group 228, 8 tiles 241).
constexpr int32_t kGroupTiles = 4;     // at most, but for the limit of kBwdMaxRows groups
constexpr int64_t kGroupFill = 4096;   // groups wanted: four per resident workgroup
constexpr int kGroupLog = 3;           // groups of a chunk of the XCD order (32 tiles)

// Register budgets follow the LDS: a displacement takes the whole 48 KB
// reservation (3 workgroups per CU), so at most 168 VGPRs (3 waves per SIMD);
// an affine job's footprint bound usually keeps a workgroup within 40 KB
// (4 per CU), so at most 128 VGPRs; its 64-bit variant would spill at that and
// takes 168 (spilled registers cost far more than a wave: scratch loads wait for
// every load before them).  NARROW (affine jobs with a bound fix_bits >= 0) takes
// the 32-bit image adjoint: a kernel of its own, as register allocation over
// both fixed-point paths spills.
template <typename T, int DISP, bool NARROW>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(
    NARROW ? 4 : 3))) void k_warp_bwd(FwdJob J, const float *__restrict__ g,
                                                       float *__restrict__ g_img,
                                                       float *__restrict__ g_disp,
                                                       double *__restrict__ partials,
                                                       double *__restrict__ ctrl_part,
                                                       int32_t ntiles, int32_t lds_cells,
                                                       int32_t fix_bits, int32_t group_tiles)
{
    const int b = blockIdx.x;
    // J is the first kernel argument
    const JobPtr Jp = (JobPtr)__builtin_amdgcn_kernarg_segment_ptr();

    double acc[12];
#pragma unroll
    for (int i = 0; i < 12; ++i)
        acc[i] = 0.0;

    // B-spline warps: this workgroup's control-grid gradient accumulators, in
    // LDS after the footprint reservation
    const bool want_ctrl = DISP == kDispSpline && ctrl_part != nullptr;
    const int32_t nctrl = 3 * J.bs.gx * J.bs.gy * J.bs.gz;
    // dV/dq (and so the staged corner values) is needed by every output but grad_img
    const bool need_dv = partials != nullptr || g_disp != nullptr || want_ctrl;
    float *s_ctrl = s_cells + lds_cells;
    if (want_ctrl) {
        for (int e = threadIdx.x; e < nctrl; e += kThreads)
            s_ctrl[e] = 0.0f;
        __syncthreads();
    }

    __shared__ __attribute__((aligned(16))) int s_red[4][8];
    __shared__ __attribute__((aligned(16))) uint32_t s_gmax[kThreads / 64];

    if constexpr (DISP == kDispNone) {
        // group g of group_tiles tiles; its row of partials is g
        const int g0 = xcd_tile<kGroupLog>(b & 7, b >> 3);
        const int t1 = min((g0 + 1) * group_tiles, ntiles);
        if (g0 * group_tiles >= ntiles)
            return;
        float gcur[4];
        load_run_g(Jp, g, g0 * group_tiles, (int)threadIdx.x, gcur);
        for (int t = g0 * group_tiles; t < t1; ++t) {
            float gnext[4];
            bwd_tile<T, DISP, NARROW>(Jp, t, false, need_dv, gcur, t + 1 < t1, Jp, g, t + 1, gnext,
                                      g_img, g_disp, s_ctrl, lds_cells, fix_bits, acc, s_red,
                                      s_gmax);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                gcur[k] = gnext[k];
        }
        if (partials) {
            __shared__ double red[kThreads / 64][12];
            write_partial_row(acc, red, partials + (int64_t)g0 * 12);
        }
        return;
    }
    XcdSlots slots(b >> 3, gridDim.x >> 3);
    for (int t = xcd_tile(b & 7, slots.slot()); t < ntiles;
         slots.next(), t = xcd_tile(b & 7, slots.slot())) {
        float gcur[4], gnext[4];
        load_run_g(Jp, g, t, (int)threadIdx.x, gcur);
        bwd_tile<T, DISP, NARROW>(Jp, t, want_ctrl, need_dv, gcur, false, Jp, g, t, gnext, g_img,
                                  g_disp, s_ctrl, lds_cells, fix_bits, acc, s_red, s_gmax);
    }

    if (want_ctrl)                         // the last tile ended with a barrier
        for (int e = threadIdx.x; e < nctrl; e += kThreads)
            ctrl_part[(int64_t)blockIdx.x * nctrl + e] = (double)s_ctrl[e];

    if (!partials)
        return;
    __shared__ double red[kThreads / 64][12];
    write_partial_row(acc, red, partials + (int64_t)blockIdx.x * 12);
}

// Batched adjoint: the groups of up to kBwdBatchMax jobs in one launch, the job
// table passed by value in the kernel arguments (no upload, nothing to
// allocate).  prefix[j] = first group of job j, prefix[njobs] = total;
// group_tiles[j] tiles each.  The FP64 parameter sums of group g of job j go to
// partials row j * kBwdMaxRows + g.
template <typename T, bool NARROW>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NARROW ? 4 : 3))) void
k_warp_bwd_batch(const BwdBatch B, double *__restrict__ partials, int32_t lds_cells)
{
    const int b = blockIdx.x;
    const int gi = xcd_tile<kGroupLog>(b & 7, b >> 3);
    if (gi >= B.prefix[B.njobs])
        return;
    int j = 0;                         // the job holding group gi (uniform)
    for (int i = 1; i < B.njobs; ++i)
        j += B.prefix[i] <= gi;
    __shared__ __attribute__((aligned(16))) int s_red[4][8];
    __shared__ __attribute__((aligned(16))) uint32_t s_gmax[kThreads / 64];
    __shared__ double red[kThreads / 64][12];
    double acc[12];
#pragma unroll
    for (int i = 0; i < 12; ++i)
        acc[i] = 0.0;
    const BwdJob &BJ = B.jobs[j];
    // B is the first kernel argument
    const JobPtr Jp = (JobPtr)((__attribute__((address_space(4))) const char *)
                                   __builtin_amdgcn_kernarg_segment_ptr() +
                               offsetof(BwdBatch, jobs) + j * sizeof(BwdJob) + offsetof(BwdJob, J));
    const int g = gi - B.prefix[j], nt = B.group_tiles[j];
    const int t1 = min((g + 1) * nt, Jp->tiles_x * Jp->tiles_y * Jp->tiles_z);
    float gcur[4];
    load_run_g(Jp, BJ.g, g * nt, (int)threadIdx.x, gcur);
    for (int t = g * nt; t < t1; ++t) {
        float gnext[4];
        bwd_tile<T, kDispNone, NARROW>(Jp, t, false, BJ.g_M != nullptr, gcur, t + 1 < t1, Jp, BJ.g,
                                       t + 1, gnext, BJ.g_img, nullptr, nullptr, lds_cells,
                                       B.fix_bits[j], acc, s_red, s_gmax);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            gcur[k] = gnext[k];
    }
    if (BJ.g_M)
        write_partial_row(acc, red, partials + ((int64_t)j * kBwdMaxRows + g) * 12);
}

// grad_M of job blockIdx.x: the rows of its groups summed in a fixed order (jobs
// without grad_M are skipped).
__global__ __launch_bounds__(kThreads) void k_reduce12_batch(const BwdBatch B,
                                                             const double *__restrict__ partials)
{
    double *out = B.jobs[blockIdx.x].g_M;
    if (!out)
        return;
    const int32_t nrows = B.prefix[blockIdx.x + 1] - B.prefix[blockIdx.x];
    const double *rows = partials + (int64_t)blockIdx.x * kBwdMaxRows * 12;
    double acc[12];
#pragma unroll
    for (int i = 0; i < 12; ++i)
        acc[i] = 0.0;
#pragma unroll 4
    for (int r = threadIdx.x; r < nrows; r += kThreads)   // loads issue ahead; sums keep their order
#pragma unroll
        for (int i = 0; i < 12; ++i)
            acc[i] += rows[(int64_t)r * 12 + i];
    __shared__ double red[kThreads / 64][12];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const double sum = wave_sum(acc[i]);
        if (lane == 63)
            red[wave][i] = sum;
    }
    __syncthreads();
    if (threadIdx.x < 12) {
        double sum = 0.0;
        for (int w = 0; w < kThreads / 64; ++w)
            sum += red[w][threadIdx.x];
        out[threadIdx.x] = sum;
    }
}

// Sum n rows of 12 doubles in a fixed order into out[12].
__global__ __launch_bounds__(kThreads) void k_reduce12(const double *__restrict__ partials,
                                                       int32_t n, double *__restrict__ out)
{
    double acc[12];
#pragma unroll
    for (int i = 0; i < 12; ++i)
        acc[i] = 0.0;

#pragma unroll 4
    for (int r = threadIdx.x; r < n; r += kThreads)   // loads issue ahead; sums keep their order
#pragma unroll
        for (int i = 0; i < 12; ++i)
            acc[i] += partials[(int64_t)r * 12 + i];
    __shared__ double red[kThreads / 64][12];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const double s = wave_sum(acc[i]);
        if (lane == 63)
            red[wave][i] = s;
    }
    __syncthreads();
    if (threadIdx.x < 12) {
        double s = 0.0;
        for (int w = 0; w < kThreads / 64; ++w)
            s += red[w][threadIdx.x];
        out[threadIdx.x] = s;
    }
}

// Control-grid rows, stage 1: group g (blockIdx.y) sums rows g*chunk ..
// (g+1)*chunk - 1 in order for 64 consecutive entries (one wave, coalesced).
__global__ __launch_bounds__(64) void k_reduce_ctrl_rows(const double *__restrict__ part,
                                                        int32_t rows, int32_t chunk, int32_t n,
                                                        double *__restrict__ groups)
{
    const int32_t e = blockIdx.x * 64 + threadIdx.x;
    if (e >= n)
        return;
    const int32_t r0 = blockIdx.y * chunk, r1 = min(r0 + chunk, rows);
    double s = 0.0;
#pragma unroll 8
    for (int32_t r = r0; r < r1; ++r)          // loads issue ahead; the sum keeps its order
        s += part[(int64_t)r * n + e];
    groups[(int64_t)blockIdx.y * n + e] = s;
}

// Stage 2: out[e] = sum over the groups in order (0 when there are none).
__global__ __launch_bounds__(kThreads) void k_reduce_ctrl_groups(const double *__restrict__ groups,
                                                                 int32_t ngroups, int32_t n,
                                                                 float *__restrict__ out)
{
    const int32_t e = blockIdx.x * kThreads + threadIdx.x;
    if (e >= n)
        return;
    double s = 0.0;
#pragma unroll 8
    for (int32_t g = 0; g < ngroups; ++g)      // loads issue ahead; the sum keeps its order
        s += groups[(int64_t)g * n + e];
    out[e] = (float)s;
}

int64_t ctrl_reduce_doubles(int64_t rows, int64_t nctrl)
{
    return (rows + std::min<int64_t>(rows, kCtrlRowGroups)) * nctrl;
}

static hipError_t reduce_ctrl(const double *part, int32_t rows, int32_t n, float *out,
                              hipStream_t s)
{
    const int32_t ngroups = std::min(rows, kCtrlRowGroups);
    const double *groups = part + (int64_t)rows * n;
    if (ngroups > 0) {
        const int32_t chunk = (rows + ngroups - 1) / ngroups;
        hipLaunchKernelGGL(k_reduce_ctrl_rows, dim3((n + 63) / 64, ngroups), dim3(64), 0, s, part,
                           rows, chunk, n, const_cast<double *>(groups));
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL(k_reduce_ctrl_groups, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0,
                       s, groups, ngroups, n, out);
    return hipGetLastError();
}

// Host replica of bs_index (the same single FP32 multiply and floor).
static int32_t host_bs_index(int64_t p, float inv_h, int32_t G)
{
    const float s = (float)p * inv_h;
    return (int32_t)std::fmin(std::floor(s), (float)(G - 4));
}

// Largest number of controls any tile of extent 2^l touches along one axis.
static int32_t max_window(int64_t n, int l, float inv_h, int32_t G)
{
    int32_t w = 0;
    for (int64_t p0 = 0; p0 < n; p0 += (int64_t)1 << l) {
        const int64_t p1 = std::min(p0 + ((int64_t)1 << l), n) - 1;
        w = std::max(w, host_bs_index(p1, inv_h, G) - host_bs_index(p0, inv_h, G) + 4);
    }
    return w;
}

bool bwd_spline_eval_ok(const BsplineGeom &B)
{
    return max_window(B.oz, kBwdTiling.lz, B.inv_hz, B.gz) <= kSplineWindow;
}

bool bwd_ctrl_fused(const BsplineGeom &B)
{
    if (3 * (int64_t)B.gx * B.gy * B.gz > kCtrlMaxEntries)
        return false;
    return bwd_spline_eval_ok(B) &&
           max_window(B.ox, kBwdTiling.lx, B.inv_hx, B.gx) <= kSplineWindow &&
           max_window(B.oy, kBwdTiling.ly, B.inv_hy, B.gy) <= kSplineWindow;
}

// Exponent b of the 32-bit fixed-point image adjoint of an affine job (see
// kFixed32MaxBits), or -1 for the 64-bit one.  Sample p reaches input cell c when
// q(p) = A p + t lies in [c - 1, c + 1) per axis, widened by the bound delta
// on q's FP32 rounding; those p lie in A^-1 of that cube, whose extent along
// output axis i is w_i = (2 + 2 delta) sum_j |A^-1_ij|, which holds at most
// floor(w_i) + 1 integer values of p_i, and the tile at most its extent.  A strongly shrinking or
// near-singular map exceeds kFixed32MaxBits and keeps 64-bit sums.
static int32_t fixed32_bits(const FwdJob &J)
{
    double a[3][3];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j)
            a[i][j] = (double)J.M[4 * i + j];
    double c[3][3];                    // cofactors
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            const int i1 = (i + 1) % 3, i2 = (i + 2) % 3, j1 = (j + 1) % 3, j2 = (j + 2) % 3;
            c[i][j] = a[i1][j1] * a[i2][j2] - a[i1][j2] * a[i2][j1];
        }
    const double det = a[0][0] * c[0][0] + a[0][1] * c[0][1] + a[0][2] * c[0][2];
    if (!std::isfinite(det) || det == 0.0)
        return -1;
    const double slack = std::max({(double)J.delta[0], (double)J.delta[1], (double)J.delta[2]});
    const int ext[3] = {1 << kBwdTiling.lx, 1 << kBwdTiling.ly, 1 << kBwdTiling.lz};
    int64_t K = 1;
    for (int i = 0; i < 3; ++i) {      // row i of A^-1 = column i of the cofactors / det
        const double w =
            (2.0 + 2.0 * slack) *
            (std::fabs(c[0][i]) + std::fabs(c[1][i]) + std::fabs(c[2][i])) / std::fabs(det);
        K *= (std::isfinite(w) && w < (double)ext[i])
                 ? std::min<int64_t>(ext[i], (int64_t)std::floor(w) + 1)
                 : ext[i];
    }
    int b = 0;
    while (((int64_t)1 << b) < K)
        ++b;
    return b <= kFixed32MaxBits ? b : -1;
}

// Workgroups the device keeps resident for kernel fn with lds bytes of dynamic
// LDS (occupancy x compute units), cached per device, kernel and LDS size.
static int resident_groups(const void *fn, size_t lds)
{
    // a fixed table (no heap allocation on the call path); when it is full
    // the occupancy is queried again on every call
    struct Entry {
        int dev;
        const void *fn;
        size_t lds;
        int groups;
    };
    constexpr int kEntries = 256;
    static std::mutex mu;
    static Entry cache[kEntries];
    static int used = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return 0;
    std::lock_guard<std::mutex> lock(mu);
    for (int i = 0; i < used; ++i)
        if (cache[i].dev == dev && cache[i].fn == fn && cache[i].lds == lds)
            return cache[i].groups;
    int cus = 0, occ = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, kThreads, lds) != hipSuccess)
        return 0;
    if (used < kEntries)
        cache[used++] = {dev, fn, lds, cus * occ};
    return cus * occ;
}

// Persistent grid: at most one wave of resident workgroups (a multiple of 8,
// as the XCD tile order assumes), at most the workspace's rows.
static int bwd_launch_grid(const void *fn, size_t lds, int64_t ntiles)
{
    const int64_t rows = bwd_grid(ntiles);
    const int resident = resident_groups(fn, lds) & ~7;
    return (int)(resident >= 8 ? std::min<int64_t>(rows, resident) : rows);
}

// Tiles of a group of an affine job of ntiles tiles, in a launch of total: fewer where
// the launch would not fill the device.
static int32_t group_size(int64_t ntiles, int64_t total)
{
    const int64_t want = std::min<int64_t>(kGroupTiles, std::max<int64_t>(1, total / kGroupFill));
    return (int32_t)std::max<int64_t>(want, (ntiles + kBwdMaxRows - 1) / kBwdMaxRows);
}

// Launches the adjoint of J; the rows of partials it writes.
template <int DISP>
static int launch_bwd_t(const FwdJob &J, int64_t ntiles, size_t lds, hipStream_t s,
                        const float *g, float *g_img, float *g_disp, double *part,
                        double *ctrl_part, int32_t cells)
{
    const int32_t fix_bits = DISP == kDispNone ? fixed32_bits(J) : -1;
    const int nt = (int)ntiles;
    const int32_t gt = group_size(ntiles, ntiles);
    int rows = 0;
    auto launch = [&](auto kern) {
        int grid;
        if (DISP == kDispNone) {
            rows = (int)((ntiles + gt - 1) / gt);
            grid = 8 * xcd_slots<kGroupLog>(rows);
        } else {
            grid = rows = bwd_launch_grid(reinterpret_cast<const void *>(kern), lds, ntiles);
        }
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, J, g, g_img, g_disp, part,
                           ctrl_part, nt, cells, fix_bits, gt);
    };
    if constexpr (DISP == kDispNone) {
        if (fix_bits >= 0) {
            if (J.dtype == kI16)
                launch(&k_warp_bwd<int16_t, DISP, true>);
            else
                launch(&k_warp_bwd<float, DISP, true>);
            return rows;
        }
    }
    if (J.dtype == kI16)
        launch(&k_warp_bwd<int16_t, DISP, false>);
    else
        launch(&k_warp_bwd<float, DISP, false>);
    return rows;
}

// LDS cells of an affine job's tiles (their window, set here); jobs whose window
// exceeds kBwdLdsMax, or has coordinates too large for one, take none and gather.
static int32_t affine_cells(FwdJob &J)
{
    const int32_t cells = set_window(J, kBwdTiling);
    if (cells > kBwdLdsMax)
        J.box_e[0] = 0;
    return J.box_e[0] != 0 ? cells : 64;
}

hipError_t launch_warp_bwd(const FwdJob &J0, const float *g, float *g_img, float *g_disp,
                           double *g_M, double *partials, double *ctrl_part, float *g_ctrl,
                           hipStream_t s)
{
    FwdJob J = J0;
    J.tiles_x = (J.ox + 7) >> 3;
    J.tiles_y = (J.oy + 7) >> 3;
    J.tiles_z = (J.oz + 15) >> 4;
    J.rcp_ty = rcp_u32((uint32_t)J.tiles_y);
    J.rcp_tz = rcp_u32((uint32_t)J.tiles_z);
    const int64_t ntiles = (int64_t)J.tiles_x * J.tiles_y * J.tiles_z;
    const int32_t nctrl = 3 * J.bs.gx * J.bs.gy * J.bs.gz;
    if (ntiles == 0) {
        if (g_ctrl && nctrl > 0) {     // no tiles, no rows: zeros
            hipError_t e = reduce_ctrl(ctrl_part, 0, nctrl, g_ctrl, s);
            if (e != hipSuccess)
                return e;
        }
        if (g_M) {
            hipLaunchKernelGGL(k_reduce12, dim3(1), dim3(kThreads), 0, s, partials, 0, g_M);
            return hipGetLastError();
        }
        return hipSuccess;
    }
    // LDS cells sized for the largest footprint of any tile (a displacement has
    // no a-priori bound: the full reservation, used when a tile fits it)
    const bool displaced = J.disp || J.ctrl;
    const int32_t cells = J.ctrl      ? kSplineBwdCells
                          : displaced ? kBwdLdsCells
                                      : affine_cells(J);
    const size_t lds = (size_t)(J.ctrl ? kBwdLdsCells : cells) * sizeof(float);
    double *part = g_M ? partials : nullptr;
    double *cpart = g_ctrl ? ctrl_part : nullptr;
    int grid;
    if (J.ctrl)
        grid = launch_bwd_t<kDispSpline>(J, ntiles, lds, s, g, g_img, g_disp, part, cpart, cells);
    else if (J.disp)
        grid = launch_bwd_t<kDispField>(J, ntiles, lds, s, g, g_img, g_disp, part, nullptr, cells);
    else
        grid = launch_bwd_t<kDispNone>(J, ntiles, lds, s, g, g_img, nullptr, part, nullptr, cells);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    if (cpart) {
        e = reduce_ctrl(cpart, grid, nctrl, g_ctrl, s);
        if (e != hipSuccess)
            return e;
    }
    if (!g_M)
        return hipSuccess;
    hipLaunchKernelGGL(k_reduce12, dim3(1), dim3(kThreads), 0, s, partials, grid, g_M);
    return hipGetLastError();
}

// Batched affine adjoint: chunks of up to kBwdBatchMax jobs, each one launch (its
// job table in the kernel arguments; every group of tiles writes its row) and
// one reduction launch.  partials: kBwdMaxRows * 12 doubles per job.
hipError_t launch_warp_bwd_batch(const BwdJob *jobs, int32_t n, double *partials, hipStream_t s)
{
    for (int32_t c0 = 0; c0 < n; c0 += kBwdBatchMax) {
        BwdBatch B;
        std::memset(&B, 0, sizeof B);
        B.njobs = std::min<int32_t>(kBwdBatchMax, n - c0);
        int64_t total = 0, all_tiles = 0;
        for (int i = 0; i < B.njobs; ++i) {
            const FwdJob &J = jobs[c0 + i].J;
            all_tiles += bwd_tiles(J.ox, J.oy, J.oz);
        }
        int32_t cells = 64;
        bool any_M = false;
        for (int i = 0; i < B.njobs; ++i) {
            B.jobs[i] = jobs[c0 + i];
            FwdJob &J = B.jobs[i].J;
            J.tiles_x = (J.ox + 7) >> 3;
            J.tiles_y = (J.oy + 7) >> 3;
            J.tiles_z = (J.oz + 15) >> 4;
            J.rcp_ty = rcp_u32((uint32_t)J.tiles_y);
            J.rcp_tz = rcp_u32((uint32_t)J.tiles_z);
            B.fix_bits[i] = fixed32_bits(J);
            const int64_t tiles = (int64_t)J.tiles_x * J.tiles_y * J.tiles_z;
            B.group_tiles[i] = group_size(tiles, all_tiles);
            B.prefix[i] = (int32_t)total;
            total += (tiles + B.group_tiles[i] - 1) / B.group_tiles[i];
            if (J.nx > 0 && J.ny > 0 && J.nz > 0 && J.ox > 0 && J.oy > 0 && J.oz > 0)
                cells = std::max(cells, affine_cells(J));
            any_M = any_M || B.jobs[i].g_M;
        }
        B.prefix[B.njobs] = (int32_t)total;
        double *part = partials ? partials + (int64_t)c0 * kBwdMaxRows * 12 : nullptr;
        const bool i16 = B.jobs[0].J.dtype == kI16;
        const size_t lds = (size_t)cells * sizeof(float);
        bool narrow = true;            // the 32-bit image adjoint when every job has a bound
        for (int i = 0; i < B.njobs; ++i)
            narrow = narrow && B.fix_bits[i] >= 0;
        using BatchKernel = void (*)(const BwdBatch, double *, int32_t);
        const BatchKernel kern =
            i16 ? (narrow ? &k_warp_bwd_batch<int16_t, true> : &k_warp_bwd_batch<int16_t, false>)
                : (narrow ? &k_warp_bwd_batch<float, true> : &k_warp_bwd_batch<float, false>);
        if (total > 0) {
            hipLaunchKernelGGL(kern, dim3((unsigned)(8 * xcd_slots<kGroupLog>((int)total))),
                               dim3(kThreads), lds, s, B, part, cells);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess)
                return e;
        }
        if (any_M) {
            hipLaunchKernelGGL(k_reduce12_batch, dim3(B.njobs), dim3(kThreads), 0, s, B, part);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess)
                return e;
        }
    }
    return hipSuccess;
}

}  // namespace ctaug
