// bspline.hip -- uniform cubic B-spline displacement field and its adjoint
// (gfx950).  Separable evaluation: for an output row (x, y) the x/y weights
// contract the control grid to a row profile P[comp][gz] once (in LDS), and
// each voxel then needs only its 4 z-weights and 12 FMAs.  The adjoint runs
// the same factorisation backwards (z in FP32 per row, then y and x in FP64,
// each in a fixed order), so the control-grid gradient is deterministic.
#include "bspline_eval.h"
#include "device_common.h"
#include "launch.h"

#include <algorithm>
#include <cmath>

namespace ctaug {

constexpr int kMaxG = 64;

// Upsampling, nrows (up to kUpRows) rows y of one x and zlen voxels of them per workgroup
// (a wave takes every fourth row).  The bound is writing the field, so what a voxel costs
// besides its 12 FMAs is shared: the rows' profiles are summed in one go, and a thread
// computes the cells and weights of its four z once for all its rows.  Neighbouring lanes
// take neighbouring z, so that rows of any extent are stored whole.  With four rows and
// four z in a row per lane: 117 x 130 x 151 in 16.3 us, now 10.4; 200 x 190 x 210 in 42,
// now 24; 256^3 42, now 39 (5.2 TB/s).  4 rows: 12, 29, 45; but four rows, and rows in
// parts, where whole rows by eight leave CUs idle (8 x 8 x 4000 18.5 us a call, now 8.0; 1 x 2000 x
// 2000 with 64^3 controls 16.6, now 13.8).
constexpr int kUpRows = 8;
constexpr int kUpBlocks = 1024;        // workgroups wanted: four per CU

__global__ __launch_bounds__(kThreads) void k_bspline_up(const float *__restrict__ ctrl,
                                                         BsplineGeom G, float *__restrict__ disp,
                                                         int nrows, int zlen)
{
    __shared__ float P[kUpRows][3][kMaxG];
    const int x = blockIdx.x;
    const int y0 = blockIdx.y * nrows;
    const int rows = min(nrows, G.oy - y0);
    const int64_t nvox = (int64_t)G.ox * G.oy * G.oz;

    for (int e = threadIdx.x; e < rows * 3 * G.gz; e += kThreads) {
        const int row = e / (3 * G.gz);
        const int rem = e - row * 3 * G.gz;
        const int comp = rem / G.gz, gz = rem - comp * G.gz;
        P[row][comp][gz] = bs_profile(ctrl, G, comp, x, y0 + row, gz);
    }
    __syncthreads();

    const int lane = threadIdx.x & 63;
    const int z0 = blockIdx.z * zlen, z1 = min(z0 + zlen, G.oz);
    for (int z = z0 + lane; z < z1; z += 256) {
        int32_t iz[4];
        float Bz[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float tz;
            bs_cell(min(z + 64 * k, G.oz - 1), G.inv_hz, G.gz, iz[k], tz);
            bs_basis(tz, Bz[k]);
        }
        for (int row = threadIdx.x >> 6; row < rows; row += kThreads / 64) {
            float *out = disp + (((int64_t)x * G.oy + y0 + row) * G.oz + z);
            float u[3][4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int comp = 0; comp < 3; ++comp) {
                    float s = 0.0f;
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        s = __builtin_fmaf(Bz[k][c], P[row][comp][iz[k] + c], s);
                    u[comp][k] = s;
                }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (z + 64 * k < z1)
#pragma unroll
                    for (int comp = 0; comp < 3; ++comp)
                        out[comp * nvox + 64 * k] = u[comp][k];
        }
    }
}

// Adjoint, z and y of one plane (component and x) per workgroup:
//   T1[y][gz] = sum_z B_{gz - iz(z)}(t(z)) g[y][z]      FP32
//   T2[gy][gz] = sum_y B_{gy - iy(y)}(t(y)) T1[y][gz]   FP64
// The bound is reading g once (coalesced, 64 bytes of a row per 4 lanes).  The
// z sums are a product of the rows with the weight matrix, so they run on the
// matrix cores in FP32 (16 rows x 16 controls x 4 voxels an instruction, one
// tile of 16 rows per wave): T1 of 64 rows goes to LDS, and each thread adds them
// to its entries of T2 in the order of y (few entries: 2 or 4 threads share one,
// each a part of every 64 rows, added in a fixed order at the end).  The weights
// come from LDS tables of the cell and the four weights of a position.  A row
// with a non-finite value is summed over its nonzero weights alone, as 0 times it
// would reach every control.  117 x 130 x 151, 8^3 controls, under the profiler: 31 us,
// where the two passes with one thread per row and per entry take 77 (z 47, y 30).
constexpr int kAdjRows = 64;           // rows of a chunk: 16 per wave
constexpr int kAdjSeg = 512;           // voxels along z whose weights are in LDS at once
constexpr int kAdjGridX = 65536;       // planes in the grid's first dimension (2^32 threads at most)

// CT: tiles of 16 controls along z.  NO: entries of T2 per thread.
template <int CT, int NO>
__global__ __launch_bounds__(kThreads) void k_bspline_adj_plane(const float *__restrict__ g,
                                                                BsplineGeom G,
                                                                double *__restrict__ T2, int vec,
                                                                int nsplit)
{
    constexpr int kPitch = CT * 16 + 1;
    __shared__ float s_t1[kAdjRows][kPitch];
    __shared__ float s_wz[kAdjSeg][4], s_wy[kAdjRows][4];
    __shared__ int s_iz[kAdjSeg], s_iy[kAdjRows];
    __shared__ double s_part[kThreads];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t p = (int64_t)blockIdx.y * kAdjGridX + blockIdx.x;        // comp * ox + x
    if (p >= 3 * (int64_t)G.ox)
        return;
    const float *plane = g + p * G.oy * G.oz;
    const int n2 = G.gy * G.gz, per = kThreads / nsplit;
    const int part = t / per, e0 = t - part * per;
    double acc[NO];
    int gy[NO], gz[NO];
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        const int e = e0 + i * per;
        acc[i] = 0.0;
        gy[i] = e < n2 ? e / G.gz : -4;            // no row reaches control -4
        gz[i] = e < n2 ? e - gy[i] * G.gz : 0;
    }
    const int r16 = lane & 15, kq = lane >> 4;     // row and voxel quad of the lane
    for (int yc = 0; yc < G.oy; yc += kAdjRows) {
        const int y = yc + 16 * wave + r16;
        const float *row = plane + (int64_t)min(y, G.oy - 1) * G.oz;
        f32x4 d[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c)
            d[c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        bool bad = false;
        for (int zs = 0; zs < G.oz; zs += kAdjSeg) {
            const int zn = min(kAdjSeg, G.oz - zs);
            __syncthreads();                       // the last chunk's T1 and tables are read
            if (yc == 0 || G.oz > kAdjSeg)
                for (int z = t; z < kAdjSeg; z += kThreads) {
                    float tz, B[4];
                    int32_t iz = 0;
                    bs_cell(min(zs + z, G.oz - 1), G.inv_hz, G.gz, iz, tz);
                    bs_basis(tz, B);
                    s_iz[z] = z < zn ? iz : -4;
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        s_wz[z][c] = B[c];
                }
            if (zs == 0 && t < kAdjRows) {
                float ty, B[4];
                int32_t iy = 0;
                bs_cell(min(yc + t, G.oy - 1), G.inv_hy, G.gy, iy, ty);
                bs_basis(ty, B);
                s_iy[t] = yc + t < G.oy ? iy : G.gy;           // no control reached
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    s_wy[t][c] = B[c];
            }
            __syncthreads();
            for (int zb = 0; zb < zn; zb += 16) {
                const int z = zs + zb + 4 * kq;
                float v[4];
                if (vec && z < G.oz) {
                    const f32x4 q = *reinterpret_cast<const f32x4 *>(row + z);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        v[j] = q[j];
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        v[j] = z + j < G.oz ? row[z + j] : 0.0f;
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    v[j] = y < G.oy ? v[j] : 0.0f;
                    bad = bad || !(fabsf(v[j]) <= 3.40282347e38f);
                    const int zt = zb + 4 * kq + j;            // < kAdjSeg
                    const int iz = s_iz[zt];
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        const int b = 16 * c + r16 - iz;       // control 16 c + r16
                        const float w = (uint32_t)b < 4u && iz >= 0 ? s_wz[zt][b & 3] : 0.0f;
                        d[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j], w, d[c], 0, 0, 0);
                    }
                }
            }
        }
        // lane: control 16 c + r16 of rows 4 kq + i of the wave's tile
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                s_t1[16 * wave + 4 * kq + i][16 * c + r16] = d[c][i];
        const uint64_t rows_bad = __ballot(bad);
        if (rows_bad) {                // rare: the wave's rows with such a value, one lane each
            const uint32_t rb = (uint32_t)(rows_bad | rows_bad >> 16 | rows_bad >> 32 |
                                           rows_bad >> 48) & 0xffffu;
            if (lane < 16 && (rb >> lane) & 1) {
                float *dst = s_t1[16 * wave + lane];
                for (int c = 0; c < G.gz; ++c)
                    dst[c] = 0.0f;
                for (int z = 0; z < G.oz; ++z) {
                    float tz, B[4];
                    int32_t iz;
                    bs_cell(z, G.inv_hz, G.gz, iz, tz);
                    bs_basis(tz, B);
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        dst[iz + c] = __builtin_fmaf(B[c], row[z], dst[iz + c]);
                }
            }
        }
        __syncthreads();
        const int nr = kAdjRows / nsplit;
        for (int r = part * nr; r < (part + 1) * nr; ++r) {
            const int iy = s_iy[r];
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                const int b = gy[i] - iy;
                if ((uint32_t)b < 4u)
                    acc[i] += (double)s_wy[r][b] * (double)s_t1[r][gz[i]];
            }
        }
    }
    double *out = T2 + p * n2;
    if (nsplit > 1) {                  // NO = 1
        s_part[t] = acc[0];
        __syncthreads();
        if (part == 0 && e0 < n2) {
            double s = s_part[e0];
            for (int p = 1; p < nsplit; ++p)
                s += s_part[p * per + e0];
            out[e0] = s;
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < NO; ++i)
        if (gy[i] >= 0)
            out[e0 + i * per] = acc[i];
}

// The same sums in two passes over memory, where a plane has too many rows or controls for
// one workgroup (bspline_adj_by_planes).  z: T1[comp][x][y][gz] = sum_z B_{gz - iz(z)}(t(z))
// g[comp][x][y][z], one thread per (comp, x, y) row streaming z with 16-byte loads when the
// rows are aligned.  The z-cell index is nondecreasing along the row, so the
// four controls a voxel touches slide as a window of four FP32 accumulators;
// each control's sum is stored once, when the window moves past it.
__global__ __launch_bounds__(kThreads) void k_bspline_adj_z(const float *__restrict__ g,
                                                            BsplineGeom G, float *__restrict__ T1,
                                                            int vec)
{
    const int64_t nrows = 3 * (int64_t)G.ox * G.oy;
    const int64_t row = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (row >= nrows)
        return;
    const float *src = g + row * G.oz;
    float *dst = T1 + row * G.gz;
    float w[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int32_t cur = 0;
    auto add = [&](int z, float v) {
        int32_t iz;
        float tz, Bz[4];
        bs_cell(z, G.inv_hz, G.gz, iz, tz);
        while (cur < iz) {             // controls below iz are complete
            dst[cur] = w[0];
            w[0] = w[1];
            w[1] = w[2];
            w[2] = w[3];
            w[3] = 0.0f;
            ++cur;
        }
        bs_basis(tz, Bz);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            w[c] = __builtin_fmaf(Bz[c], v, w[c]);
    };
    if (vec) {
        for (int z = 0; z < G.oz; z += 4) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(src + z);
            add(z, v.x);
            add(z + 1, v.y);
            add(z + 2, v.z);
            add(z + 3, v.w);
        }
    } else {
        for (int z = 0; z < G.oz; ++z)
            add(z, src[z]);
    }
    for (int c = 0; c < 4; ++c)
        dst[cur + c] = w[c];
    for (int gz = cur + 4; gz < G.gz; ++gz)
        dst[gz] = 0.0f;
}

// y: T2[comp][x][gy][gz] = sum_y B_{gy - iy(y)}(t(y)) T1[comp][x][y][gz], FP64,
// one thread per output, y in a fixed order.
__global__ __launch_bounds__(kThreads) void k_bspline_adj_y(const float *__restrict__ T1,
                                                            BsplineGeom G, double *__restrict__ T2)
{
    const int64_t total = 3 * (int64_t)G.ox * G.gy * G.gz;
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e >= total)
        return;
    const int gz = (int)(e % G.gz);
    const int gy = (int)((e / G.gz) % G.gy);
    const int64_t cx = e / ((int64_t)G.gz * G.gy);          // comp * ox + x
    // rows y whose cell reaches control gy: iy in [gy - 3, gy]
    double s = 0.0;
    for (int y = 0; y < G.oy; ++y) {
        int32_t iy;
        float ty, By[4];
        bs_cell(y, G.inv_hy, G.gy, iy, ty);
        const int b = gy - iy;
        if (b < 0 || b > 3)
            continue;
        bs_basis(ty, By);
        s += (double)By[b] * (double)T1[(cx * G.oy + y) * G.gz + gz];
    }
    T2[e] = s;
}

// grad_ctrl[comp][gx][gy][gz] = sum_x B_{gx - ix(x)}(t(x)) T2[comp][x][gy][gz], FP64: blocks
// of control plane comp * Gx + gx.  SPLIT: 64 entries a block; each wave sums a quarter of
// the planes that reach gx, in order, and the quarters are added in order (one thread per
// entry took 27 us for 117 planes, waiting for each load).  Otherwise 256 entries, all
// planes in order: up to 16 of them are in flight at once, and the quarters would cost
// more than they save (4 to 30 planes with 64^3 controls: 4 to 12 % slower).
constexpr int kAdjSplitPlanes = 16;

template <bool SPLIT>
__global__ __launch_bounds__(kThreads) void k_bspline_adj_x(const double *__restrict__ T2,
                                                            BsplineGeom G,
                                                            float *__restrict__ grad_ctrl)
{
    const int n2 = G.gy * G.gz;
    const int comp = blockIdx.x / G.gx, gx = blockIdx.x - comp * G.gx;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int e = SPLIT ? blockIdx.y * 64 + lane : blockIdx.y * kThreads + threadIdx.x;
    // planes x0 .. x1 - 1 hold every x with 0 <= gx - ix(x) <= 3: ix does not decrease,
    // and the estimate, ix's own product and a plane number past 2^24 are each rounded by
    // less than 2^-23 of ox
    int x0 = 0, x1 = G.ox;
    if (G.inv_hx > 0.0f) {
        const float h = 1.0f / G.inv_hx, n = (float)G.ox, spare = 3.0f + n * 0x1p-21f;
        x0 = min((int)fminf(fmaxf((float)(gx - 3) * h - spare, 0.0f), n), G.ox);
        if (gx < G.gx - 4)
            x1 = min((int)fminf((float)(gx + 1) * h + spare, n), G.ox);
    }
    const int quarter = SPLIT ? (max(x1 - x0, 0) + 3) >> 2 : 0;
    const int xa = SPLIT ? x0 + wave * quarter : x0, xb = SPLIT ? min(xa + quarter, x1) : x1;
    const double *src = T2 + (int64_t)comp * G.ox * n2 + min(e, n2 - 1);
    double s = 0.0;
#pragma unroll 8
    for (int x = xa; x < xb; ++x) {    // loads issue ahead; the sum keeps its order
        int32_t ix;
        float tx, Bx[4];
        bs_cell(x, G.inv_hx, G.gx, ix, tx);
        bs_basis(tx, Bx);
        const int a = gx - ix;
        const float w = a == 0 ? Bx[0] : a == 1 ? Bx[1] : a == 2 ? Bx[2] : Bx[3];
        const double v = src[(int64_t)x * n2];
        s = (uint32_t)a < 4u ? s + (double)w * v : s;
    }
    if constexpr (SPLIT) {
        __shared__ double s_part[kThreads / 64][64];
        s_part[wave][lane] = s;
        __syncthreads();
        if (wave == 0 && e < n2)
            grad_ctrl[(int64_t)blockIdx.x * n2 + e] =
                (float)(((s_part[0][lane] + s_part[1][lane]) + s_part[2][lane]) + s_part[3][lane]);
    } else if (e < n2) {
        grad_ctrl[(int64_t)blockIdx.x * n2 + e] = (float)s;
    }
}

int bspline_max_grid() { return kMaxG; }

// Workspace of the adjoint: T1 (FP32, 3 x ox x oy x Gz; the passes' alone), then T2 (FP64,
// 3 x ox x Gy x Gz) at a 256-byte aligned offset.
static int64_t adj_t1_bytes(const int64_t od[3], const int64_t G[3])
{
    return ((3 * od[0] * od[1] * G[2] * (int64_t)sizeof(float)) + 255) & ~(int64_t)255;
}

int64_t bspline_adj_ws_bytes(const int64_t od[3], const int64_t G[3])
{
    return adj_t1_bytes(od, G) + 3 * od[0] * G[1] * G[2] * (int64_t)sizeof(double);
}

hipError_t launch_bspline_up(const float *ctrl, const int64_t G[3], const int64_t od[3],
                             float *disp, hipStream_t s)
{
    if (od[0] == 0 || od[1] == 0 || od[2] == 0)
        return hipSuccess;
    const BsplineGeom g = bspline_geom(G, od);
    // x and y apart: together they can pass 2^32 threads in a dimension
    const int64_t by8 = od[0] * ((od[1] + kUpRows - 1) / kUpRows);
    const int nrows = by8 <= kUpBlocks ? kUpRows / 2 : kUpRows;
    const int64_t ny = (od[1] + nrows - 1) / nrows, runs = (od[2] + 255) / 256;
    const int64_t nz = std::min(runs, std::max<int64_t>(1, kUpBlocks / (od[0] * ny)));
    const int64_t zlen = 256 * ((runs + nz - 1) / nz);
    const dim3 grid((unsigned)od[0], (unsigned)ny, (unsigned)((od[2] + zlen - 1) / zlen));
    hipLaunchKernelGGL(k_bspline_up, grid, dim3(kThreads), 0, s, ctrl, g, disp, nrows,
                       (int)zlen);
    return hipGetLastError();
}

// Whether the z and y sums go plane by plane (k_bspline_adj_plane) or in a pass each.  A
// plane's workgroup walks 64 rows at a time, 16 voxels a step, then adds these rows to
// its entries one after the other, so its time grows with the plane and the grid,
// whatever else is idle; the passes take every row and every entry at once, but read
// and write the field's rows singly.  Estimates in us, fitted to 430 pairs of 33 fields
// (20^3 to 256^3, 20000 x 1 x 4 to 1 x 2000 x 2000) and 13 grids, of which they choose the
// slower one by more than 7 % in three.  Passes against planes, measured: 128^3 with 8^3
// controls 55 / 28, 16^3 45 / 32, 32^3 47 / 53, 64^3 108 / 119; 16 x 512 x 512 with 8^3
// 150 / 153, 32^3 105 / 375; 1 x 2000 x 2000 with 8^3 549 / 2530; 8 x 8 x 4000 with 8^3
// 300 / 110; 512 x 512 x 64 with 32^3 618 / 302.
bool bspline_adj_by_planes(const BsplineGeom &g, bool vec)
{
    const double planes = 3.0 * g.ox, n2 = (double)g.gy * g.gz;
    const double rows = n2 <= 64 ? 16.0 : n2 <= 128 ? 32.0 : 64.0;     // per thread of a chunk
    const double entry = n2 > 4 * kThreads                        ? 0.77
                         : g.gz > 16 || n2 > (double)kThreads ? 0.17
                                                              : 0.08;
    const double chunk = std::ceil(g.oz / 16.0) * (g.gz > 16 ? 0.9 : 0.52) + rows * entry;
    const double by_planes = std::ceil(g.oy / (double)kAdjRows) * chunk *
                             std::pow(std::max(1.0, planes / 900.0), 0.75);
    const double z = std::max(g.oz * (vec ? 0.086 : 0.18),
                              planes * g.oy * g.oz * (vec ? 1.7e-6 : 5.6e-6));
    const double y = g.oy * (0.045 + 0.20 * std::min(1.0, 4.0 / (g.gy - 3))) +
                     planes * n2 * g.oy * 0.17e-6;
    return by_planes <= z + y + 3.4;
}

hipError_t launch_bspline_adj(const float *grad_disp, const int64_t od[3], const int64_t G[3],
                              float *grad_ctrl, double *ws, hipStream_t s)
{
    BsplineGeom g = bspline_geom(G, od);
    if (od[0] == 0 || od[1] == 0 || od[2] == 0)
        g.ox = 0;                      // no voxels: every control gradient is 0
    const int n2 = g.gy * g.gz;
    float *T1 = reinterpret_cast<float *>(ws);
    double *T2 = reinterpret_cast<double *>(reinterpret_cast<char *>(ws) + adj_t1_bytes(od, G));
    if (g.ox > 0) {
        const bool vec = od[2] % 4 == 0 && (reinterpret_cast<uintptr_t>(grad_disp) & 15u) == 0;
        const int64_t planes = 3 * od[0];
        if (bspline_adj_by_planes(g, vec)) {
            const int nsplit = n2 <= 64 ? 4 : n2 <= 128 ? 2 : 1;
            const dim3 grid((unsigned)std::min<int64_t>(planes, kAdjGridX),
                            (unsigned)((planes + kAdjGridX - 1) / kAdjGridX));
            auto launch = [&](auto kern) {
                hipLaunchKernelGGL(kern, grid, dim3(kThreads), 0, s, grad_disp, g, T2, vec ? 1 : 0,
                                   nsplit);
            };
            if (g.gz <= 16) {
                if (n2 <= kThreads)
                    launch(&k_bspline_adj_plane<1, 1>);
                else
                    launch(&k_bspline_adj_plane<1, 4>);        // at most 64 x 16
            } else if (n2 <= 4 * kThreads) {
                launch(&k_bspline_adj_plane<4, 4>);
            } else {
                launch(&k_bspline_adj_plane<4, 16>);
            }
        } else {
            auto blocks = [](int64_t n) { return dim3((unsigned)((n + kThreads - 1) / kThreads)); };
            hipLaunchKernelGGL(k_bspline_adj_z, blocks(planes * od[1]), dim3(kThreads), 0, s,
                               grad_disp, g, T1, vec ? 1 : 0);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess)
                return e;
            hipLaunchKernelGGL(k_bspline_adj_y, blocks(planes * n2), dim3(kThreads), 0, s, T1, g,
                               T2);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    // planes that reach a control: its four cells' of h
    const double reach = std::min((double)g.ox, 4.0 * g.ox / (g.gx - 3) + 2.0);
    const bool split = reach > kAdjSplitPlanes;
    const int per = split ? 64 : kThreads;
    hipLaunchKernelGGL(split ? &k_bspline_adj_x<true> : &k_bspline_adj_x<false>,
                       dim3((unsigned)(3 * g.gx), (unsigned)((n2 + per - 1) / per)),
                       dim3(kThreads), 0, s, T2, g, grad_ctrl);
    return hipGetLastError();
}

}  // namespace ctaug
