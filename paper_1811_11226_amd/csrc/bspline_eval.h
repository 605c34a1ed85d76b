// bspline_eval.h -- evaluation of the uniform cubic B-spline displacement
// field (internal), shared by the upsampling kernel, the fused warp and the
// fused adjoint so that every path computes the same bits.
//
// Control j of an axis with n output voxels and G controls sits at output
// coordinate (j - 1) h with h = (n - 1) / (G - 3); output voxel p lies in cell
// i = min(floor(p / h), G - 4) at fraction t = p / h - i and takes
//   u(p) = sum_{a,b,c} B_a(t_x) B_b(t_y) B_c(t_z) C[i_x + a][i_y + b][i_z + c]
// with the uniform cubic B-spline basis B_0..B_3.  Order of operations (FP32,
// every multiply-add fused and written out): the row profile
//   P(x, y, gz) = sum_a B_a(t_x) (sum_b B_b(t_y) C[i_x + a][i_y + b][gz])
// accumulated b = 0..3 inside a = 0..3, then u = sum_c B_c(t_z) P(x, y, i_z + c)
// accumulated c = 0..3.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ctaug {

struct BsplineGeom {
    int32_t ox, oy, oz;                // output (field) dims
    int32_t gx, gy, gz;                // control grid dims, each >= 4
    float inv_hx, inv_hy, inv_hz;      // (G - 3) / (n - 1), or 0 when n == 1
};

// Cell index and fraction of output coordinate p on one axis.
__device__ __forceinline__ void bs_cell(int32_t p, float inv_h, int32_t G, int32_t &i, float &t)
{
    const float s = (float)p * inv_h;
    const float f = fminf(floorf(s), (float)(G - 4));
    i = (int32_t)f;
    t = s - f;
}

__device__ __forceinline__ int32_t bs_index(int32_t p, float inv_h, int32_t G)
{
    return (int32_t)fminf(floorf((float)p * inv_h), (float)(G - 4));
}

__device__ __forceinline__ void bs_basis(float t, float B[4])
{
    const float t2 = t * t, t3 = t2 * t, m = 1.0f - t;
    const float sixth = 1.0f / 6.0f;
    B[0] = m * m * m * sixth;
    B[1] = __builtin_fmaf(3.0f, t3, __builtin_fmaf(-6.0f, t2, 4.0f)) * sixth;
    B[2] = __builtin_fmaf(-3.0f, t3, __builtin_fmaf(3.0f, t2, __builtin_fmaf(3.0f, t, 1.0f))) * sixth;
    B[3] = t3 * sixth;
}

// Row profile P(x, y, gz) of component comp (control layout [3][gx][gy][gz]).
// SLIM: four loads in flight instead of sixteen (registers).
template <bool SLIM = false>
__device__ __forceinline__ float bs_profile(const float *__restrict__ ctrl, const BsplineGeom &G,
                                            int comp, int32_t x, int32_t y, int32_t gz)
{
    int32_t ix, iy;
    float tx, ty, Bx[4], By[4];
    bs_cell(x, G.inv_hx, G.gx, ix, tx);
    bs_basis(tx, Bx);
    bs_cell(y, G.inv_hy, G.gy, iy, ty);
    bs_basis(ty, By);
    const int64_t gstride = (int64_t)G.gx * G.gy * G.gz;
    float s = 0.0f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        float sa = 0.0f;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            sa = __builtin_fmaf(By[b],
                                ctrl[comp * gstride + ((int64_t)(ix + a) * G.gy + (iy + b)) * G.gz + gz],
                                sa);
        s = __builtin_fmaf(Bx[a], sa, s);
        if (SLIM)
            __builtin_amdgcn_sched_barrier(0);
    }
    return s;
}

// Displacement of one thread's run of a tile of 8 x 8 rows (x, y) by 16 voxels
// along z, evaluated from the control grid by a workgroup of 256 threads:
// thread tid has row tid >> 2 (x = x0 + (row >> 3), y = y0 + (row & 7)) and the voxels z + k
// zstep, k < nvalid, of the tile (z1 - z0 < 16).  With at most kSplineWindow
// controls per axis in the tile's window, the sums of bs_profile are shared: the
// window C[a][b][c] and the weights of the tile's 8 + 8 + 16 positions go to LDS,
// then
//   S[a][y][c] = sum_b B_b(y) C[a][b][c],  P[x][y][c] = sum_a B_a(x) S[a][y][c]
// and each thread contracts c for its own voxels (the fmaf chains of bs_profile
// in the same order, so the same bits).  Lane = 8 (b or y) + c throughout and a
// wave takes one (a or x, component) at a time, so that every address is the
// lane plus a scalar and no index is divided (most of the 322 VALU instructions
// per voxel of the 256^3 warp were such divisions; it went from 185 to 160 us).  Wider windows along x or y take the profiles
// one by one; along z (controls closer than about 4 voxels) every voxel its own when PER_VOXEL
// is set; without it the caller guarantees that every z window fits.  s_prof:
// kSplineTileLdsFloats floats of LDS, 16-byte aligned.  Contains workgroup
// barriers: every thread of the workgroup calls it.
constexpr int kSplineWindow = 8;
constexpr int kSplineTileLdsFloats = 3 * 3 * kSplineWindow * 64 + 32 * 4 + 32;

template <bool PER_VOXEL = true>
__device__ __forceinline__ void spline_tile_u(const float *__restrict__ ctrl, const BsplineGeom &B,
                                              int x0, int y0, int z0, int x1, int y1, int z1,
                                              int x, int y, int z, int zstep, int nvalid,
                                              bool mine, int tid, float *s_prof, float (&u)[3][4])
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    float *Wc = s_prof;                            // [a][comp][b][c]
    float *S = Wc + 3 * kSplineWindow * 64;        // [a][comp][y][c]
    float *P = S + 3 * kSplineWindow * 64;         // [x][comp][y][c]
    f32x4 *T = reinterpret_cast<f32x4 *>(P + 3 * 8 * 64);  // weights: 8 x, 8 y, 16 z
    int *I = reinterpret_cast<int *>(T + 32);      // their cells, from the window's first
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // position pos of the 32: its cell in lane pos (and pos + 32) of every wave
    const int pos = lane & 31;
    const bool ax = pos < 8, ay = pos < 16;
    const int p = min((ax ? x0 : ay ? y0 - 8 : z0 - 16) + pos, ax ? x1 : ay ? y1 : z1);
    int32_t ci;
    float ct;
    bs_cell(p, ax ? B.inv_hx : ay ? B.inv_hy : B.inv_hz, ax ? B.gx : ay ? B.gy : B.gz, ci, ct);
    const int ixl = __builtin_amdgcn_readlane(ci, 0), iyl = __builtin_amdgcn_readlane(ci, 8),
              izl = __builtin_amdgcn_readlane(ci, 16);
    const int ncx = __builtin_amdgcn_readlane(ci, 7) - ixl + 4,
              ncy = __builtin_amdgcn_readlane(ci, 15) - iyl + 4,
              ncz = __builtin_amdgcn_readlane(ci, 31) - izl + 4;
    if (!PER_VOXEL || ncz <= kSplineWindow) {
        if (wave == 0 && lane < 32) {
            float Bw[4];
            bs_basis(ct, Bw);
            T[lane] = f32x4{Bw[0], Bw[1], Bw[2], Bw[3]};
            I[lane] = ci - (ax ? ixl : ay ? iyl : izl);
        }
        const int64_t gstride = (int64_t)B.gx * B.gy * B.gz;
        const int c = lane & 7, yr = lane >> 3;
        if (ncx <= kSplineWindow && ncy <= kSplineWindow) {
            if (c < ncz && yr < ncy) {
                const int32_t e = (iyl + yr) * B.gz + izl + c;
                for (int ac = wave; ac < 3 * ncx; ac += 4) {
                    const int a = ac / 3, comp = ac - 3 * a;
                    Wc[ac * 64 + lane] =
                        ctrl[comp * gstride + (int64_t)(ixl + a) * B.gy * B.gz + e];
                }
            }
            __syncthreads();
            {
                const f32x4 By = T[8 + yr];
                const float *w = Wc + I[8 + yr] * 8 + c;
                for (int ac = wave; ac < 3 * ncx; ac += 4) {
                    float sa = 0.0f;
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        sa = __builtin_fmaf(By[b], w[ac * 64 + b * 8], sa);
                    S[ac * 64 + lane] = sa;
                }
            }
            __syncthreads();
            for (int xr = wave; xr < 8; xr += 4) {
                const f32x4 Bx = T[xr];
                const float *sp = S + I[xr] * (3 * 64) + lane;
#pragma unroll
                for (int comp = 0; comp < 3; ++comp) {
                    float sv = 0.0f;
#pragma unroll
                    for (int a = 0; a < 4; ++a)
                        sv = __builtin_fmaf(Bx[a], sp[(3 * a + comp) * 64], sv);
                    P[(xr * 3 + comp) * 64 + lane] = sv;
                }
            }
        } else if (c < ncz) {
#pragma unroll 1
            for (int xc = wave; xc < 24; xc += 4)
                P[xc * 64 + lane] = bs_profile<true>(ctrl, B, xc % 3, min(x0 + xc / 3, x1),
                                               min(y0 + yr, y1), izl + c);
        }
        __syncthreads();
        if (!mine)
            return;
        const int row = tid >> 2;
        const float *pr = P + (row >> 3) * (3 * 64) + (row & 7) * 8;
        f32x4 Bz[4];
        int iz[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int e = 16 + min(z - z0 + k * zstep, 15);
            Bz[k] = T[e];
            iz[k] = I[e];
        }
        if (__all(iz[0] == iz[3])) {   // cells do not decrease along z: one for all four
#pragma unroll
            for (int comp = 0; comp < 3; ++comp) {
                float v[4];
#pragma unroll
                for (int cc = 0; cc < 4; ++cc)
                    v[cc] = pr[comp * 64 + iz[0] + cc];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float s = 0.0f;
#pragma unroll
                    for (int cc = 0; cc < 4; ++cc)
                        s = __builtin_fmaf(Bz[k][cc], v[cc], s);
                    u[comp][k] = s;
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int comp = 0; comp < 3; ++comp) {
                    float s = 0.0f;
#pragma unroll
                    for (int cc = 0; cc < 4; ++cc)
                        s = __builtin_fmaf(Bz[k][cc], pr[comp * 64 + iz[k] + cc], s);
                    u[comp][k] = s;
                }
        }
    } else if (PER_VOXEL && mine) {
#pragma unroll 1
        for (int k = 0; k < nvalid; ++k) {
            int32_t iz;
            float tz, Bz[4];
            bs_cell(z + k * zstep, B.inv_hz, B.gz, iz, tz);
            bs_basis(tz, Bz);
#pragma unroll
            for (int comp = 0; comp < 3; ++comp) {
                float s = 0.0f;
#pragma unroll 1
                for (int c = 0; c < 4; ++c) {
                    const float bz = c == 0 ? Bz[0] : c == 1 ? Bz[1] : c == 2 ? Bz[2] : Bz[3];
                    s = __builtin_fmaf(bz, bs_profile<true>(ctrl, B, comp, x, y, iz + c), s);
                }
                u[comp][k] = s;
            }
        }
    }
}

// Host: geometry of a control grid G over output dims od.
inline BsplineGeom bspline_geom(const int64_t G[3], const int64_t od[3])
{
    BsplineGeom g;
    g.ox = (int32_t)od[0];
    g.oy = (int32_t)od[1];
    g.oz = (int32_t)od[2];
    g.gx = (int32_t)G[0];
    g.gy = (int32_t)G[1];
    g.gz = (int32_t)G[2];
    g.inv_hx = od[0] > 1 ? (float)((double)(G[0] - 3) / (double)(od[0] - 1)) : 0.0f;
    g.inv_hy = od[1] > 1 ? (float)((double)(G[1] - 3) / (double)(od[1] - 1)) : 0.0f;
    g.inv_hz = od[2] > 1 ? (float)((double)(G[2] - 3) / (double)(od[2] - 1)) : 0.0f;
    return g;
}

}  // namespace ctaug
