// smooth.hip -- separable Gaussian smoothing of the resampling pre-step
// (gfx950).  Each axis is acc = w0 v, then acc = fma(w_d, v(-d) + v(+d), acc)
// for d = 1 .. R, x first, then y, then z, with edge voxels repeated beyond
// the volume; FP32 with weights normalised on the host in FP64.  One fused pass
// (k_smooth_fused) where the radii and the volume's size allow and pay for it
// (smooth_fused_ok), else a pass per axis (k_smooth_axis); both evaluate the same
// chains, so the results are the same bits.
#include "device_common.h"
#include "launch.h"

#include <algorithm>
#include <cmath>

namespace ctaug {

// One pass over one axis, one thread per output voxel: the 2R+1 taps come from
// L1/L2 (neighbouring threads share them).  For radii past kFusedMaxR and small
// volumes (smooth_fused_ok): reading and writing the volume once per axis took 1.29
// ms for a 512 x 512 x 320 int16 scan smoothed along all three axes.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_smooth_axis(const T *__restrict__ in,
                                                          float *__restrict__ out, int32_t nx,
                                                          int32_t ny, int32_t nz, int32_t axis,
                                                          GaussTaps K)
{
    const int z = blockIdx.x * kThreads + threadIdx.x;
    const int y = blockIdx.y, x = blockIdx.z;
    if (z >= nz)
        return;
    const int32_t e = (x * ny + y) * nz + z;
    const int i = axis == 0 ? x : axis == 1 ? y : z;
    const int n = axis == 0 ? nx : axis == 1 ? ny : nz;
    const int32_t stride = axis == 0 ? ny * nz : axis == 1 ? nz : 1;
    float acc = K.w[0] * (float)in[e];
    for (int d = 1; d <= K.R; ++d) {
        const int lo = max(i - d, 0) - i, hi = min(i + d, n - 1) - i;
        acc = __builtin_fmaf(K.w[d], (float)in[e + lo * stride] + (float)in[e + hi * stride], acc);
    }
    out[e] = acc;
}

// All three axes in one pass.  The bound is the volume's own traffic (input read
// once, output written once), so nothing else goes to memory:
//  - a workgroup of 8 waves takes 8 kRowsOut output rows (y) of one z segment and
//    walks along x; lane l holds the two voxels z = zs + 2 (l - H), + 1 of every
//    row its wave loads, H lanes at either end being the z halo;
//  - x: each wave keeps the 2 RM + 1 last planes of its rows in registers (a ring
//    indexed at compile time, the x loop unrolled over it), the next plane's
//    loads in flight while this one is used;
//  - y: the x-smoothed rows meet in LDS (two buffers, one barrier per plane); a
//    wave takes kRowsOut consecutive output rows, so kRowsOut + 2 RM rows are read
//    for kRowsOut results;
//  - z: neighbours come from the lanes beside (DPP wave shifts).
// A wait for the next plane's loads has to pass over the stores issued after them:
// with branches around the stores it waited for those as well, once a plane, and
// with a load per voxel (512 x 512 x 320 int16 scan: 190 us; 126 now, 4.0 TB/s).
// Rows, planes and lanes beyond the volume hold the edge voxel (their loads are
// clamped), which is what each axis repeats there.  Rows of 120 or 124 voxels per
// wave fit ordinary z extents better than 4 voxels a lane would.
constexpr int kFusedMaxR = 4;
constexpr int kFusedWaves = 8;
constexpr int kRowsOut = 4;

struct FusedTaps {
    int32_t R[3];
    float w[3][kFusedMaxR + 1];
};

// v of the lane before (shift -1) or after (+1); the end lanes keep their own.
__device__ __forceinline__ float lane_before(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x138,
                                                      0xF, 0xF, false));
}
__device__ __forceinline__ float lane_after(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x130,
                                                      0xF, 0xF, false));
}

// nyt row tiles, nzs z segments of zlen (even) outputs, x chunks of cx planes; block
// (chunk * nyt + row tile) * nzs + segment.  PAIR: nz is even and a lane's two voxels
// are aligned, in both volumes.
template <typename T, int RM, bool PAIR>
__global__ __launch_bounds__(64 * kFusedWaves) void k_smooth_fused(
    const T *__restrict__ in, float *__restrict__ out, int32_t nx, int32_t ny, int32_t nz,
    int32_t nyt, int32_t nzs, int32_t zlen, int32_t cx, FusedTaps K)
{
    constexpr int P = 2 * RM + 1;                  // planes in the ring
    constexpr int H = (RM + 1) / 2;                // halo lanes at either end
    constexpr int RT = kFusedWaves * kRowsOut + 2 * RM;        // rows of a plane in LDS
    constexpr int NR = (RT + kFusedWaves - 1) / kFusedWaves;   // rows a wave loads
    __shared__ float2 s_rows[2][RT][64];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int zs = (blockIdx.x % nzs) * zlen;
    const int by = blockIdx.x / nzs;
    const int y0 = (by % nyt) * (kFusedWaves * kRowsOut);
    const int x0 = (by / nyt) * cx, x1 = min(x0 + cx, nx);
    const int z = zs + 2 * (lane - H);
    // PAIR: both voxels in one load, moved inside at the ends (nz is even, z too)
    const uint32_t za = min(max(z, 0), PAIR ? nz - 2 : nz - 1) * (int)sizeof(T),
                   zb = min(max(z + 1, 0), nz - 1) * (int)sizeof(T);
    const bool before = z < 0, past = z >= nz;
    const uint32_t bytes_in = (uint32_t)(ny * nz) * (uint32_t)sizeof(T);
    // A lane's stores, one per output row: past the end of the plane's buffer (they are
    // dropped) where there is nothing to store, so that every path through the x loop
    // issues the same ones and a wait for a load passes over them.
    const bool mine = lane >= H && lane < 64 - H && z < min(zs + zlen, nz);
    const uint32_t bytes_out = (uint32_t)(ny * nz) * 4u;
    uint32_t oz[kRowsOut];
#pragma unroll
    for (int j = 0; j < kRowsOut; ++j) {
        const int y = y0 + wave * kRowsOut + j;
        oz[j] = mine && y < ny ? 4u * (uint32_t)(y * nz + z) : bytes_out;
    }

    // row i of the wave is row y0 - RM + wave + 8 i of the plane (a byte offset)
    int32_t row[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i)
        row[i] = min(max(y0 - RM + wave + kFusedWaves * i, 0), ny - 1) * nz * (int)sizeof(T);
    typedef T pair_t __attribute__((ext_vector_type(2)));
    pair_t next[NR];
    auto fetch = [&](int x) {
        const rsrc_t plane = make_rsrc(in + (int64_t)min(max(x, 0), nx - 1) * ny * nz, bytes_in);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if constexpr (PAIR && sizeof(T) == 2) {
                next[i] = __builtin_bit_cast(
                    pair_t, __builtin_amdgcn_raw_buffer_load_b32(plane, za, row[i], 0));
            } else if constexpr (PAIR) {
                next[i] = __builtin_bit_cast(
                    pair_t, __builtin_amdgcn_raw_buffer_load_b64(plane, za, row[i], 0));
            } else {
                next[i][0] = Elem<T>::raw(plane, za, row[i]);
                next[i][1] = Elem<T>::raw(plane, zb, row[i]);
            }
        }
    };
    auto place = [&](float (&r)[2], const pair_t &n) {
        const float a = (float)n[0], b = (float)n[1];
        r[0] = PAIR && past ? b : a;
        r[1] = PAIR && before ? a : b;
    };
    float ring[P][NR][2];
#pragma unroll
    for (int p = 0; p < P - 1; ++p) {              // planes x0 - RM .. x0 + RM - 1
        fetch(x0 - RM + p);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            place(ring[p][i], next[i]);
        }
    }
    fetch(x0 + RM);
    for (int xb = x0; xb < x1; xb += P) {
#pragma unroll
        for (int p = 0; p < P; ++p) {              // plane x in ring slot (p + RM) % P
            const int x = xb + p;
            if (x >= x1)
                break;
            constexpr int kNew = P - 1;
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                place(ring[(p + kNew) % P][i], next[i]);
            }
            fetch(x + 1 + RM);
            float2(*buf)[64] = s_rows[(x - x0) & 1];
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                if (wave + kFusedWaves * i >= RT)
                    break;
                float v[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    v[c] = K.w[0][0] * ring[(p + RM) % P][i][c];
#pragma unroll
                    for (int d = 1; d <= RM; ++d)
                        if (d <= K.R[0])
                            v[c] = __builtin_fmaf(
                                K.w[0][d],
                                ring[(p + RM - d) % P][i][c] + ring[(p + RM + d) % P][i][c], v[c]);
                }
                buf[wave + kFusedWaves * i][lane] = make_float2(v[0], v[1]);
            }
            __syncthreads();
            const rsrc_t oplane = make_rsrc(out + (int64_t)x * ny * nz, bytes_out);
            float2 r[kRowsOut + 2 * RM];
#pragma unroll
            for (int j = 0; j < kRowsOut + 2 * RM; ++j)
                r[j] = buf[wave * kRowsOut + j][lane];
#pragma unroll
            for (int j = 0; j < kRowsOut; ++j) {
                float a = K.w[1][0] * r[j + RM].x, b = K.w[1][0] * r[j + RM].y;
#pragma unroll
                for (int d = 1; d <= RM; ++d)
                    if (d <= K.R[1]) {
                        a = __builtin_fmaf(K.w[1][d], r[j + RM - d].x + r[j + RM + d].x, a);
                        b = __builtin_fmaf(K.w[1][d], r[j + RM - d].y + r[j + RM + d].y, b);
                    }
                // n[RM + k]: the row's value at z + k
                float n[2 * RM + 2];
                float pa = a, pb = b, na = a, nb = b;
                n[RM] = a;
                n[RM + 1] = b;
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    pa = lane_before(pa);
                    pb = lane_before(pb);
                    na = lane_after(na);
                    nb = lane_after(nb);
                    n[RM - 1 - 2 * h] = pb;
                    n[RM + 2 + 2 * h] = na;
                    if (RM - 2 - 2 * h >= 0) {
                        n[RM - 2 - 2 * h >= 0 ? RM - 2 - 2 * h : 0] = pa;
                        n[RM - 2 - 2 * h >= 0 ? RM + 3 + 2 * h : 0] = nb;
                    }
                }
                a = K.w[2][0] * n[RM];
                b = K.w[2][0] * n[RM + 1];
#pragma unroll
                for (int d = 1; d <= RM; ++d)
                    if (d <= K.R[2]) {
                        a = __builtin_fmaf(K.w[2][d], n[RM - d] + n[RM + d], a);
                        b = __builtin_fmaf(K.w[2][d], n[RM + 1 - d] + n[RM + 1 + d], b);
                    }
                const uint32_t ab[2] = {__float_as_uint(a), __float_as_uint(b)};
                if (PAIR) {
                    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{ab[0], ab[1]}, oplane, oz[j], 0, 0);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b32(ab[0], oplane, oz[j], 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b32(
                        ab[1], oplane, z + 1 < nz ? oz[j] + 4u : bytes_out, 0, 0);
                }
            }
        }
    }
}

int32_t gauss_radius(float sigma)
{
    return sigma > 0.0f ? (int32_t)std::floor(3.0 * (double)sigma / std::sqrt(2.0) + 0.5) : 0;
}

GaussTaps gauss_taps(float sigma)
{
    GaussTaps K;
    K.R = gauss_radius(sigma);
    double w[kMaxGaussRadius + 1];
    double sum = 0.0;
    for (int d = 0; d <= K.R; ++d) {
        // R = 0 (sigma = 0 included): the single tap 1
        w[d] = K.R == 0 ? 1.0 : std::exp(-(double)d * (double)d / ((double)sigma * (double)sigma));
        sum += d == 0 ? w[d] : 2.0 * w[d];
    }
    for (int d = 0; d <= kMaxGaussRadius; ++d)
        K.w[d] = d <= K.R ? (float)(w[d] / sum) : 0.0f;
    return K;
}

// Launch shape of the fused pass at largest radius rm: nyt row tiles, nzs z segments of
// zlen outputs, nxc x chunks of cx planes.  At most 1024 workgroups in all where the
// chunks decide, which is a round at R = 1 (4 resident per CU), two at R = 2 and 3 (2, by
// their registers) and four at R = 4 (1); and at least 4 P planes a chunk, as a chunk
// starts by loading P - 1 planes anew.
struct FusedShape {
    int32_t nyt, nzs, zlen, cx, nxc;
};
static FusedShape fused_shape(int32_t rm, const int32_t dim[3])
{
    const int32_t seg = 2 * (64 - 2 * ((rm + 1) / 2)), rows = kFusedWaves * kRowsOut;
    FusedShape S;
    S.nzs = (dim[2] + seg - 1) / seg;
    S.zlen = ((dim[2] + S.nzs - 1) / S.nzs + 1) & ~1;
    S.nyt = (dim[1] + rows - 1) / rows;
    const int64_t tiles = (int64_t)S.nyt * S.nzs;
    const int32_t most = std::max(1, dim[0] / (4 * (2 * rm + 1)));
    S.nxc = (int32_t)std::min<int64_t>(most, std::max<int64_t>(1, 1024 / tiles));
    S.cx = (dim[0] + S.nxc - 1) / S.nxc;
    S.nxc = (dim[0] + S.cx - 1) / S.cx;
    return S;
}

// Whether the axes go in one pass: a plane's byte offsets are 31-bit (scalar offsets of
// its buffer), radii fit the ring, and it is the faster way.  The fused pass walks its
// planes in turn, a barrier each, in as many workgroups as the volume gives; a pass per
// axis is bound by its blocks (one per row and 256 voxels) and, the larger the radius, by
// its loads, and is not under 5 us a launch.  Times in us, fitted to measurements from
// 32^3 to 512^2 x 64 voxels: a fused pass takes 3.5 and per plane walked 0.67, 0.87, 1.23
// or 1.61 (R = 1 .. 4), in each round of resident workgroups; an axis 3, 0.43 per 1000
// blocks, and per 10^6 voxels 0.33, 0.5, 0.83 or 1.5.  Volumes from 4 * 10^6 voxels on
// are fused for nearly all radii (there the fused pass is bound by memory).  Per axis
// against fused, measured: 64^3 R = 4 21 / 107 us; 96^3 R = 2 21 / 25, R = 3 23 / 44; 128 x
// 128 x 60 R = 2 32 / 23, R = 3 32 / 44; 160 x 160 x 100 R = 3 48 / 44, R = 4 53 / 70; 192
// x 192 x 96 R = 4 71 / 68, z alone with R = 2 19 / 24.
bool smooth_fused_ok(const int32_t R[3], const int32_t dim[3])
{
    if ((int64_t)dim[1] * dim[2] >= (int64_t)1 << 29)
        return false;
    int32_t rm = 1;
    for (int a = 0; a < 3; ++a) {
        if (R[a] > kFusedMaxR)
            return false;
        rm = std::max(rm, R[a]);
    }
    constexpr double kPlane[kFusedMaxR + 1] = {0.0, 0.67, 0.87, 1.23, 1.61};
    constexpr double kVoxels[kFusedMaxR + 1] = {0.0, 0.33e-6, 0.5e-6, 0.83e-6, 1.5e-6};
    constexpr int32_t kResident[kFusedMaxR + 1] = {0, 1024, 512, 512, 256};
    const FusedShape S = fused_shape(rm, dim);
    const double groups = (double)S.nyt * S.nzs * S.nxc;
    const double fused = 3.5 + std::ceil(groups / kResident[rm]) * S.cx * kPlane[rm];
    const double rows = (double)dim[0] * dim[1];
    const double axis = 3.0 + 0.43e-3 * rows * ((dim[2] + kThreads - 1) / kThreads);
    double passes = 0.0;
    for (int a = 0; a < 3; ++a)
        passes += R[a] > 0 ? std::max(axis + kVoxels[R[a]] * rows * dim[2], 5.0) : 0.0;
    return fused <= passes;
}

template <int RM>
static void launch_fused_r(const void *in, bool in_i16, float *out, const int32_t dim[3],
                           const FusedTaps &K, hipStream_t s)
{
    const FusedShape S = fused_shape(RM, dim);
    const int64_t grid = (int64_t)S.nyt * S.nzs * S.nxc;
    const uintptr_t at = reinterpret_cast<uintptr_t>(in);
    const bool pair = dim[2] % 2 == 0 && (reinterpret_cast<uintptr_t>(out) & 7u) == 0 &&
                      (at & (in_i16 ? 3u : 7u)) == 0;
    auto launch = [&](auto kern, auto *src) {
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * kFusedWaves), 0, s, src, out,
                           dim[0], dim[1], dim[2], S.nyt, S.nzs, S.zlen, S.cx, K);
    };
    if (in_i16)
        launch(pair ? &k_smooth_fused<int16_t, RM, true> : &k_smooth_fused<int16_t, RM, false>,
               static_cast<const int16_t *>(in));
    else
        launch(pair ? &k_smooth_fused<float, RM, true> : &k_smooth_fused<float, RM, false>,
               static_cast<const float *>(in));
}

hipError_t launch_smooth_fused(const void *in, bool in_i16, float *out, const int32_t dim[3],
                               const float sigma[3], hipStream_t s)
{
    FusedTaps F;
    int32_t rm = 1;
    for (int a = 0; a < 3; ++a) {
        const GaussTaps K = gauss_taps(sigma[a]);
        F.R[a] = K.R;
        rm = std::max(rm, K.R);
        for (int d = 0; d <= kFusedMaxR; ++d)
            F.w[a][d] = K.w[d];
    }
    switch (rm) {
    case 1: launch_fused_r<1>(in, in_i16, out, dim, F, s); break;
    case 2: launch_fused_r<2>(in, in_i16, out, dim, F, s); break;
    case 3: launch_fused_r<3>(in, in_i16, out, dim, F, s); break;
    default: launch_fused_r<4>(in, in_i16, out, dim, F, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_smooth_axis(const void *in, bool in_i16, float *out, const int32_t dim[3],
                              int axis, const GaussTaps &K, hipStream_t s)
{
    const dim3 grid((unsigned)((dim[2] + kThreads - 1) / kThreads), (unsigned)dim[1],
                    (unsigned)dim[0]);
    if (in_i16)
        hipLaunchKernelGGL(k_smooth_axis<int16_t>, grid, dim3(kThreads), 0, s,
                           static_cast<const int16_t *>(in), out, dim[0], dim[1], dim[2], axis, K);
    else
        hipLaunchKernelGGL(k_smooth_axis<float>, grid, dim3(kThreads), 0, s,
                           static_cast<const float *>(in), out, dim[0], dim[1], dim[2], axis, K);
    return hipGetLastError();
}

}  // namespace ctaug
