// tile_geom.h -- geometry of an output box's input footprint and its staging
// into LDS (internal; shared by the forward and adjoint kernels).
//
// The coordinate is affine in the output voxel, so over a box its extremes
// per axis are the value at the box origin plus the negative / positive parts
// of A_ij * span_j, widened by a bound on FP32 rounding.  From them: whether
// every sample of the box fails the guard (outside), whether every trilinear
// cell lies inside the volume (interior), and its window: the input cells
// floor(q) .. floor(q) + 1 of every sample once coordinates are moved into
// [-2, n] (guard_coord), of the same extents for all boxes of a job.
#pragma once

#include "device_common.h"

#include <climits>

namespace ctaug {

enum : int { kOutside = 0, kInterior = 1, kBoundary = 2 };

// LDS row pitch for rows of e cells: whole quads of 4 cells, and an odd
// number of quads so that neighbouring rows start in different LDS banks
// (rows a multiple of 8 cells apart would all fall on the same banks).
__device__ __host__ __forceinline__ int lds_pitch(int e)
{
    const int p = (e + 3) & ~3;
    return (p & 4) ? p : p + 4;
}

// A footprint window, uniform over the workgroup.
struct TileGeom {
    int lo[3], e[3];                   // input cells [lo, lo + e)
    int quads;                         // 4-cell quads staged per row: ceil(e[2] / 4)
    int pitch;                         // LDS row pitch: 4 * quads, padded to 4 mod 8 cells
};

__device__ __forceinline__ void store4(float *dst, const float v[4])
{
    *reinterpret_cast<f32x4 *>(dst) = f32x4{v[0], v[1], v[2], v[3]};
}

__device__ __forceinline__ void store4(int16_t *dst, const int16_t v[4])
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    *reinterpret_cast<u32x2 *>(dst) =
        u32x2{(uint32_t)(uint16_t)v[0] | ((uint32_t)(uint16_t)v[1] << 16),
              (uint32_t)(uint16_t)v[2] | ((uint32_t)(uint16_t)v[3] << 16)};
}

// Four consecutive input cells at byte offset `off` copied into LDS cells of
// type LT with one buffer load (16 bytes of FP32 or 8 bytes of int16; the
// offset need only be element-aligned).
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void copy_quad(rsrc_t r, uint32_t off, float *dst, float)
{
    *reinterpret_cast<u32x4 *>(dst) = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}

__device__ __forceinline__ void copy_quad(rsrc_t r, uint32_t off, int16_t *dst, int16_t)
{
    *reinterpret_cast<u32x2 *>(dst) = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
}

__device__ __forceinline__ void copy_quad(rsrc_t r, uint32_t off, float *dst, int16_t)
{
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
    *reinterpret_cast<f32x4 *>(dst) =
        f32x4{(float)(int16_t)(w.x & 0xffffu), (float)((int32_t)w.x >> 16),
              (float)(int16_t)(w.y & 0xffffu), (float)((int32_t)w.y >> 16)};
}

// The raw bytes of four consecutive input cells of type T at element offset e
// (one wide load), and their store as LDS cells of type LT.
template <typename T> struct QuadRaw;
template <> struct QuadRaw<float> {
    typedef u32x4 type;
    // at byte offset off + base (base uniform)
    static __device__ __forceinline__ type load_at(rsrc_t r, uint32_t off, uint32_t base)
    {
        return __builtin_amdgcn_raw_buffer_load_b128(r, off, base, 0);
    }
    static __device__ __forceinline__ void store(type w, float *dst)
    {
        *reinterpret_cast<u32x4 *>(dst) = w;
    }
    static __device__ __forceinline__ void cells(type w, float (&c)[4])
    {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            c[u] = __uint_as_float(w[u]);
    }
};
template <> struct QuadRaw<int16_t> {
    typedef u32x2 type;
    static __device__ __forceinline__ type load_at(rsrc_t r, uint32_t off, uint32_t base)
    {
        return __builtin_amdgcn_raw_buffer_load_b64(r, off, base, 0);
    }
    template <typename LT> static __device__ __forceinline__ void cells(type w, LT (&c)[4])
    {
        c[0] = (LT)(int16_t)(w.x & 0xffffu);
        c[1] = (LT)(int16_t)(w.x >> 16);
        c[2] = (LT)(int16_t)(w.y & 0xffffu);
        c[3] = (LT)(int16_t)(w.y >> 16);
    }
    static __device__ __forceinline__ void store(type w, int16_t *dst)
    {
        *reinterpret_cast<u32x2 *>(dst) = w;
    }
    static __device__ __forceinline__ void store(type w, float *dst)
    {
        *reinterpret_cast<f32x4 *>(dst) =
            f32x4{(float)(int16_t)(w.x & 0xffffu), (float)((int32_t)w.x >> 16),
                  (float)(int16_t)(w.y & 0xffffu), (float)((int32_t)w.y >> 16)};
    }
};

// floor(a / b) for 0 <= a < 2^20, 0 < b < 2^16: FP32 estimate from rcp_b =
// rcp_small(b), off by at most one (the reciprocal is good to 2^-23 and the product
// to 2^-24, together less than 2^-2 of a quotient), and one integer correction step.
// An IEEE quotient for the reciprocal took 11 instructions more, five times a tile.
__device__ __forceinline__ float rcp_small(int b) { return __builtin_amdgcn_rcpf((float)b); }
__device__ __forceinline__ int div_small(int a, int b, float rcp_b)
{
    int q = (int)((float)a * rcp_b);
    const int r = a - q * b;
    q += (r >= b) - (r < 0);
    return q;
}

// A quad of four input cells (gx, gy, gz0 .. gz0 + 3) wholly inside the volume,
// at element offset e: one wide load.
template <typename T, typename LT>
__device__ __forceinline__ void quad_inside(const Src &S, uint32_t e, LT *dst)
{
    copy_quad(S.img, e * (uint32_t)sizeof(T), dst, T());
}

// A quad of an in-volume row (element offset e_row0 of its z = 0 cell) whose
// z range leaves the volume: each cell is loaded from its z clamped into the
// volume (every load stays in range) and replaced by fill outside.
template <typename T, typename LT>
__device__ __forceinline__ void quad_partial(const FwdJob &J, const Src &S, int e_row0, int gz0,
                                             LT *dst)
{
    constexpr uint32_t es = sizeof(T);
    const LT tfill = (LT)J.fill;
    LT v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int gz = gz0 + u;
        const uint32_t e = (uint32_t)(e_row0 + min(max(gz, 0), J.nz - 1));
        const T raw = Elem<T>::raw(S.img, e * es, 0);
        v[u] = (unsigned)gz < (unsigned)J.nz ? (LT)raw : tfill;
    }
    store4(dst, v);
}

// A quad of a row outside the volume: fill, nothing loaded.
template <typename LT>
__device__ __forceinline__ void quad_fill(const FwdJob &J, LT *dst)
{
    const LT tfill = (LT)J.fill;
    const LT v[4] = {tfill, tfill, tfill, tfill};
    store4(dst, v);
}

// Row walk of the footprint staging: the lane takes rows row, row + rpp, ...
// (rpp = rows per pass), tracking the row's input cell (cx, cy), its element
// offset and its LDS offset by additions of per-tile constants.
struct RowWalk {
    int row, cx, cy, e_row, l_row;     // e_row: element offset of cell (lo0 + cx, lo1 + cy, 0)
    int rpp, step_x, step_y, ey, de, de_wrap, dl;

    __device__ __forceinline__ void init(const Src &S, const TileGeom &G, int first_row,
                                         int rows_per_pass, int lane_cell)
    {
        ey = G.e[1];
        rpp = rows_per_pass;
        const float rcp_y = rcp_small(ey);
        step_x = div_small(rpp, ey, rcp_y);            // rpp = step_x * ey + step_y
        step_y = rpp - step_x * ey;
        row = first_row;
        cx = div_small(row, ey, rcp_y);
        cy = row - cx * ey;
        const int plane = S.ry * S.rsy;                 // elements per x plane
        e_row = (G.lo[0] + cx) * plane + (G.lo[1] + cy) * S.rsy;
        de = step_x * plane + step_y * S.rsy;
        de_wrap = plane - ey * S.rsy;
        l_row = row * G.pitch + lane_cell;
        dl = rpp * G.pitch;
    }
    __device__ __forceinline__ void next()
    {
        row += rpp;
        cx += step_x;
        cy += step_y;
        e_row += de;
        l_row += dl;
        if (cy >= ey) {
            cy -= ey;
            cx += 1;
            e_row += de_wrap;
        }
    }
};

// Copy the tile's input image footprint into LDS in the LDS cell type, with
// fill in cells outside the volume (labels are gathered from global memory
// while sampling, so that the LDS holds image cells only): windows that
// stage_window does not take, of volumes of fewer than 4 cells along z or rows of
// more quads than a workgroup has threads.  The footprint is e[0] x e[1] rows of
// `quads` quads of 4 cells (row pitch G.pitch cells).  A row of at most 16 quads
// is taken by `quads` consecutive lanes, one quad each; a longer row by 16 lanes (a
// lane takes quads q, q + 16, ...).  Rows advance by additions (RowWalk).  Rows
// outside the volume are filled without loads, quads crossing its z ends load
// per cell from clamped indices.
template <typename T, typename LT>
__device__ __forceinline__ void stage_footprint(const FwdJob &J, const Src &S, const TileGeom &G,
                                                LT *s_img)
{
    const int qpr = G.quads, rows = G.e[0] * G.e[1];
    int lpr, ql, row0, rpp;
    if (qpr <= 16) {
        // qpr lanes per row, floor(256 / qpr) rows per pass; lanes past the
        // last whole row stay idle (ql = qpr)
        lpr = qpr;
        row0 = div_small(threadIdx.x, qpr, rcp_small(qpr));
        rpp = kThreads / qpr;
        ql = row0 < rpp ? threadIdx.x - row0 * qpr : qpr;
    } else {
        lpr = 16;
        row0 = threadIdx.x >> 4;
        rpp = kThreads >> 4;
        ql = threadIdx.x & 15;
    }
    RowWalk W;
    W.init(S, G, row0, rpp, 4 * min(ql, qpr - 1));
    for (; W.row < rows; W.next()) {
        const int gx = G.lo[0] + W.cx, gy = G.lo[1] + W.cy;
        const bool row_in = (unsigned)gx < (unsigned)J.nx && (unsigned)gy < (unsigned)J.ny;
        for (int q = ql; q < qpr; q += lpr) {
            const int gz0 = G.lo[2] + 4 * q;
            LT *dst = s_img + W.l_row + 4 * (q - ql);
            if (!row_in)
                quad_fill<LT>(J, dst);
            else if (gz0 >= 0 && gz0 + 3 < J.nz)
                quad_inside<T, LT>(S, (uint32_t)(W.e_row + gz0), dst);
            else
                quad_partial<T, LT>(J, S, W.e_row, gz0, dst);
        }
    }
}

// A job in constant memory (kernel arguments or the batch's table, which no
// kernel writes): its fields are scalar loads.  reload() hides the pointer's
// origin, so that a phase's fields are loaded anew there rather than kept in
// scalar registers through the phases before it (all of them together spill).
typedef __attribute__((address_space(4))) const FwdJob *JobPtr;
__device__ __forceinline__ JobPtr reload(JobPtr p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// A coordinate moved into [-2, n] without changing its sample: at or below -1
// (and NaN) it goes to -2, at or above n to n.  There every corner is outside the volume,
// so the trilinear value is fill and the nearest voxel is outside, which is what
// the guard (-1, n) gives; a footprint of cells within [-2, n + 2), fill where
// outside the volume, then needs no test per sample.
__device__ __forceinline__ float guard_coord(float q, float n)
{
    return fminf(q > -1.0f ? q : -2.0f, n);
}

// The quads (4 cells of a row) of a footprint window that this thread copies: quad
// ql of rows row0, row0 + rpp, ... (mine of them), (cx, cy) the plane and row of the
// first within the window.  The windows of a job's sub-tiles have the same
// extents, so this is laid out once per tile.  NT threads take part.
constexpr int kStageChunk = 4;
struct StageWalk {
    int row0, ql, cx, cy, mine;
    int rpp, step_x, step_y, passes;   // uniform; rpp = step_x ey + step_y
};

template <int NT> __device__ __forceinline__ StageWalk stage_walk(int rows, int ey, int quads,
                                                                       int tid)
{
    StageWalk W;
    W.row0 = W.ql = W.cx = W.cy = W.mine = W.step_x = W.step_y = 0;
    W.passes = 0;
    W.rpp = __builtin_amdgcn_readfirstlane(div_small(NT, quads, rcp_small(quads)));
    if (W.rpp == 0)
        return W;
    W.passes = __builtin_amdgcn_readfirstlane(
        div_small(rows + W.rpp - 1, W.rpp, rcp_small(W.rpp)));
    W.row0 = div_small(tid, quads, rcp_small(quads));
    W.ql = tid - W.row0 * quads;
    const float rcp_y = rcp_small(ey);
    W.step_x = __builtin_amdgcn_readfirstlane(div_small(W.rpp, ey, rcp_y));
    W.step_y = W.rpp - W.step_x * ey;
    W.cx = div_small(W.row0, ey, rcp_y);
    W.cy = W.row0 - W.cx * ey;
    W.mine = W.row0 < W.rpp ? (W.row0 + (W.passes - 1) * W.rpp < rows ? W.passes : W.passes - 1)
                            : 0;
    return W;
}

// Four raw cells c loaded from z = zc of a row, of which the quad's cell u is
// c[s + u] (fill where s + u is not 0 .. 3, or ok is false), written as LDS cells.
template <typename LT>
__device__ __forceinline__ void store_shifted(const LT (&c)[4], int s, bool ok, LT fill, LT *dst)
{
    LT v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        v[u] = fill;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            v[u] = s + u == j ? c[j] : v[u];
        v[u] = ok ? v[u] : fill;
    }
    store4(dst, v);
}

// Copies a window into LDS, kStageChunk loads of a thread in flight at once (12
// took as long: lines fetched count, not round trips, and the registers cost a
// wave per SIMD).  Quads that no sample of the box can use are not loaded
// (FwdJob::reach; their cells are never read): a rotated box fills about half of
// its window (CLIP; displaced boxes copy every quad).  That took the 16-volume
// batch from 250 to 237 us.
// inside: the window (whole quads) lies in the volume.  Otherwise each quad is
// loaded from the nearest place inside the volume (of at least 4 cells along
// z), and its cells outside the volume become fill as they are written.
template <typename T, typename LT, bool CLIP>
__device__ __forceinline__ void stage_window(const FwdJob &J, const Src &S, const StageWalk &W,
                                             const int (&lo)[3], const float (&g)[3], int ey,
                                             int pitch, bool inside, uint8_t *s_lds)
{
    constexpr int N = kStageChunk;
    const float zq = (float)(4 * W.ql) + 1.5f;
    float gz[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        gz[k] = CLIP ? __builtin_fmaf(J.inv[3 * k + 2], zq, g[k]) : 0.0f;
    // whether a sample of the box can use the quad at row (cx, cy) of the window
    auto reach = [&](int cx, int cy) {
        if (!CLIP)
            return true;
        const float fx = (float)cx, fy = (float)cy;
        bool r = true;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            r = r && fabsf(__builtin_fmaf(J.inv[3 * k], fx,
                                          __builtin_fmaf(J.inv[3 * k + 1], fy, gz[k]))) <=
                         J.reach[k];
        return r;
    };
    constexpr uint32_t kNowhere = 0xffffffffu;     // past the buffer's end: no access, reads 0
    typename QuadRaw<T>::type w[N];
    uint32_t l = (uint32_t)(W.row0 * pitch + 4 * W.ql) * (uint32_t)sizeof(LT);
    const uint32_t step = (uint32_t)(W.rpp * pitch) * (uint32_t)sizeof(LT);
    int cx = W.cx, cy = W.cy;
    if (inside) {
        const int plane = S.ry * S.rsy;                    // elements
        const uint32_t base = (uint32_t)(lo[0] * plane + lo[1] * S.rsy + lo[2]) *
                              (uint32_t)sizeof(T);
        uint32_t o = (uint32_t)(W.cx * plane + cy * S.rsy + 4 * W.ql) * (uint32_t)sizeof(T);
        const uint32_t d = (uint32_t)(W.step_x * plane + W.step_y * S.rsy) * (uint32_t)sizeof(T);
        const uint32_t dw = (uint32_t)(plane - ey * S.rsy) * (uint32_t)sizeof(T) + d;
        for (int p0 = 0; p0 < W.passes; p0 += N) {
#pragma unroll
            for (int u = 0; u < N; ++u) {
                w[u] = QuadRaw<T>::load_at(S.img, p0 + u < W.mine && reach(cx, cy) ? o : kNowhere,
                                           base);
                const int c = cy + W.step_y;
                o += c >= ey ? dw : d;
                cx += c >= ey ? W.step_x + 1 : W.step_x;
                cy = c >= ey ? c - ey : c;
            }
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (p0 + u < W.mine)
                    QuadRaw<T>::store(w[u], reinterpret_cast<LT *>(s_lds + (l + u * step)));
            l += N * step;
        }
        return;
    }
    const int gz0 = lo[2] + 4 * W.ql;
    const int zc = min(max(gz0, 0), J.nz - 4), s = gz0 - zc;
    const bool shifted = __any(s != 0);
    const LT fill = (LT)J.fill;
    for (int p0 = 0; p0 < W.passes; p0 += N) {
        uint32_t rows_in = 0;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int gx = lo[0] + cx, gy = lo[1] + cy;
            const bool in = (uint32_t)gx < (uint32_t)J.nx && (uint32_t)gy < (uint32_t)J.ny;
            rows_in |= (in ? 1u : 0u) << u;
            w[u] = QuadRaw<T>::load_at(
                S.img,
                in && p0 + u < W.mine && reach(cx, cy)
                    ? elem_index(S, gx, gy, zc) * (uint32_t)sizeof(T)
                    : kNowhere,
                0);
            const int c = cy + W.step_y;
            cx += c >= ey ? W.step_x + 1 : W.step_x;
            cy = c >= ey ? c - ey : c;
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (p0 + u < W.mine) {
                LT c[4];
                QuadRaw<T>::cells(w[u], c);
                LT *dst = reinterpret_cast<LT *>(s_lds + (l + u * step));
                const bool ok = (rows_in >> u) & 1;
                if (shifted) {
                    store_shifted<LT>(c, s, ok, fill, dst);
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        c[v] = ok ? c[v] : fill;
                    store4(dst, c);
                }
            }
        l += N * step;
    }
}

// Class of the sub-tile of an affine job whose first voxel is (x, y, z), the first
// cell lo of its window (FwdJob::box_*; inside the volume for an interior one,
// inside [-2, n + 2) otherwise) and the constants gr of its quad test
// (stage_window).  Any lane's or a uniform voxel.
__device__ __forceinline__ int box_window(const FwdJob &J, float x, float y, float z, int (&lo)[3],
                                          float (&gr)[3])
{
    if (J.nx == 0 || J.ny == 0 || J.nz == 0)
        return kOutside;               // empty input: every sample is fill
    const int n[3] = {J.nx, J.ny, J.nz};
    const int e[3] = {J.box_e[0], J.box_e[1], (J.box_e[2] + 3) & ~3};
    float rb[3], qc[3];
    row_base(J.M, x, y, rb);
    bool outside = false, interior = true;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float q0 = coord(J.M, i, rb, z);
        qc[i] = q0 + J.box_mid[i];
        const float l = q0 + J.box_dn[i], h = q0 + J.box_up[i];
        outside = outside || h <= -1.0f || l >= (float)n[i];
        interior = interior && l >= 0.0f && h < (float)(n[i] - 1) && e[i] <= n[i];
        lo[i] = (int)fminf(fmaxf(floorf(l), -2.0f), (float)n[i]);
    }
    const int cls = outside ? kOutside : interior ? kInterior : kBoundary;
#pragma unroll
    for (int i = 0; i < 3; ++i)
        lo[i] = min(lo[i], cls == kInterior ? n[i] - e[i] : n[i] + 2 - J.box_e[i]);
#pragma unroll
    for (int k = 0; k < 3; ++k)
        gr[k] = __builtin_fmaf(J.inv[3 * k], (float)lo[0] - qc[0],
                               __builtin_fmaf(J.inv[3 * k + 1], (float)lo[1] - qc[1],
                                              J.inv[3 * k + 2] * ((float)lo[2] - qc[2])));
    return cls;
}

// Workgroup-wide min of mn[] and max of mx[] (3 ints each); every thread gets
// the result, as scalars.  s_red: 4 x 8 ints of LDS, 16-byte aligned.  Contains
// one barrier; the caller passes another before it calls again.
//
// In a wave by DPP row shifts and broadcasts, lane 63 holding the results: one VALU
// instruction a step (a lane without a source takes the operation's identity, so that
// the move folds into it; with the lane's own value instead it was three) and the
// six values in turn (a value's steps wait for each other).  Tiles of 256^3 B-spline
// warps, bound by vector instructions, spent 150 of 860 here; it is 60.
__device__ __forceinline__ void block_minmax3(int mn[3], int mx[3], int (*s_red)[8])
{
    static_assert(kThreads == 256, "four waves");
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    typedef int i32x2 __attribute__((ext_vector_type(2)));
    int m[6] = {mn[0], mn[1], mn[2], ~mx[0], ~mx[1], ~mx[2]};  // max: min of the complement
#define CTAUG_DPP_MIN(ctrl, rows)                                                                 \
    _Pragma("unroll") for (int i = 0; i < 6; ++i) m[i] =                                          \
        min(m[i], __builtin_amdgcn_update_dpp(INT_MAX, m[i], ctrl, rows, 0xF, false))
    CTAUG_DPP_MIN(0x111, 0xF);         // row_shr:1, 2, 4, 8: lane 15 of each row of 16
    CTAUG_DPP_MIN(0x112, 0xF);
    CTAUG_DPP_MIN(0x114, 0xF);
    CTAUG_DPP_MIN(0x118, 0xF);
    CTAUG_DPP_MIN(0x142, 0xA);         // row_bcast:15 into rows 1 and 3
    CTAUG_DPP_MIN(0x143, 0xC);         // row_bcast:31 into rows 2 and 3
#undef CTAUG_DPP_MIN
    if ((threadIdx.x & 63) == 63) {
        int *w = s_red[threadIdx.x >> 6];
        *reinterpret_cast<i32x4 *>(w) = i32x4{m[0], m[1], m[2], m[3]};
        *reinterpret_cast<i32x2 *>(w + 4) = i32x2{m[4], m[5]};
    }
    __syncthreads();
    i32x4 a[4];
    i32x2 b[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        a[w] = *reinterpret_cast<const i32x4 *>(s_red[w]);
        b[w] = *reinterpret_cast<const i32x2 *>(s_red[w] + 4);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int r = i < 4 ? min(min(a[0][i], a[1][i]), min(a[2][i], a[3][i]))
                            : min(min(b[0][i - 4], b[1][i - 4]), min(b[2][i - 4], b[3][i - 4]));
        const int s = __builtin_amdgcn_readfirstlane(r);
        (i < 3 ? mn[i] : mx[i - 3]) = i < 3 ? s : ~s;
    }
}

}  // namespace ctaug
