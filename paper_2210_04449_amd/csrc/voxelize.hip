// Voxelization of a triangle mesh into the coarse grid (paper Sec. 2.1).
//
// The paper renders the scene three times with an orthographic camera along
// +x, +y and +z, depth writes off, and marks the voxel under every fragment.
// gfx950 has no raster pipeline, so this is a compute kernel that applies an
// exact integer version of that rule: vertices snapped to 1/256 voxel, a
// column covered when its centre is inside or on the projected triangle, and
// the voxel holding the triangle's depth at that centre marked.
//
// Work mapping: a projection whose bounding box holds at most kSmallPixels
// column centres is rasterized by one lane in 32-bit integers (three
// projections a lane: a triangle's vertices are snapped once); larger ones by
// a whole wavefront, and those of more than kWavePixels (room walls cover
// whole faces of the grid) by the whole workgroup, in 64-bit integers.
// Triangles are dealt to workgroups one by one, so the large projections of
// consecutive triangles (the walls of a room come one after another) land in
// different workgroups instead of queueing in one.
//
// Bound by the latency of its gathers and its largest projections: with the
// fill of the seeds, 1.0 M triangles at 256^3 355 -> 151 us, 211 k at 128^3
// 108 -> 48 us, 1,880 large ones at 256^3 432 -> 54 us, 322 at 32^3 16 -> 11 us
// (against one lane per (triangle, axis) in 64-bit integers, which snapped each
// vertex three times and left a wall's 65,536 columns to one wavefront).
#include <algorithm>
#include <cmath>

#include "common.hpp"

namespace rtsdf {

constexpr int kSmallPixels = 16;

struct VoxTri {
    int64_t px[3], py[3], z[3];  // projected snapped coordinates, depth
    int64_t area2;               // > 0 (counter-clockwise after the swap)
    int i0, i1, j0, j1;          // column range (inclusive)
    int axis;
};

__device__ __forceinline__ int64_t floor_div_pos(int64_t a, int64_t b)  // b > 0
{
    int64_t q = a / b;
    if ((a % b) != 0 && a < 0) --q;
    return q;
}

// A vertex snapped to 1/256 voxel (batches; snap32 below gives the same numbers).
__device__ __forceinline__ bool snap(const float *__restrict__ v, int vi, const rtsdf_grid &g, int64_t X[3])
{
    const double side = (double)g.n * (double)g.h;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double rel = (double)v[3 * vi + a] - (double)g.lo[a];
        if (!(rel >= -side && rel <= 2.0 * side)) return false;
        X[a] = (int64_t)__builtin_rint(rel / (double)g.h * 256.0);
    }
    return true;
}

// Sets up the projection of triangle t along `axis`; false if it covers
// nothing (zero area or box outside the grid).
__device__ bool vox_setup(const int64_t X[3][3], int axis, int n, VoxTri &T)
{
    const int e1 = (axis + 1) % 3, e2 = (axis + 2) % 3;
    for (int k = 0; k < 3; ++k) {
        T.px[k] = X[k][e1];
        T.py[k] = X[k][e2];
        T.z[k] = X[k][axis];
    }
    int64_t area2 = (T.px[1] - T.px[0]) * (T.py[2] - T.py[0]) - (T.py[1] - T.py[0]) * (T.px[2] - T.px[0]);
    if (area2 == 0) return false;
    if (area2 < 0) {
        int64_t tx = T.px[1], ty = T.py[1], tz = T.z[1];
        T.px[1] = T.px[2]; T.py[1] = T.py[2]; T.z[1] = T.z[2];
        T.px[2] = tx; T.py[2] = ty; T.z[2] = tz;
        area2 = -area2;
    }
    T.area2 = area2;
    T.axis = axis;
    const int64_t minx = min(T.px[0], min(T.px[1], T.px[2])), maxx = max(T.px[0], max(T.px[1], T.px[2]));
    const int64_t miny = min(T.py[0], min(T.py[1], T.py[2])), maxy = max(T.py[0], max(T.py[1], T.py[2]));
    // column centre 256 i + 128 within [min, max]
    int64_t i0 = floor_div_pos(minx - 128 + 255, 256), i1 = floor_div_pos(maxx - 128, 256);
    int64_t j0 = floor_div_pos(miny - 128 + 255, 256), j1 = floor_div_pos(maxy - 128, 256);
    i0 = max(i0, (int64_t)0);
    j0 = max(j0, (int64_t)0);
    i1 = min(i1, (int64_t)n - 1);
    j1 = min(j1, (int64_t)n - 1);
    if (i0 > i1 || j0 > j1) return false;
    T.i0 = (int)i0; T.i1 = (int)i1; T.j0 = (int)j0; T.j1 = (int)j1;
    return true;
}

// Tests column (i, j); marks the voxel if covered.
__device__ __forceinline__ void vox_column(const VoxTri &T, int i, int j, int n, int32_t *__restrict__ seeds)
{
    const int64_t cx = 256 * (int64_t)i + 128, cy = 256 * (int64_t)j + 128;
    const int64_t w0 = (T.px[2] - T.px[1]) * (cy - T.py[1]) - (T.py[2] - T.py[1]) * (cx - T.px[1]);
    const int64_t w1 = (T.px[0] - T.px[2]) * (cy - T.py[2]) - (T.py[0] - T.py[2]) * (cx - T.px[2]);
    const int64_t w2 = (T.px[1] - T.px[0]) * (cy - T.py[0]) - (T.py[1] - T.py[0]) * (cx - T.px[0]);
    if ((w0 | w1 | w2) < 0) return;
    const int64_t num = w0 * T.z[0] + w1 * T.z[1] + w2 * T.z[2];
    const int64_t den = T.area2 * 256;
    int64_t L;
    if (num == (int64_t)n * den) {
        L = n - 1;
    } else {
        // floor(num / den) from a double estimate, corrected exactly (the
        // estimate is off by at most one; num < 2^56, den < 2^45).
        L = (int64_t)floor((double)num / (double)den);
        if (L * den > num) --L;
        if ((L + 1) * den <= num) ++L;
        if (L < 0 || L >= n) return;
    }
    int q[3];
    const int a = T.axis;
    q[a] = (int)L;
    q[(a + 1) % 3] = i;
    q[(a + 2) % 3] = j;
    const int idx = q[0] + n * (q[1] + n * q[2]);
    seeds[idx] = idx;
}

// Lane part of one (triangle, axis) item of a batch: snap, set up, rasterize a small
// projection directly; returns true when the projection is large and left to
// the whole wavefront.
__device__ __forceinline__ bool vox_item(const float *__restrict__ v, int nv, const int32_t *__restrict__ f, int t,
                                         int axis, const rtsdf_grid &g, int32_t *__restrict__ seeds, VoxTri &T)
{
    int vid[3] = {f[3 * t], f[3 * t + 1], f[3 * t + 2]};
    for (int k = 0; k < 3; ++k)
        if (vid[k] < 0 || vid[k] >= nv) {
            if (axis == 0) raise_error(RTSDF_ERR_FACE_INDEX);
            return false;
        }
    int64_t X[3][3];
    for (int k = 0; k < 3; ++k)
        if (!snap(v, vid[k], g, X[k])) {
            if (axis == 0) raise_error(RTSDF_ERR_VERTEX_RANGE);
            return false;
        }
    if (!vox_setup(X, axis, g.n, T)) return false;
    const int npix = (T.i1 - T.i0 + 1) * (T.j1 - T.j0 + 1);
    if (npix <= kSmallPixels) {
        for (int j = T.j0; j <= T.j1; ++j)
            for (int i = T.i0; i <= T.i1; ++i) vox_column(T, i, j, g.n, seeds);
        return false;
    }
    return true;
}

// Large projections of the wavefront's lanes in a batch, rasterized by all 64
// lanes in turn; `seeds` / `n` may differ per lane (many scenes per launch).
__device__ __forceinline__ void vox_wave_big(bool big, const VoxTri &T, int32_t *seeds, int n)
{
    const int lane = threadIdx.x & (kWave - 1);
    uint64_t pending = __ballot(big);
    while (pending) {
        const int src = __ffsll((unsigned long long)pending) - 1;
        pending &= pending - 1;
        VoxTri B;
        for (int k = 0; k < 3; ++k) {
            B.px[k] = __shfl(T.px[k], src);
            B.py[k] = __shfl(T.py[k], src);
            B.z[k] = __shfl(T.z[k], src);
        }
        B.area2 = __shfl(T.area2, src);
        B.i0 = __shfl(T.i0, src);
        B.i1 = __shfl(T.i1, src);
        B.j0 = __shfl(T.j0, src);
        B.j1 = __shfl(T.j1, src);
        B.axis = __shfl(T.axis, src);
        int32_t *bs = reinterpret_cast<int32_t *>(__shfl((long long)reinterpret_cast<intptr_t>(seeds), src));
        const int bn = __shfl(n, src);
        const int w = B.i1 - B.i0 + 1;
        const int npix = w * (B.j1 - B.j0 + 1);
        for (int p = lane; p < npix; p += kWave) vox_column(B, B.i0 + p % w, B.j0 + p / w, bn, bs);
    }
}

// Threads per workgroup and fewest workgroups (four for each compute unit, so a small mesh's large projections do not
// share one).  With 1024 threads a million triangles at 256^3 take 175 us, with 512 151, with 256 146, but 1,880 large
// ones 54, 54 and 68; four consecutive triangles per workgroup (their faces in one cache line) 208 and 111.
constexpr int kVoxThreads = 512;
constexpr int kVoxBlocks = 1024;
constexpr int kWavePixels = 512;   // largest projection a single wavefront takes
constexpr int kSmallExtent = 8192;  // 32 voxels, also outside the grid: edge functions below 2^28 in 32 bits

// A vertex snapped to 1/256 voxel; POW2: the voxel size is a power of two, so its inverse is exact and multiplies.
template <bool POW2>
__device__ __forceinline__ bool snap32(const float *__restrict__ v, const rtsdf_grid &g, double inv_h, int32_t X[3])
{
    const double side = (double)g.n * (double)g.h;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double rel = (double)v[a] - (double)g.lo[a];
        if (!(rel >= -side && rel <= 2.0 * side)) return false;
        X[a] = (int32_t)__builtin_rint((POW2 ? rel * inv_h : rel / (double)g.h) * 256.0);
    }
    return true;
}

// One projection by one lane.  Returns true when it is left to more lanes: many columns, or long edges.
__device__ __forceinline__ bool vox_small(const int32_t (&X)[3][3], int axis, int n, int32_t *__restrict__ seeds)
{
    const int e1 = (axis + 1) % 3, e2 = (axis + 2) % 3;
    const int32_t x0 = X[0][e1], x1 = X[1][e1], x2 = X[2][e1], y0 = X[0][e2], y1 = X[1][e2], y2 = X[2][e2];
    const int32_t minx = min(x0, min(x1, x2)), maxx = max(x0, max(x1, x2));
    const int32_t miny = min(y0, min(y1, y2)), maxy = max(y0, max(y1, y2));
    // column centre 256 i + 128 within [min, max]
    const int i0 = max((minx + 127) >> 8, 0), i1 = min((maxx - 128) >> 8, n - 1);
    const int j0 = max((miny + 127) >> 8, 0), j1 = min((maxy - 128) >> 8, n - 1);
    if (i0 > i1 || j0 > j1) return false;
    if (maxx - minx > kSmallExtent || maxy - miny > kSmallExtent || (i1 - i0 + 1) * (j1 - j0 + 1) > kSmallPixels)
        return true;
    int32_t area = (x1 - x0) * (y2 - y0) - (y1 - y0) * (x2 - x0);
    if (area == 0) return false;
    // edge functions times the orientation: all >= 0 inside or on the boundary, their sum |area|
    const int32_t s = area < 0 ? -1 : 1;
    area *= s;
    const double den = (double)area * 256.0, inv = 1.0 / den;
    const double z0 = X[0][axis], z1 = X[1][axis], z2 = X[2][axis];
    const int sx = axis == 0 ? n : axis == 1 ? n * n : 1, sy = axis == 0 ? n * n : axis == 1 ? 1 : n;
    const int sz = axis == 0 ? 1 : axis == 1 ? n : n * n;
    for (int j = j0; j <= j1; ++j) {
        const int32_t cy = 256 * j + 128;
        for (int i = i0; i <= i1; ++i) {
            const int32_t cx = 256 * i + 128;
            const int32_t w0 = s * ((x2 - x1) * (cy - y1) - (y2 - y1) * (cx - x1));
            const int32_t w1 = s * ((x0 - x2) * (cy - y2) - (y0 - y2) * (cx - x2));
            const int32_t w2 = area - w0 - w1;
            if ((w0 | w1 | w2) < 0) continue;
            // depth num / den, every product and sum below 2^53: exact
            const double num = (double)w0 * z0 + (double)w1 * z1 + (double)w2 * z2;
            double L = floor(num * inv);  // off by at most one
            const double rem = fma(-L, den, num);
            if (rem < 0.0) L -= 1.0;
            else if (rem >= den) L += 1.0;
            if (num == (double)n * den) L = (double)(n - 1);
            if (L < 0.0 || L >= (double)n) continue;
            const int idx = (int)L * sz + i * sx + j * sy;
            seeds[idx] = idx;
        }
    }
    return false;
}

// One projection by many lanes: lane (lx, ly) of a block of 64 x ny columns.
__device__ __forceinline__ void vox_wide(const int32_t (&X32)[3][3], int axis, int n, int lx, int ly, int ny,
                                         int32_t *__restrict__ seeds)
{
    int64_t X[3][3];
    for (int k = 0; k < 3; ++k)
        for (int a = 0; a < 3; ++a) X[k][a] = X32[k][a];
    VoxTri T;
    if (!vox_setup(X, axis, n, T)) return;
    for (int j = T.j0 + ly; j <= T.j1; j += ny)
        for (int i = T.i0 + lx; i <= T.i1; i += kWave) vox_column(T, i, j, n, seeds);
}

template <bool POW2>
__global__ void __launch_bounds__(kVoxThreads) voxelize_kernel(const float *__restrict__ v, int nv,
                                                               const int32_t *__restrict__ f, int nt, rtsdf_grid g,
                                                               double inv_h, int32_t *__restrict__ seeds)
{
    __shared__ uint32_t big[3 * kVoxThreads];  // projections left to the workgroup: thread << 2 | axis
    __shared__ uint32_t nbig;
    if (threadIdx.x == 0) nbig = 0u;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const auto tri_of = [&](uint32_t thread) { return (int64_t)thread * gridDim.x + blockIdx.x; };
    const auto load = [&](int64_t t, int32_t (&X)[3][3]) {  // 0, or the error bit
        for (int k = 0; k < 3; ++k) {
            const int vi = f[3 * t + k];
            if (vi < 0 || vi >= nv) return (uint32_t)RTSDF_ERR_FACE_INDEX;
            X[k][0] = vi;
        }
        for (int k = 0; k < 3; ++k)
            if (!snap32<POW2>(v + 3 * (int64_t)X[k][0], g, inv_h, X[k])) return (uint32_t)RTSDF_ERR_VERTEX_RANGE;
        return 0u;
    };
    const int64_t t = tri_of(threadIdx.x);
    int32_t X[3][3];
    uint32_t wide = 0;  // axes left to the wavefront
    if (t < nt) {
        const uint32_t err = load(t, X);
        if (err) raise_error(err);
        else
            for (int axis = 0; axis < 3; ++axis)
                if (vox_small(X, axis, g.n, seeds)) {
                    // columns of the box in the grid, as above
                    const int e1 = (axis + 1) % 3, e2 = (axis + 2) % 3;
                    const int w = min((max(X[0][e1], max(X[1][e1], X[2][e1])) - 128) >> 8, g.n - 1) -
                                  max((min(X[0][e1], min(X[1][e1], X[2][e1])) + 127) >> 8, 0) + 1;
                    const int h = min((max(X[0][e2], max(X[1][e2], X[2][e2])) - 128) >> 8, g.n - 1) -
                                  max((min(X[0][e2], min(X[1][e2], X[2][e2])) + 127) >> 8, 0) + 1;
                    if (w * h <= kWavePixels) wide |= 1u << axis;
                    else big[atomicAdd(&nbig, 1u)] = threadIdx.x << 2 | (uint32_t)axis;
                }
    }
    // the wavefront's projections, one after another
    for (int axis = 0; axis < 3; ++axis) {
        uint64_t pending = __ballot((wide >> axis & 1u) != 0u);
        while (pending) {
            const int src = __ffsll((unsigned long long)pending) - 1;
            pending &= pending - 1;
            int32_t B[3][3];
            for (int k = 0; k < 3; ++k)
                for (int a = 0; a < 3; ++a) B[k][a] = __builtin_amdgcn_readlane(X[k][a], src);
            int64_t B64[3][3];
            for (int k = 0; k < 3; ++k)
                for (int a = 0; a < 3; ++a) B64[k][a] = B[k][a];
            VoxTri T;
            if (!vox_setup(B64, axis, g.n, T)) continue;
            const int w = T.i1 - T.i0 + 1, npix = w * (T.j1 - T.j0 + 1);
            for (int p = lane; p < npix; p += kWave) vox_column(T, T.i0 + p % w, T.j0 + p / w, g.n, seeds);
        }
    }
    __syncthreads();
    const uint32_t n = nbig;
    for (uint32_t q = 0; q < n; ++q) {
        const uint32_t e = big[q];
        int32_t B[3][3];
        (void)load(tri_of(e >> 2), B);  // (checked by its own lane)
        vox_wide(B, (int)(e & 3u), g.n, lane, threadIdx.x >> 6, kVoxThreads / kWave, seeds);
    }
}

}  // namespace rtsdf

extern "C" int rtsdf_voxelize(const float *vertices, int32_t nv, const int32_t *faces, int32_t nt,
                              rtsdf_grid coarse, int32_t *seeds, rtsdf_stream stream)
{
    using namespace rtsdf;
    if (!grid_ok(coarse) || !is_pow2(coarse.n) || coarse.n < 8 || coarse.n > 256) return RTSDF_EINVAL;
    if (!seeds || nv < 0 || nt < 0 || (nt > 0 && (!vertices || !faces))) return RTSDF_EINVAL;
    if ((int64_t)nt * 3 > (int64_t)INT32_MAX) return RTSDF_EINVAL;
    hipStream_t s = as_stream(stream);
    const int64_t nvox = (int64_t)coarse.n * coarse.n * coarse.n;
    int rc = launch_fill<int32_t>(seeds, -1, nvox, s);
    if (rc != RTSDF_OK) return rc;
    if (nt == 0) return RTSDF_OK;
    const int blocks = std::max((nt + kVoxThreads - 1) / kVoxThreads, std::min(nt, kVoxBlocks));
    const dim3 grid((unsigned)blocks), block(kVoxThreads);
    int e = 0;
    const double inv_h = 1.0 / (double)coarse.h;
    if (frexpf(coarse.h, &e) == 0.5f)  // a power of two
        voxelize_kernel<true><<<grid, block, 0, s>>>(vertices, nv, faces, nt, coarse, inv_h, seeds);
    else
        voxelize_kernel<false><<<grid, block, 0, s>>>(vertices, nv, faces, nt, coarse, inv_h, seeds);
    RTSDF_CHECK_LAUNCH();
    return RTSDF_OK;
}
