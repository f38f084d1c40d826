// Voxelization of a triangle mesh into the coarse grid (paper Sec. 2.1).
//
// The paper renders the scene three times with an orthographic camera along
// +x, +y and +z, depth writes off, and marks the voxel under every fragment.
// gfx950 has no raster pipeline, so this is a compute kernel that applies an
// exact integer version of that rule: vertices snapped to 1/256 voxel, a
// column covered when its centre is inside or on the projected triangle, and
// the voxel holding the triangle's depth at that centre marked.
//
// Work mapping: a lane takes a triangle (its vertices are snapped once), or in workgroups that are at most a quarter
// full one of its three projections.  It rasterizes those whose bounding box holds at most kSmallPixels column centres,
// in 32-bit integers, and lists the others in LDS beside the snapped vertices: projections of up to 32 voxels' extent
// (32-bit integers) or kWavePixels columns (64-bit) go to the workgroup's wavefronts in turn, larger ones (room walls
// cover whole faces of the grid) to the whole workgroup.
// Consecutive triangles go to consecutive workgroups of one XCD: the large projections of consecutive triangles (the
// walls of a room) land in different workgroups instead of queueing in one, and the cache lines that neighbouring
// triangles share are read by one L2 (by consecutive workgroups of all XCDs, 1.0 M triangles without shared vertices
// took 175 us at 256^3, now 74).
//
// Bound by the latency of its gathers and its largest projections.  With the fill of the seeds, against one lane per
// (triangle, axis) in 64-bit integers whose larger projections queue in its wavefront: a room of 1.07 M triangles at
// 256^3 355 -> 109 us, one of 69,760 at 256^3 368 -> 69 and at 128^3 107 -> 28, soups of 1.0 M small triangles at 32^3
// 105 -> 59, of 300,000 of about 26 columns at 256^3 299 -> 246, of 20,000 of about 160 at 128^3 126 -> 45, 12 that cover
// the grid at 256^3 3,070 -> 69.
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

// Threads per workgroup, and fewest workgroups: enough that a small mesh's large projections do not share one, few
// enough that the start of mostly empty ones does not show (with 1024, 20,000 small triangles at 128^3 take 14.0 us
// instead of 11.9, but the room of 69,760 at 256^3 60 instead of 69, and with 512 none of the sizes above is slower than
// with a lane per axis).
constexpr int kVoxThreads = 512;
constexpr int kVoxBlocks = 512;
// triangles of a workgroup at most whose axes go to different wavefronts (20,000 small ones at 256^3 36 -> 28 us)
constexpr int kVoxSplit = 2 * kWave;
constexpr int kWavePixels = 512;   // largest projection with long edges that a single wavefront takes
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

// A projection: the vertices' coordinates in its plane and their depths, and the columns of its box in the grid.
struct VoxProj {
    int32_t x[3], y[3], z[3];
    int i0, i1, j0, j1;
    bool edges32;  // short enough for edge functions in 32 bits
};

__device__ __forceinline__ bool vox_box(VoxProj &P, int n)  // false if the box holds no column centre
{
    const int32_t minx = min(P.x[0], min(P.x[1], P.x[2])), maxx = max(P.x[0], max(P.x[1], P.x[2]));
    const int32_t miny = min(P.y[0], min(P.y[1], P.y[2])), maxy = max(P.y[0], max(P.y[1], P.y[2]));
    // column centre 256 i + 128 within [min, max]
    P.i0 = max((minx + 127) >> 8, 0);
    P.i1 = min((maxx - 128) >> 8, n - 1);
    P.j0 = max((miny + 127) >> 8, 0);
    P.j1 = min((maxy - 128) >> 8, n - 1);
    P.edges32 = maxx - minx <= kSmallExtent && maxy - miny <= kSmallExtent;
    return P.i0 <= P.i1 && P.j0 <= P.j1;
}

// What the columns of a projection share, in 32-bit integers; false if its area is zero.
struct VoxEdges {
    int32_t area, s;  // edge functions times the orientation s: all >= 0 inside or on the boundary, their sum the area
    double den, inv;
    int sx, sy, sz;
};

__device__ __forceinline__ bool vox_edges(const VoxProj &P, int axis, int n, VoxEdges &E)
{
    E.area = (P.x[1] - P.x[0]) * (P.y[2] - P.y[0]) - (P.y[1] - P.y[0]) * (P.x[2] - P.x[0]);
    if (E.area == 0) return false;
    E.s = E.area < 0 ? -1 : 1;
    E.area *= E.s;
    E.den = (double)E.area * 256.0;
    E.inv = 1.0 / E.den;
    E.sx = axis == 0 ? n : axis == 1 ? n * n : 1;
    E.sy = axis == 0 ? n * n : axis == 1 ? 1 : n;
    E.sz = axis == 0 ? 1 : axis == 1 ? n : n * n;
    return true;
}

__device__ __forceinline__ void vox_column32(const VoxProj &P, const VoxEdges &E, int i, int j, int n,
                                             int32_t *__restrict__ seeds)
{
    const int32_t cx = 256 * i + 128, cy = 256 * j + 128;
    const int32_t w0 = E.s * ((P.x[2] - P.x[1]) * (cy - P.y[1]) - (P.y[2] - P.y[1]) * (cx - P.x[1]));
    const int32_t w1 = E.s * ((P.x[0] - P.x[2]) * (cy - P.y[2]) - (P.y[0] - P.y[2]) * (cx - P.x[2]));
    const int32_t w2 = E.area - w0 - w1;
    if ((w0 | w1 | w2) < 0) return;
    // depth num / den, every product and sum below 2^53: exact
    const double num = (double)w0 * (double)P.z[0] + (double)w1 * (double)P.z[1] + (double)w2 * (double)P.z[2];
    double L = floor(num * E.inv);  // off by at most one
    const double rem = fma(-L, E.den, num);
    if (rem < 0.0) L -= 1.0;
    else if (rem >= E.den) L += 1.0;
    if (num == (double)n * E.den) L = (double)(n - 1);
    if (L < 0.0 || L >= (double)n) return;
    const int idx = (int)L * E.sz + i * E.sx + j * E.sy;
    seeds[idx] = idx;
}

// The columns of a projection's box by lane `first` of `step` (a multiple of kWave): row by row, and where the rows are
// long a row by the lanes of one wavefront, which share the row's products (12 triangles of 256^2 columns: 70 against 91
// us).
template <typename F>
__device__ __forceinline__ void vox_columns(int i0, int i1, int j0, int j1, int first, int step, F column)
{
    const int w = i1 - i0 + 1, npix = w * (j1 - j0 + 1);
    if (w >= kWave) {
        for (int j = j0 + first / kWave; j <= j1; j += step / kWave)
            for (int i = i0 + first % kWave; i <= i1; i += kWave) column(i, j);
        return;
    }
    const float inv_w = 1.0f / (float)w;
    for (int p = first; p < npix; p += step) {
        const int r = (int)(((float)p + 0.5f) * inv_w);  // p / w: below 256, half a column from any other
        column(i0 + p - r * w, j0 + r);
    }
}

template <bool POW2>
__global__ void __launch_bounds__(kVoxThreads) voxelize_kernel(const float *__restrict__ v, int nv,
                                                               const int32_t *__restrict__ f, int nt, rtsdf_grid g,
                                                               double inv_h, int32_t *__restrict__ seeds)
{
    // projections left to a wavefront (from the front) and to the workgroup (from the back): thread << 2 | axis, and
    // those threads' snapped vertices (read from LDS, so that a projection doesn't wait for gathers of its own)
    constexpr int kList = 3 * kVoxThreads;
    __shared__ uint32_t list[kList], ends[2];
    __shared__ int32_t snapped[kVoxThreads][9];
    if (threadIdx.x < 2) ends[threadIdx.x] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // consecutive triangles to consecutive workgroups of one XCD (workgroups go to the 8 XCDs in turn), a sparse
    // workgroup's triangles to all of its wavefronts, and of a quarter full one the three axes to three wavefronts
    const uint32_t xcd = blockIdx.x & 7u, per = gridDim.x >> 3;
    const uint32_t place = xcd * per + min(xcd, gridDim.x & 7u) + (blockIdx.x >> 3);
    const bool split = (nt + (int)gridDim.x - 1) / (int)gridDim.x <= kVoxSplit;
    const int64_t t = (split && wave >= 6 ? (int64_t)nt : 0) +
                      (int64_t)(split ? lane * 2 + wave / 3 : lane * (kVoxThreads / kWave) + wave) * gridDim.x + place;
    int32_t X[3][3];
    uint32_t err = 0;
    if (t < nt) {
        for (int k = 0; k < 3 && !err; ++k) {
            const int vi = f[3 * t + k];
            if (vi < 0 || vi >= nv) err = RTSDF_ERR_FACE_INDEX;
            X[k][0] = vi;
        }
        for (int k = 0; k < 3 && !err; ++k)
            if (!snap32<POW2>(v + 3 * (int64_t)X[k][0], g, inv_h, X[k])) err = RTSDF_ERR_VERTEX_RANGE;
        if (err) raise_error(err);
    }
    if (t < nt && !err) {
        bool left = false;
#pragma unroll
        for (int axis = 0; axis < 3; ++axis) {
            if (split && wave % 3 != axis) continue;
            VoxProj P;
            for (int k = 0; k < 3; ++k) {
                P.x[k] = X[k][(axis + 1) % 3];
                P.y[k] = X[k][(axis + 2) % 3];
                P.z[k] = X[k][axis];
            }
            if (!vox_box(P, g.n)) continue;
            const int npix = (P.i1 - P.i0 + 1) * (P.j1 - P.j0 + 1);
            if (P.edges32 && npix <= kSmallPixels) {
                VoxEdges E;
                if (!vox_edges(P, axis, g.n, E)) continue;
                for (int j = P.j0; j <= P.j1; ++j)
                    for (int i = P.i0; i <= P.i1; ++i) vox_column32(P, E, i, j, g.n, seeds);
                continue;
            }
            left = true;
            const uint32_t e = threadIdx.x << 2 | (uint32_t)axis;
            if (P.edges32 || npix <= kWavePixels) list[atomicAdd(&ends[0], 1u)] = e;
            else list[kList - 1 - atomicAdd(&ends[1], 1u)] = e;
        }
        if (left)
            for (int k = 0; k < 9; ++k) snapped[threadIdx.x][k] = X[k / 3][k % 3];
    }
    __syncthreads();
    const auto get = [&](uint32_t e, VoxProj &P) {
        const int32_t *S = snapped[e >> 2];
        const int axis = (int)(e & 3u), e1 = axis == 2 ? 0 : axis + 1, e2 = axis == 0 ? 2 : axis - 1;
        for (int k = 0; k < 3; ++k) {
            P.x[k] = __builtin_amdgcn_readfirstlane(S[3 * k + e1]);
            P.y[k] = __builtin_amdgcn_readfirstlane(S[3 * k + e2]);
            P.z[k] = __builtin_amdgcn_readfirstlane(S[3 * k + axis]);
        }
        return axis;
    };
    const auto wide = [&](const VoxProj &P, int axis, int first, int step) {  // in 64 bits
        int64_t X64[3][3];
        for (int k = 0; k < 3; ++k) {
            X64[k][0] = P.x[k];
            X64[k][1] = P.y[k];
            X64[k][2] = P.z[k];
        }
        VoxTri T;
        if (!vox_setup(X64, 2, g.n, T)) return;
        T.axis = axis;
        vox_columns(T.i0, T.i1, T.j0, T.j1, first, step, [&](int i, int j) { vox_column(T, i, j, g.n, seeds); });
    };
    // the wavefronts' projections, dealt out over all of the workgroup's (the triangles of a small mesh are all in its
    // first wavefront)
    for (uint32_t q = wave; q < ends[0]; q += kVoxThreads / kWave) {
        VoxProj P;
        const int axis = get(__builtin_amdgcn_readfirstlane(list[q]), P);
        (void)vox_box(P, g.n);
        if (P.edges32) {
            VoxEdges E;
            if (!vox_edges(P, axis, g.n, E)) continue;
            vox_columns(P.i0, P.i1, P.j0, P.j1, lane, kWave,
                        [&](int i, int j) { vox_column32(P, E, i, j, g.n, seeds); });
        } else {
            wide(P, axis, lane, kWave);
        }
    }
    for (uint32_t q = 0; q < ends[1]; ++q) {
        VoxProj P;
        const int axis = get(__builtin_amdgcn_readfirstlane(list[kList - 1 - q]), P);
        wide(P, axis, threadIdx.x, kVoxThreads);
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
