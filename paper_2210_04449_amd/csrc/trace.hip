// Fine-SDF ray tracing and temporal accumulation (paper Sec. 2.2, Eq. (1)),
// the vertex gradient of the traced distances, and two helper entry points
// (directions, closest hits) that expose the same arithmetic.
//
// Per selected texel and frame, rays_per_texel rays leave the texel centre
// towards uniformly random points of the unit sphere; each ray's closest hit
// distance is found in the bounding volume hierarchy; the smallest of the
// frame is r_t, which enters Eq. (1); front/back counts of the closest hits
// vote the sign.
//
// Random directions: Philox4x64 with 10 rounds (Salmon et al., SC'11) keyed
// by (seed, 0) with counter (texel, frame << 32 | ray, scene, attempt); 32-bit
// halves become odd multiples of 2^-23 in (-1, 1); Marsaglia's 1972 mapping of
// the first pair inside the unit disc gives the direction.  Every float
// operation there is an explicitly rounded intrinsic, so the directions are
// reproducible bit for bit on any IEEE machine.
//
// Closest hit: software traversal of the two-wide hierarchy with a per-lane
// stack in LDS (its depth is the hierarchy's depth, so it never overflows)
// and the watertight ray/triangle test of Woop, Benthin and Wald (JCGT 2013):
// vertices are mapped into a ray space where the ray is the +z axis (a
// per-ray affine map: axis permutation plus shear), 2D edge functions decide
// coverage (re-evaluated in double when one is exactly zero), so a ray that
// crosses a shared edge hits at least one of its triangles.  Ties in t go to
// the lower triangle index; t must be > 0.
//
// Entry points: the rays of a tile start in one small block, so the upper
// levels of the hierarchy are the same work for all of them.  The queued loop
// opens those levels once per tile (tile_setup) and starts each ray from the
// subtrees it can meet.
//
// Work distribution: persistent wavefronts; one lane owns one selected texel
// and traces its rays one after another.  Lanes whose texel is finished are
// refilled from the compacted queue by one atomic add per wavefront (ballot +
// mbcnt to hand out the slots), so the queue is consumed in Morton order and
// no lane waits for a whole wavefront of texels to finish.
#include <algorithm>

#include "common.hpp"

namespace rtsdf {

// ------------------------------------------------------------------ RNG ----

// a * b in full: four 32-bit multiply-adds whose partial sums serve both halves (a product per half, from
// __umul64hi and *, repeats the cross products: 7 multiplies)
__device__ __forceinline__ void mul_wide(uint64_t a, uint64_t b, uint64_t &hi, uint64_t &lo)
{
    const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
    const uint64_t p00 = (uint64_t)a0 * b0;
    const uint64_t p10 = (uint64_t)a1 * b0 + (p00 >> 32);
    const uint64_t p01 = (uint64_t)a0 * b1 + (uint32_t)p10;
    hi = (uint64_t)a1 * b1 + (p10 >> 32) + (p01 >> 32);
    lo = (p01 << 32) | (uint32_t)p00;
}

__device__ __forceinline__ void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1)
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += W0;
            k1 += W1;
        }
        uint64_t hi0, lo0, hi1, lo1;
        mul_wide(M0, c[0], hi0, lo0);
        mul_wide(M1, c[2], hi1, lo1);
        const uint64_t y0 = hi1 ^ c[1] ^ k0, y2 = hi0 ^ c[3] ^ k1;
        c[0] = y0;
        c[1] = lo1;
        c[2] = y2;
        c[3] = lo0;
    }
}

__device__ __forceinline__ float uniform_pm1(uint32_t h)
{
    return (float)((int32_t)((h >> 9) << 1) + 1 - 8388608) * 0x1p-23f;
}

__device__ __forceinline__ float3 sphere_dir(uint64_t seed, uint32_t texel, uint32_t frame, uint32_t ray, uint32_t scene)
{
    for (uint32_t attempt = 0; attempt < 8; ++attempt) {
        uint64_t c[4] = {(uint64_t)texel, ((uint64_t)frame << 32) | ray, (uint64_t)scene, (uint64_t)attempt};
        philox4x64_10(c, seed, 0);
        // the first of the four pairs inside the disc (without branches: some lane of a wavefront needs the third
        // or fourth pair nearly every time)
        float x1 = 0.0f, x2 = 0.0f, s = 2.0f;
#pragma unroll
        for (int p = 3; p >= 0; --p) {
            const float y1 = uniform_pm1((uint32_t)c[p]);
            const float y2 = uniform_pm1((uint32_t)(c[p] >> 32));
            const float t = rn_add(rn_mul(y1, y1), rn_mul(y2, y2));
            const bool in = t < 1.0f;
            x1 = in ? y1 : x1;
            x2 = in ? y2 : x2;
            s = in ? t : s;
        }
        if (s < 1.0f) {
            const float q = rn_sqrt(rn_sub(1.0f, s));
            return make_float3(rn_mul(rn_mul(2.0f, x1), q), rn_mul(rn_mul(2.0f, x2), q),
                               rn_sub(1.0f, rn_mul(2.0f, s)));
        }
    }
    return make_float3(0.0f, 0.0f, 1.0f);
}

// texel centre: lo + (i + 1/2) h per axis, float ops rounded once each
__device__ __forceinline__ float texel_coord(float lo, int i, float h)
{
    return rn_add(lo, rn_mul(rn_add((float)i, 0.5f), h));
}

// ------------------------------------------------------------- geometry ----

struct RaySetup {
    float ix, iy, iz;    // 1 / direction (zero components replaced by +-1e-12)
    float oix, oiy, oiz; // origin * inverse
    float ox, oy, oz;    // origin
    float dx, dy, dz;    // direction
};

// |direction|, which turns a hit's ray parameter into a distance (computed where it is needed, from the
// stored direction, so the traversal loop does not keep it; the fused multiply-adds are spelled out so every
// kernel rounds it alike)
__device__ __forceinline__ float ray_len(const RaySetup &R)
{
    return __builtin_amdgcn_sqrtf(fmaf(R.dz, R.dz, fmaf(R.dy, R.dy, R.dx * R.dx)));
}

__device__ __forceinline__ float safe_inv(float d)
{
    const float a = fabsf(d) < 1e-12f ? copysignf(1e-12f, d) : d;
    return __builtin_amdgcn_rcpf(a);
}

__device__ __forceinline__ void ray_setup(float ox, float oy, float oz, float dx, float dy, float dz, RaySetup &R)
{
    R.ix = safe_inv(dx);
    R.iy = safe_inv(dy);
    R.iz = safe_inv(dz);
    R.oix = ox * R.ix;
    R.oiy = oy * R.iy;
    R.oiz = oz * R.iz;
    R.ox = ox;
    R.oy = oy;
    R.oz = oz;
    R.dx = dx;
    R.dy = dy;
    R.dz = dz;
}

// Watertight ray/triangle test (Woop, Benthin and Wald 2013): the vertices are
// taken into a ray space where the ray is the +z axis (permute so the largest
// direction component is z, then shear), and the three 2-D edge functions
// decide; edges shared by two triangles get the same values in both, so no
// ray passes between them.  Zero edge functions are recomputed in double
// precision.  Returns t of a front-face hit, -t of a back-face hit, 0 for a
// miss (hits have t > 0).
__device__ __noinline__ float tri_watertight(float ox, float oy, float oz, float dx, float dy, float dz,
                                             const float4 *tp)
{
    const float4 a = tp[0], b = tp[1], c = tp[2];
    const float ax = fabsf(dx), ay = fabsf(dy), az = fabsf(dz);
    int kz = ay > ax ? 1 : 0;
    if (az > fmaxf(ax, ay)) kz = 2;
    int kx = kz == 2 ? 0 : kz + 1;
    int ky = kx == 2 ? 0 : kx + 1;
    const float d[3] = {dx, dy, dz};
    if (d[kz] < 0.0f) {
        const int t = kx;
        kx = ky;
        ky = t;
    }
    // the shear only has to be the same for every triangle a ray meets, not correctly rounded
    const float Sz = __builtin_amdgcn_rcpf(d[kz]), Sx = d[kx] * Sz, Sy = d[ky] * Sz;
    const float o[3] = {ox, oy, oz};
    const float va[3] = {a.x - o[0], a.y - o[1], a.z - o[2]};
    const float vb[3] = {b.x - o[0], b.y - o[1], b.z - o[2]};
    const float vc[3] = {c.x - o[0], c.y - o[1], c.z - o[2]};
    const float Ax = va[kx] - Sx * va[kz], Ay = va[ky] - Sy * va[kz];
    const float Bx = vb[kx] - Sx * vb[kz], By = vb[ky] - Sy * vb[kz];
    const float Cx = vc[kx] - Sx * vc[kz], Cy = vc[ky] - Sy * vc[kz];
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    if (U == 0.0f || V == 0.0f || W == 0.0f) {
        U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
        V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
        W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
    }
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return 0.0f;
    const float det = U + V + W;
    if (det == 0.0f) return 0.0f;
    const float T = U * (Sz * va[kz]) + V * (Sz * vb[kz]) + W * (Sz * vc[kz]);
    const float t = T / det;
    // T is past the largest float where large triangles are far: a t of +inf would equal the bound of a ray that has met
    // nothing yet, which has no triangle whose id could be compared
    if (!(t > 0.0f && t <= 3.0e38f)) return 0.0f;
    return det > 0.0f ? t : -t;
}

// Fast test through the triangle's precomputed map (see the scene layout):
// t from the plane coordinate, then the barycentrics at the crossing.  Where
// the smallest barycentric is within a rounding margin of zero -- the ray
// passes near an edge or a vertex -- the decision is left to the watertight
// test, so rays cannot slip between neighbouring triangles.  Updates the
// closest hit (t, leaf-order index) with ties going to the lower original
// triangle id.
constexpr float kEdgeMargin = 0x1p-12f;  // relative to the magnitude of the terms of the barycentrics

// Whether the ray (origin o, direction d) meets the triangle at leaf-order index i (rows r0, r1, r2 of its
// map) at some 0 < t <= tlim; the distance t and the facing (front: the ray meets the front face).  The
// decision and t do not depend on tlim, which only filters the result: whichever bound a traversal holds when
// it tests the triangle, the closest hit over all tested triangles is the same.
__device__ __forceinline__ bool tri_hit_rows(float ox, float oy, float oz, float dx, float dy, float dz, float4 r0,
                                             float4 r1, float4 r2, const float4 *tris, int i, float tlim, float &t,
                                             bool &fr)
{
    const float pz = fmaf(r2.x, ox, fmaf(r2.y, oy, fmaf(r2.z, oz, r2.w)));
    const float qz = fmaf(r2.x, dx, fmaf(r2.y, dy, r2.z * dz));
    const float p0 = fmaf(r0.x, ox, fmaf(r0.y, oy, fmaf(r0.z, oz, r0.w)));
    const float q0 = fmaf(r0.x, dx, fmaf(r0.y, dy, r0.z * dz));
    const float p1 = fmaf(r1.x, ox, fmaf(r1.y, oy, fmaf(r1.z, oz, r1.w)));
    const float q1 = fmaf(r1.x, dx, fmaf(r1.y, dy, r1.z * dz));
    t = -pz * __builtin_amdgcn_rcpf(qz);
    const float b1 = fmaf(t, q0, p0), b2 = fmaf(t, q1, p1);
    const float bmin = fminf(1.0f - b1 - b2, fminf(b1, b2));
    const float margin = kEdgeMargin * (fmaf(t, fabsf(q0) + fabsf(q1), fabsf(p0) + fabsf(p1)) + 1.0f);
    const bool in_range = t > 0.0f && t <= 3.0e38f;
    bool hit = in_range && bmin > margin;
    fr = qz < 0.0f;
    if (in_range && !(bmin > margin) && !(bmin < -margin)) {
        // near an edge or a vertex (or not a number): the watertight test decides
        const float4 *tp = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(tris) + rec48(i));
        const float h = tri_watertight(ox, oy, oz, dx, dy, dz, tp);
        t = fabsf(h);
        fr = h > 0.0f;
        hit = h != 0.0f;
    }
    return hit && t <= tlim;
}

__device__ __forceinline__ void tri_test_rows(const RaySetup &R, float4 r0, float4 r1, float4 r2, const float4 *tris,
                                              int i, float &tbest, int &ibest, bool &front)
{
    float t;
    bool fr;
    if (!tri_hit_rows(R.ox, R.oy, R.oz, R.dx, R.dy, R.dz, r0, r1, r2, tris, i, tbest, t, fr)) return;
    if (t == tbest) {  // equal distances: the lower original triangle id wins
        const float4 *tp = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(tris) + rec48(i));
        const float4 *tb = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(tris) + rec48(ibest));
        if (!(__float_as_int(tp[0].w) < __float_as_int(tb[0].w))) return;
    }
    tbest = t;
    ibest = i;
    front = fr;
}

__device__ __forceinline__ void tri_test(const RaySetup &R, const float4 *tmap, const float4 *tris, int i,
                                         float &tbest, int &ibest, bool &front)
{
    // the whole record in one round trip, and no branch before the decision
    const float4 *mp = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(tmap) + rec48(i));
    tri_test_rows(R, mp[0], mp[1], mp[2], tris, i, tbest, ibest, front);
}

// original id of the triangle at leaf-order index i
__device__ __forceinline__ int tri_id(const float4 *tris, int i)
{
    return __float_as_int(reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(tris) + rec48(i))->w);
}

// slab test against a padded box: whether the ray meets it before tbest (a NaN slab misses), the entry
// distance and the exit distance (capped at tbest)
__device__ __forceinline__ bool box_hit2(const RaySetup &R, float lx, float hx, float ly, float hy, float lz, float hz,
                                         float tbest, float &t_entry, float &t_exit)
{
    const float x0 = fmaf(lx, R.ix, -R.oix), x1 = fmaf(hx, R.ix, -R.oix);
    const float y0 = fmaf(ly, R.iy, -R.oiy), y1 = fmaf(hy, R.iy, -R.oiy);
    const float z0 = fmaf(lz, R.iz, -R.oiz), z1 = fmaf(hz, R.iz, -R.oiz);
    const float tmin = fmaxf(fmaxf(fminf(x0, x1), fminf(y0, y1)), fmaxf(fminf(z0, z1), 0.0f));
    const float tmax = fminf(fminf(fmaxf(x0, x1), fmaxf(y0, y1)), fminf(fmaxf(z0, z1), tbest));
    t_entry = tmin;
    t_exit = tmax;
    return tmin <= tmax;
}

__device__ __forceinline__ bool box_hit(const RaySetup &R, float lx, float hx, float ly, float hy, float lz, float hz,
                                        float tbest, float &t_entry)
{
    float t_exit;
    return box_hit2(R, lx, hx, ly, hy, lz, hz, tbest, t_entry, t_exit);
}

constexpr int kDone = INT32_MIN;

struct BvhView {
    const BvhNode *nodes;
    const float4 *tris;  // vertices (v0 carrying the original id), leaf order
    const float4 *tmap;  // triangle-space maps, leaf order
};

// One traversal step of one lane: an internal node tests both child boxes
// and descends into the nearer hit child (pushing the farther); a leaf tests
// its triangles; then the lane pops.  `stk` points at the lane's stack slot 0
// in LDS, entries `stride` words apart.
template <bool STATS = false>
__device__ __forceinline__ void trav_step(const BvhView &S, const RaySetup &R, int &node, int &sp, int *stk,
                                          int stride, float &tbest, int &ibest, bool &front, uint32_t *nodes_visited = nullptr,
                                          uint32_t *tris_tested = nullptr)
{
    if (node >= 0) {
        if (STATS) ++*nodes_visited;
        const BvhNode *nd = S.nodes + node;
        const float4 a = nd->xy0, b = nd->xy1, z = nd->z01;
        const int4 m = nd->meta;
        float t0, t1;
        const bool h0 = box_hit(R, a.x, a.y, a.z, a.w, z.x, z.y, tbest, t0);
        const bool h1 = box_hit(R, b.x, b.y, b.z, b.w, z.z, z.w, tbest, t1);
        if (h0 && h1) {
            const bool first0 = t0 <= t1;
            stk[sp * stride] = first0 ? m.y : m.x;
            ++sp;
            node = first0 ? m.x : m.y;
            return;
        }
        if (h0 || h1) {
            node = h0 ? m.x : m.y;
            return;
        }
    } else {
        const int first = leaf_first(node), cnt = leaf_count(node);
        if (STATS) *tris_tested += (uint32_t)cnt;
        for (int i = first; i < first + cnt; ++i) tri_test(R, S.tmap, S.tris, i, tbest, ibest, front);
    }
    node = sp > 0 ? stk[--sp * stride] : kDone;
}

// ------------------------------------------------------ persistent tracer ----

// Everything the tracer needs to know about one scene.
struct TraceScene {
    BvhView bvh;
    const BvhNode *nodes4;  // 4-wide copy (WIDE launches)
    int nt;
    const int32_t *queue;
    const int32_t *count;
    int32_t queue_cap;
    const float *coarse_sdf;
    int nc, logr, nf, lognf;
    float lox, loy, loz, hf;
    int rays;
    uint32_t scene_id;
    float alpha;
    int sign_policy;  // RTSDF_SIGN_VOTE or RTSDF_SIGN_SHELL
    float shell;
    float *u;
    uint32_t *hits;
    int32_t *arg_tri;
    int32_t *arg_ray;
    float *fine;
};

struct TraceArgs {
    TraceScene one;              // the scene of a single-scene launch
    const TraceScene *scenes;    // batched launch: per-scene records ...
    const int32_t *tile_offset;  // ... and the first global tile of each scene ([nscenes + 1])
    int nscenes;
    int32_t *cursor;             // global tile counter
    uint32_t frame;
    const uint32_t *frame_ptr;
    uint64_t seed;
    int32_t *spill;              // deep stack entries: [(depth - SL) * spill_stride + lane]
    int spill_stride;            // lanes in the launch
    int bin_directions;          // sort each tile's rays by direction bin
    int tile_cap;                // texels per wavefront tile at most (16, 32 or 64)
    int few_rays;                // single scene: queued loop without entry points (see kFewRays)
    float4 *dirs;                // per wavefront: kTileRays directions, then kTileRays records in bin order
};

constexpr int kTraceWaves = 4;
constexpr int kTileRays = 768;  // rays per wavefront tile
constexpr int kTileTexels = 64;

// frame indices share the argmin record with the ray index (frame << 8 | ray)
constexpr uint32_t kMaxFrame = 1u << 23;

__host__ __device__ __forceinline__ int tile_texels_for(int rays, int cap)
{
    return rays >= kTileRays ? 1 : min(cap, kTileRays / rays);
}

// Texels per tile of a single-scene launch.  A wavefront's time for N rays in tiles of r is about (N / r) (o + r), o
// the cost of setting a tile up in rays, and the launch waits about one tile longer for the last wavefront: r = sqrt(o N) is
// the best size while the launch is short.  o = 100 (30 to 200 measured): a 9 k-triangle mesh at 64^3 / 128^3 with 32
// rays 5,890 -> 5,470 us for 6 updates, 230 k texels x 16 rays 841 -> 635 us, 87 k texels x 4 rays 234 -> 204 us; 734 k
// texels x 4 rays 432 -> 438 us.  Whole records of 64 rays, at least two (one: 220 us for the last but one).
__device__ __forceinline__ int tile_texels_auto(int rays, int cap, int total, int waves)
{
    const float r = __builtin_amdgcn_sqrtf(100.0f * (float)total * (float)rays / (float)waves);
    const int n = max(2 * kWave, ((int)fminf(r, 2.0f * kTileRays) + kWave / 2) & ~(kWave - 1));
    return max(1, min(tile_texels_for(rays, cap), n / rays));
}

typedef __attribute__((address_space(3))) int lds_int;

__device__ __forceinline__ const BvhNode *node_ptr(const BvhNode *base, int node)
{
    return reinterpret_cast<const BvhNode *>(reinterpret_cast<const char *>(base) + (uint32_t)node * 64u);
}

// the same record read through the scalar cache (wave-uniform node index)
typedef __attribute__((address_space(4))) const float sfloat;
__device__ __forceinline__ const sfloat *node_sptr(const BvhNode *base, int node)
{
    return (const sfloat *)(reinterpret_cast<uintptr_t>(base) + (uintptr_t)(uint32_t)node * 64u);
}

__device__ __forceinline__ const float4 *tri_ptr(const float4 *base, int tri)
{
    return reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(base) + rec48(tri));
}

template <int SL>
__device__ __forceinline__ void stack_push(int stride, int &sp, lds_int *stk, int32_t *spill, int v)
{
    if (sp < SL) stk[sp * kWave] = v;
    else spill[__umul24((uint32_t)(sp - SL), (uint32_t)stride)] = v;  // stride < 2^24 lanes
    ++sp;
}

template <int SL>
__device__ __forceinline__ int stack_pop(int stride, int &sp, const lds_int *stk, const int32_t *spill)
{
    if (sp == 0) return kDone;
    --sp;
    int v;
    if (sp < SL) v = stk[sp * kWave];
    else v = spill[__umul24((uint32_t)(sp - SL), (uint32_t)stride)];
    return v;
}

// The same stack by the address of its next entry (queued loop): the address is the register itself, and as a lane's
// entries are kWave words apart in its wavefront's part, the bounds are compares with wave-uniform addresses.
__device__ __forceinline__ void stack_push_at(int stride, lds_int *&top, lds_int *end, int32_t *spill, int v)
{
    if (top < end) *top = v;
    else spill[__umul24((uint32_t)(top - end) / kWave, (uint32_t)stride)] = v;
    top += kWave;
}

// (of a stack that is not empty)
__device__ __forceinline__ int stack_pop_at(int stride, lds_int *&top, lds_int *end, const int32_t *spill)
{
    top -= kWave;
    if (top < end) return *top;
    return spill[__umul24((uint32_t)(top - end) / kWave, (uint32_t)stride)];
}

// One internal node: test both children's boxes, descend into the nearer hit
// child and push the farther one; pop when neither is hit.
template <int SL, bool STATS>
__device__ __forceinline__ void inner_step(const BvhView &S, int stride, const RaySetup &R, int &node, int &sp,
                                           lds_int *stk, int32_t *spill, float tbest, uint32_t &st_nodes)
{
    if (STATS) ++st_nodes;
    const BvhNode *nd = node_ptr(S.nodes, node);
    const float4 a = nd->xy0, b = nd->xy1, z = nd->z01;
    const int4 m = nd->meta;
    float t0, t1;
    const bool h0 = box_hit(R, a.x, a.y, a.z, a.w, z.x, z.y, tbest, t0);
    const bool h1 = box_hit(R, b.x, b.y, b.z, b.w, z.z, z.w, tbest, t1);
    if (h0 && h1) {
        const bool first0 = t0 <= t1;
        stack_push<SL>(stride, sp, stk, spill, first0 ? m.y : m.x);
        node = first0 ? m.x : m.y;
    } else if (h0 || h1) {
        node = h0 ? m.x : m.y;
    } else {
        node = stack_pop<SL>(stride, sp, stk, spill);
    }
}

// Same, but a leaf child is opened at once (its triangle range becomes the
// lane's current work) instead of costing an iteration of its own.
template <int SL, bool STATS>
__device__ __forceinline__ void node_step(const BvhView &S, int stride, const RaySetup &R, int &node, int &sp,
                                          lds_int *stk, int32_t *spill, float tbest, int &tri_cur, int &tri_end,
                                          uint32_t &st_nodes)
{
    if (STATS) ++st_nodes;
    const BvhNode *nd = node_ptr(S.nodes, node);
    const float4 a = nd->xy0, b = nd->xy1, z = nd->z01;
    const int4 m = nd->meta;
    float t0, t1;
    const bool h0 = box_hit(R, a.x, a.y, a.z, a.w, z.x, z.y, tbest, t0);
    const bool h1 = box_hit(R, b.x, b.y, b.z, b.w, z.z, z.w, tbest, t1);
    if (h0 && h1) {
        const bool first0 = t0 <= t1;
        const int near = first0 ? m.x : m.y, far = first0 ? m.y : m.x;
        if (near < 0) {
            tri_cur = leaf_first(near);
            tri_end = tri_cur + leaf_count(near);
            node = far;
        } else {
            stack_push<SL>(stride, sp, stk, spill, far);
            node = near;
        }
    } else if (h0 || h1) {
        const int c = h0 ? m.x : m.y;
        if (c < 0) {
            tri_cur = leaf_first(c);
            tri_end = tri_cur + leaf_count(c);
            node = stack_pop<SL>(stride, sp, stk, spill);
        } else {
            node = c;
        }
    } else {
        node = stack_pop<SL>(stride, sp, stk, spill);
    }
}

// One 4-wide node (two records: children 0, 1 in a, b, z, m and 2, 3 in a2,
// b2, z2, m2): test the four boxes, order the hit children by entry
// distance (a five-comparator sorting network), go to the nearest (a leaf
// becomes the triangle range at once, the next nearest child is then next)
// and request pushes of the other hit children, farthest first.
__device__ __forceinline__ void swap_if_greater(float &ta, int &ca, float &tb, int &cb)
{
    const bool sw = ta > tb;
    const float t = sw ? tb : ta;
    tb = sw ? ta : tb;
    ta = t;
    const int c = sw ? cb : ca;
    cb = sw ? ca : cb;
    ca = c;
}

__device__ __forceinline__ void node4_step_regs(const RaySetup &R, float4 a, float4 b, float4 z, int2 m, float4 a2,
                                                float4 b2, float4 z2, int2 m2, int &node, float tbest, int &tri_cur,
                                                int &tri_end, bool &p1, bool &p2, bool &p3, int &v1, int &v2, int &v3,
                                                bool &pop)
{
    const float inf = __builtin_inff();
    float t0, t1, t2, t3;
    const bool h0 = box_hit(R, a.x, a.y, a.z, a.w, z.x, z.y, tbest, t0);
    const bool h1 = box_hit(R, b.x, b.y, b.z, b.w, z.z, z.w, tbest, t1);
    const bool h2 = box_hit(R, a2.x, a2.y, a2.z, a2.w, z2.x, z2.y, tbest, t2);
    const bool h3 = box_hit(R, b2.x, b2.y, b2.z, b2.w, z2.z, z2.w, tbest, t3);
    float e0 = h0 ? t0 : inf, e1 = h1 ? t1 : inf, e2 = h2 ? t2 : inf, e3 = h3 ? t3 : inf;
    int c0 = m.x, c1 = m.y, c2 = m2.x, c3 = m2.y;
    swap_if_greater(e0, c0, e1, c1);
    swap_if_greater(e2, c2, e3, c3);
    swap_if_greater(e0, c0, e2, c2);
    swap_if_greater(e1, c1, e3, c3);
    swap_if_greater(e1, c1, e2, c2);
    const bool any = e0 < inf;
    const bool leaf0 = any && c0 < 0;
    if (leaf0) {
        tri_cur = leaf_first(c0);
        tri_end = tri_cur + leaf_count(c0);
    }
    node = leaf0 ? c1 : c0;
    pop = !any || (leaf0 && !(e1 < inf));
    p3 = e3 < inf;
    p2 = e2 < inf;
    p1 = e1 < inf && !leaf0;
    v1 = c1;
    v2 = c2;
    v3 = c3;
}

// Lanes whose ray is finished (or that have none): a ballot of each compare, combined on the scalar unit (a
// ballot of the combined condition would first be materialised lane by lane).
__device__ __forceinline__ uint64_t wave_done(bool busy, int node, int tri_cur, int tri_end)
{
    return ~__builtin_amdgcn_ballot_w64(busy) |
           (__builtin_amdgcn_ballot_w64(node == kDone) & __builtin_amdgcn_ballot_w64(tri_cur >= tri_end));
}

// Same decisions as node_step, written as selects: the caller performs the
// (at most one) push and the (at most one) pop after the lane's work of the
// iteration, so every lane shares one copy of the stack code.
__device__ __forceinline__ void node_decide(bool h0, bool h1, bool first0, int4 m, int &node, int &tri_cur,
                                            int &tri_end, bool &push, int &push_val, bool &pop)
{
    const bool any = h0 || h1, both = h0 && h1;
    const int near = first0 ? m.x : m.y, far = first0 ? m.y : m.x;
    const bool near_leaf = any && near < 0;
    // a leaf child's triangles become the lane's range; otherwise the range is left empty (the lane is idle,
    // so its range is empty already)
    tri_cur = leaf_first(near);
    tri_end = tri_cur + (near_leaf ? leaf_count(near) : 0);
    // next: the nearer internal child; after a leaf child, the other hit child; else pop
    push = both && !near_leaf;
    push_val = far;
    pop = !any || (near_leaf && !both);
    node = near_leaf ? far : near;
}

__device__ __forceinline__ void node_step_regs(const RaySetup &R, float4 a, float4 b, float4 z, int4 m, int &node,
                                               float tbest, int &tri_cur, int &tri_end, bool &push, int &push_val,
                                               bool &pop)
{
    float t0, t1, e0, e1;
    const bool h0 = box_hit2(R, a.x, a.y, a.z, a.w, z.x, z.y, tbest, t0, e0);
    const bool h1 = box_hit2(R, b.x, b.y, b.z, b.w, z.z, z.w, tbest, t1, e1);
    // the nearer entry first; equal entries (the origin inside both boxes): the child the ray leaves first
    // (bitwise, so the compiler keeps it branch-free)
    const bool second = h1 & ((t1 < t0) | ((t1 == t0) & (e1 < e0)));
    node_decide(h0, h1, h0 & !second, m, node, tri_cur, tri_end, push, push_val, pop);
}

// Queued loop: a lane's pending triangles as one word, their number above the first one's leaf-order index, so that a
// leaf child is unpacked by a rotation and "one pending", "two pending" are compares of the word itself.
constexpr uint32_t kPendOne = 1u << 27;
static_assert(kMaxRefs <= 1 << 26, "an index shifted by the queue entries' six lane bits loses only the number");
__device__ __forceinline__ uint32_t leaf_pending(int code)
{
    return __builtin_amdgcn_alignbit(~(uint32_t)code, ~(uint32_t)code, 5);
}

// node_step's decisions for the queued loop.  The best distance is compared, not folded into the exits (its bits come
// from LDS: a minimum would first have to quiet it), and of two equal entries the first child is taken: rays start at
// their entry points, few of which contain them.
__device__ __forceinline__ void node_step_queued(const RaySetup &R, float4 a, float4 b, float4 z, int2 m, int &node,
                                                 float tbest, uint32_t &pend, bool &push, int &push_val, bool &pop)
{
    const auto slab = [&](float lx, float hx, float ly, float hy, float lz, float hz, float &t) {
        const float x0 = fmaf(lx, R.ix, -R.oix), x1 = fmaf(hx, R.ix, -R.oix);
        const float y0 = fmaf(ly, R.iy, -R.oiy), y1 = fmaf(hy, R.iy, -R.oiy);
        const float z0 = fmaf(lz, R.iz, -R.oiz), z1 = fmaf(hz, R.iz, -R.oiz);
        t = fmaxf(fmaxf(fminf(x0, x1), fminf(y0, y1)), fmaxf(fminf(z0, z1), 0.0f));
        return t <= fminf(fminf(fmaxf(x0, x1), fmaxf(y0, y1)), fmaxf(z0, z1)) && t <= tbest;
    };
    float t0, t1;
    const bool h0 = slab(a.x, a.y, a.z, a.w, z.x, z.y, t0);
    const bool h1 = slab(b.x, b.y, b.z, b.w, z.z, z.w, t1);
    const bool any = h0 || h1, both = h0 && h1;
    const bool first0 = h0 && !(h1 && t1 < t0);
    const int near = first0 ? m.x : m.y, far = first0 ? m.y : m.x;
    const bool near_leaf = any && near < 0;
    pend = near_leaf ? leaf_pending(near) : 0u;
    push = both && !near_leaf;
    push_val = far;
    pop = !any || (near_leaf && !both);
    node = near_leaf ? far : near;
}

__device__ __forceinline__ void node_step_flat(const BvhView &S, const RaySetup &R, int &node, float tbest,
                                               int &tri_cur, int &tri_end, bool &push, int &push_val, bool &pop)
{
    const BvhNode *nd = node_ptr(S.nodes, node);
    node_step_regs(R, nd->xy0, nd->xy1, nd->z01, nd->meta, node, tbest, tri_cur, tri_end, push, push_val, pop);
}

// Octahedral direction bin (8 x 8 cells of the octahedral map, numbered in
// Morton order so consecutive bins are neighbours on the sphere).
constexpr int kBins = 64;
__device__ __forceinline__ int direction_bin(float3 d)
{
    const float s = __builtin_amdgcn_rcpf(fabsf(d.x) + fabsf(d.y) + fabsf(d.z));  // (a bin only orders the rays)
    float u = d.x * s, v = d.y * s;
    if (d.z < 0.0f) {
        const float uu = (1.0f - fabsf(v)) * (u >= 0.0f ? 1.0f : -1.0f);
        const float vv = (1.0f - fabsf(u)) * (v >= 0.0f ? 1.0f : -1.0f);
        u = uu;
        v = vv;
    }
    const int bu = min(7, max(0, (int)((u + 1.0f) * 4.0f)));
    const int bv = min(7, max(0, (int)((v + 1.0f) * 4.0f)));
    return (bu & 1) | ((bv & 1) << 1) | ((bu & 2) << 1) | ((bv & 2) << 2) | ((bu & 4) << 2) | ((bv & 4) << 3);
}

// queued loop: triangle tests queued per wavefront (a power of two, at least two wavefronts' worth)
constexpr int kQueueCap = 128;
constexpr unsigned long long kBestInit = 0x7F800000FFFFFFFFull;  // t = +inf, no triangle
constexpr int kMaxQueuedRefs = 1 << 26;  // queue entries: leaf-order index << 6 | lane
static_assert(2 * kWave <= kQueueCap && (kQueueCap & (kQueueCap - 1)) == 0, "queue size");
static_assert(kBins + kWave <= kQueueCap, "the bin counters share the queue's words");

// Entry points of a tile at most: the bits of two mask words, the last of which marks the end.  At 31, 46 and 62 the
// room (216k triangles, 128^3 / 256^3, 16 rays) traces in 22.4, 21.5 and 21.1 ms and visits 17.9, 15.3 and 13.1 nodes a
// ray, against 28.0 ms and 34.3 without entry points; each entry point costs one box test per ray, at full width.
constexpr int kEntries = 62;
constexpr int kEntryEnd = 63;
constexpr int kEntryStack = 4;  // stack entries per lane whose LDS the two contexts' entry points take
// A node is opened while its box's half area over the squared distance to it from the tile's block (plus the block's
// half diagonal squared) exceeds kOpen: about the chance that a ray meets it, times 8 pi.  4 (one ray in six) and 8 are
// within 0.3 %, 16 costs the smaller scenes 3 %.  kOpenTogether: a round opens every node above this share of the
// round's largest such value, so that the nodes that matter most are open when the 62 run out (0.25: 2 % slower; one
// node at a time, 61 rounds instead of about 25: 4 % slower; all above kOpen: 20 % slower).
constexpr float kOpen = 4.0f, kOpenTogether = 0.5f;
// A single scene whose tiles can have at most this many rays, by their number per texel and the tile_texels of the
// tuning (1 or 2 rays with the default 64), starts its rays at the root: loop shape 5, chosen at launch.  Choosing entry
// points, and their place in the traversal loop, cost more than the node visits they save.  With entry points, 64 texels
// x 1 ray trace 2 to 4 % slower (room-like scene, 128^3 / 256^3: 2,206 against 2,284 us an update), x 2 rays 1.5 %
// slower, x 3 rays 9 % faster (4,243 against 3,864 us).  The line is not that of the tile a launch ends up with: small
// launches of more rays, whose tiles tile_texels_auto cuts down to 128 rays, are as fast or faster with entry points
// (traces of 4 rays: 322 triangles at 32^3 / 64^3 143 against 142 us, a room at 32^3 251 against 257, at 64^3 779
// against 854).  Batches always choose them: of 12 rooms at 64^3 1 ray is 5 % slower (4,410 against 4,189 us a step),
// 2 rays are even (6,200 against 6,190), and of 6 at 128^3 2 rays are 2 % faster (20,365 against 20,684).
constexpr int kFewRays = 128;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) v4f gv4f;
typedef __attribute__((address_space(1))) v2u gv2u;
typedef __attribute__((address_space(1))) const int32_t gint;

// Maxima over the wavefront's 64 lanes of N unsigned values, as scalars (data-parallel-primitive steps within rows of
// 16 lanes, then across rows; the values' chains are interleaved).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
}
template <int N>
__device__ __forceinline__ void wave_umax(uint32_t (&v)[N])
{
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = max(v[k], dpp_or_zero<0x111>(v[k]));  // row_shr 1, 2, 4, 8
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = max(v[k], dpp_or_zero<0x112>(v[k]));
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = max(v[k], dpp_or_zero<0x114>(v[k]));
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = max(v[k], dpp_or_zero<0x118>(v[k]));
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = max(v[k], dpp_or_zero<0x142>(v[k]));  // row_bcast 15, 31
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = max(v[k], dpp_or_zero<0x143>(v[k]));
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = (uint32_t)__builtin_amdgcn_readlane((int)v[k], 63);
}

// A wavefront's LDS: the texel results of two tile contexts (the tile whose rays are handed out and the one
// before it, whose last rays may still be in flight; context c holds entries c * kTileTexels + slot), each
// lane's best hit key (queued loop) and the triangle-test queue, whose words hold the direction-bin counters
// while a tile's rays are sorted (the queue is empty then).
template <bool ENTRIES>
struct WaveTile {
    // per context: the entry points of its rays (child code, bits of the least distance to it), nearest first
    v2i entry[ENTRIES ? 2 * (kEntryEnd + 1) : 1];
    int32_t tex[2 * kTileTexels];
    unsigned long long key[2 * kTileTexels];  // min over rays of (distance bits << 32 | ray << 26 | triangle)
    uint32_t cnt[2 * kTileTexels];            // front | back << 16 for this frame
    unsigned long long best[kWave];  // each lane's ray: min of (t bits << 32 | triangle id << 1 | front)
    union {
        uint32_t q[kQueueCap];       // queued triangle tests: leaf-order index << 6 | lane of the ray
        uint32_t bin[kBins];         // bin counts, then bin cursors
    };
};

template <bool ENTRIES>
using lds_tile = __attribute__((address_space(3))) WaveTile<ENTRIES>;
typedef __attribute__((address_space(3))) v2i lds_v2i;
typedef __attribute__((address_space(4))) const TraceScene *scene_ptr;
static_assert(offsetof(TraceArgs, one) == 0, "a single scene's record is read at the start of the kernel arguments");

__device__ __forceinline__ uint64_t uniform64(uint64_t x)
{
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32 |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
}

// the next entry point of a ray (child code); kDone when none is left, or when the next one, and so every later one,
// lies beyond the ray's best distance
struct EntryCursor {
    uint32_t m0, m1;     // entry points not yet visited: the current word, the next one
    const lds_v2i *tab;  // the current word's table
};
__device__ __forceinline__ int entry_pop(EntryCursor &E, float tbest)
{
    if (E.m0 == 0u) {
        E.m0 = E.m1;
        E.tab += 32;
    }
    const v2i e = E.tab[__builtin_ctz(E.m0)];
    E.m0 &= E.m0 - 1u;
    return tbest < __int_as_float(e.y) ? kDone : e.x;
}

// Sets up a tile of rays in a wavefront's context c: draws the directions, sorts the rays by direction bin into
// records, and (ENTRIES) chooses the tile's entry points and which of them each ray meets.
//
// Entry points: starting from the root, the nodes most likely to be met by rays from the tile's block are replaced by
// their children (lane k holds entry point k), so every ray starts at the subtrees it meets, nearest first, instead of
// descending through the levels above them: half to two thirds of its node visits, each a fetch of scattered records
// and a step at partial width, become box tests at full width whose boxes come by the scalar cache.  Which rays meet an
// entry point is decided 64 sorted records at a time: lane k first tests entry point k against the bounds of the 64
// directions, and only those it may concern are tested ray by ray.  A box's slab test holds whenever that of a box
// inside it does, so the leaves a ray reaches are those it reaches from the root.
//
// Not inlined: its registers (41) are then not the traversal loop's (80: six wavefronts per SIMD), and the loop's state
// is saved once per tile.  Inlined, both spilled (a batch's loop reloaded 24 registers each round, 24.1 against 17.8 ms
// per step on 12 scenes).  Arguments arrive in vector registers and are made scalar here.  Its cost is bound by vector
// instructions: about 1,400 per 64 rays, half of them the generator's.
template <bool ENTRIES>
__device__ __noinline__ void tile_setup(scene_ptr P_, lds_tile<ENTRIES> *T_, gv4f *dirs_, int base_, int nt_, int c_,
                                        uint64_t seed_, uint32_t frame_, int bin_directions_)
{
    const scene_ptr P = (scene_ptr)uniform64((uint64_t)P_);
    lds_tile<ENTRIES> *T =
        (lds_tile<ENTRIES> *)(uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)T_);
    gv4f *dirs = (gv4f *)uniform64((uint64_t)dirs_);
    gv4f *recs = dirs + kTileRays;
    const int base = __builtin_amdgcn_readfirstlane(base_), nt = __builtin_amdgcn_readfirstlane(nt_);
    const int c = __builtin_amdgcn_readfirstlane(c_), bin_directions = __builtin_amdgcn_readfirstlane(bin_directions_);
    const uint64_t seed = uniform64(seed_);
    const uint32_t frame = (uint32_t)__builtin_amdgcn_readfirstlane((int)frame_);
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    // q / R as a multiply-high, as in the tracer
    const int R = P->rays, nrays = nt * R, lognf = P->lognf, qm = P->nf - 1;
    const uint32_t rdiv = R > 1 ? (uint32_t)(((1ull << 32) + (uint64_t)R - 1) / (uint64_t)R) : 0u;
    const float lox = P->lox, loy = P->loy, loz = P->loz, hf = P->hf;
    const BvhNode *nodes = P->bvh.nodes;
    const uint64_t ntex_grid = (uint64_t)1 << (3 * lognf);
    const int c0 = c * kTileTexels;
    int jt = -1;
    if (lane < nt) {
        jt = ((gint *)(uintptr_t)P->queue)[base + lane];
        if (jt < 0 || (uint64_t)jt >= ntex_grid) jt = -1;
        T->tex[c0 + lane] = jt;
        T->key[c0 + lane] = ~0ull;
        T->cnt[c0 + lane] = 0u;
    }
    T->bin[lane] = 0u;  // the queue is empty between traversal rounds
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // ---- bin the tile's rays by direction (the bin rides in the direction record's w)
    const uint32_t scene_id = P->scene_id;
#pragma unroll 1
    for (int q = lane; q < nrays; q += kWave) {
        const int qs = R > 1 ? (int)__umulhi((uint32_t)q, rdiv) : q, qr = q - qs * R;
        const int j = T->tex[c0 + qs];
        int b = 0;
        if (j >= 0) {
            // drawn once at full width; the lane that later takes the ray reads it back
            const float3 d = sphere_dir(seed, (uint32_t)j, frame, (uint32_t)qr, scene_id);
            if (bin_directions) b = direction_bin(d);
            dirs[q] = v4f{d.x, d.y, d.z, __int_as_float(b)};
        }
        __hip_atomic_fetch_add(&T->bin[b], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    {  // exclusive scan of the 64 bin counts, one per lane
        const uint32_t cb = T->bin[lane];
        uint32_t x = cb;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t y = __shfl_up(x, off);
            if (lane >= off) x += y;
        }
        T->bin[lane] = x - cb;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // ---- the records in bin order (each lane re-reads the directions it stored)
#pragma unroll 1
    for (int q = lane; q < nrays; q += kWave) {
        const int qs = R > 1 ? (int)__umulhi((uint32_t)q, rdiv) : q;
        v4f d = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        if (T->tex[c0 + qs] >= 0) d = dirs[q];
        const uint32_t pos = __hip_atomic_fetch_add(&T->bin[__float_as_int(d.w)], 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_WORKGROUP);
        d.w = __int_as_float(q);
        recs[pos] = d;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // also orders the stored records
    __builtin_amdgcn_wave_barrier();
    if constexpr (ENTRIES) {
        gv2u *masks = (gv2u *)dirs;
        lds_v2i *entry = T->entry + c * (kEntryEnd + 1);
        if (lane == 0) entry[kEntryEnd] = v2i{kDone, 0};
        if (P->nt == 0) {  // nothing to meet
            for (int i = lane; i < nrays; i += kWave) masks[i] = v2u{0u, 0u};
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
            return;
        }
        // ---- the tile's entry points
        uint32_t bb[6] = {0u, 0u, 0u, 0u, 0u, 0u};
        if (jt >= 0) {
            const uint32_t x = (uint32_t)(jt & qm), y = (uint32_t)((jt >> lognf) & qm);
            const uint32_t z = (uint32_t)(jt >> (2 * lognf));
            bb[0] = 2047u - x;
            bb[1] = x;
            bb[2] = 2047u - y;
            bb[3] = y;
            bb[4] = 2047u - z;
            bb[5] = z;
        }
        wave_umax<6>(bb);
        const float bx0 = texel_coord(lox, (int)(2047u - bb[0]), hf), bx1 = texel_coord(lox, (int)bb[1], hf);
        const float by0 = texel_coord(loy, (int)(2047u - bb[2]), hf), by1 = texel_coord(loy, (int)bb[3], hf);
        const float bz0 = texel_coord(loz, (int)(2047u - bb[4]), hf), bz1 = texel_coord(loz, (int)bb[5], hf);
        // rounding of the block's differences with box planes (box padding covers it unless the grid lies far outside)
        const float slack = 0x1p-21f * (fabsf(bx0) + fabsf(bx1) + fabsf(by0) + fabsf(by1) + fabsf(bz0) + fabsf(bz1));
        const float ex = bx1 - bx0 + hf, ey = by1 - by0 + hf, ez = bz1 - bz0 + hf;
        const float s2 = 0.25f * (ex * ex + ey * ey + ez * ez);
        // lane k holds entry point k: child code, its box's place (node << 1 | slot), priority, squared distance
        int nentry = 1, ecode = lane < nentry ? 0 : kDone, eref = 0;
        float eprio = 1e30f, ed2 = 0.0f;
        const int cap = min(kEntries, 14 + (nrays >> 4));
        while (true) {
            const int room = cap - nentry;
            uint32_t top[1] = {ecode >= 0 ? __float_as_uint(eprio) : 0u};
            wave_umax<1>(top);
            float tau = kOpenTogether * __uint_as_float(top[0]);
            if (!(__uint_as_float(top[0]) > kOpen) || room <= 0) break;
            uint64_t want = __builtin_amdgcn_ballot_w64(ecode >= 0 && eprio > fmaxf(tau, kOpen));
            while (__popcll(want) > room) {
                tau *= 1.25f;
                want = __builtin_amdgcn_ballot_w64(ecode >= 0 && eprio > fmaxf(tau, kOpen));
            }
            if (want == 0) break;
            const bool op = (want >> lane) & 1;
            gv4f *nd = (gv4f *)((uintptr_t)nodes + (uintptr_t)(uint32_t)(op ? ecode : 0) * 64u);
            const v4f a = nd[0], b = nd[1], z = nd[2], m = nd[3];
            const auto eval = [&](float lx, float hx, float ly, float hy, float lz, float hz, float &prio, float &d2) {
                const float dx = fmaxf(fmaxf(lx - bx1, bx0 - hx), 0.0f);
                const float dy = fmaxf(fmaxf(ly - by1, by0 - hy), 0.0f);
                const float dz = fmaxf(fmaxf(lz - bz1, bz0 - hz), 0.0f);
                const float wx = hx - lx, wy = hy - ly, wz = hz - lz;
                d2 = dx * dx + dy * dy + dz * dz;
                prio = (wx * wy + wy * wz + wz * wx) * __builtin_amdgcn_rcpf(d2 + s2);
            };
            float p0, q0, p1, q1;
            eval(a.x, a.y, a.z, a.w, z.x, z.y, p0, q0);
            eval(b.x, b.y, b.z, b.w, z.z, z.w, p1, q1);
            const int m0 = __float_as_int(m.x), m1 = __float_as_int(m.y), parent = ecode;
            const bool two = op && !(m1 < 0 && leaf_count(m1) == 0);  // (a one-leaf scene has an empty second leaf)
            const uint64_t twos = __builtin_amdgcn_ballot_w64(two);
            if (two)
                T->q[__builtin_amdgcn_mbcnt_hi((uint32_t)(twos >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)twos, 0u))] =
                    (uint32_t)lane;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int added = (int)__popcll(twos);
            const bool isnew = lane >= nentry && lane < nentry + added;
            const int src = isnew ? (int)T->q[lane - nentry] << 2 : 0;
            const int n_code = __builtin_amdgcn_ds_bpermute(src, m1);
            const int n_parent = __builtin_amdgcn_ds_bpermute(src, parent);
            const float n_prio = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(p1)));
            const float n_d2 = __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(q1)));
            if (op) {
                ecode = m0;
                eref = parent << 1;
                eprio = p0;
                ed2 = q0;
            }
            if (isnew) {
                ecode = n_code;
                eref = n_parent << 1 | 1;
                eprio = n_prio;
                ed2 = n_d2;
            }
            nentry += added;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        // nearest first; of those that the block touches, the smallest first
        float eord = ed2 > 0.0f ? ed2 : -__builtin_amdgcn_rcpf(eprio);
        if (!(eord == eord)) eord = 0.0f;  // (the ranks have to be distinct)
        int rank = 0;
        for (int k = 0; k < nentry; ++k) {
            const float ok = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(eord), k));
            rank += ok < eord || (ok == eord && k < lane);
        }
        if (lane < nentry) {
            // (past the largest float the order is not known: such an entry point ends no ray)
            const float least = ed2 < __builtin_inff() ? 0.9999f * __builtin_amdgcn_sqrtf(ed2) - slack : 0.0f;
            entry[rank] = v2i{ecode, __float_as_int(least)};
            T->q[rank] = (uint32_t)eref;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        eref = lane < nentry ? (int)T->q[lane] : 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // ---- which entry points each ray meets, 64 records (similar directions) at a time
        gv4f *en = (gv4f *)((uintptr_t)nodes + (uintptr_t)(uint32_t)(eref >> 1) * 64u);
        const v4f exy = en[eref & 1], ezz = en[2];
        const float elz = eref & 1 ? ezz.z : ezz.x, ehz = eref & 1 ? ezz.w : ezz.y;
        const float Lx = exy.x - bx1 - slack, Hx = exy.y - bx0 + slack, Ly = exy.z - by1 - slack,
                    Hy = exy.w - by0 + slack, Lz = elz - bz1 - slack, Hz = ehz - bz0 + slack;
    #pragma unroll 1
        for (int i0 = 0; i0 < nrays; i0 += kWave) {
            const int i = i0 + lane;
            const v4f d = recs[min(i, nrays - 1)];
            const int q = __float_as_int(d.w), qs = R > 1 ? (int)__umulhi((uint32_t)q, rdiv) : q;
            const int j = T->tex[c0 + qs];
            RaySetup Q;
            ray_setup(texel_coord(lox, j & qm, hf), texel_coord(loy, (j >> lognf) & qm, hf),
                      texel_coord(loz, j >> (2 * lognf), hf), d.x, d.y, d.z, Q);
            // lane k: whether a ray from the tile's block, its direction in these 64 rays' bounds, can meet entry point k
            uint32_t db[6] = {__float_as_uint(2.0f - d.x), __float_as_uint(2.0f + d.x), __float_as_uint(2.0f - d.y),
                              __float_as_uint(2.0f + d.y), __float_as_uint(2.0f - d.z), __float_as_uint(2.0f + d.z)};
            wave_umax<6>(db);
            float t0 = 0.0f, t1 = __builtin_inff();
            const auto axis = [&](uint32_t lo, uint32_t hi, float L, float H) {
                const float d0 = 1.999999f - __uint_as_float(lo), d1 = __uint_as_float(hi) - 1.999999f;
                const float i0 = __builtin_amdgcn_rcpf(d0), i1 = __builtin_amdgcn_rcpf(d1);
                if (L > 0.0f) t0 = fmaxf(t0, d1 > 0.0f ? L * i1 : __builtin_inff());
                if (H < 0.0f) t0 = fmaxf(t0, d0 < 0.0f ? H * i0 : __builtin_inff());
                if (d0 > 0.0f) t1 = fminf(t1, H * i0);
                if (d1 < 0.0f) t1 = fminf(t1, L * i1);
            };
            axis(db[0], db[1], Lx, Hx);
            axis(db[2], db[3], Ly, Hy);
            axis(db[4], db[5], Lz, Hz);
            uint64_t cand = __builtin_amdgcn_ballot_w64(lane < nentry && !(t0 * 0.9999f > t1 * 1.0001f));
            v2u mask = v2u{0u, 0u};
            const auto meet = [&](int k) {
                const int ref = __builtin_amdgcn_readlane(eref, k);
                const sfloat *xy = node_sptr(nodes, ref >> 1) + 4 * (ref & 1);
                const sfloat *zz = node_sptr(nodes, ref >> 1) + 8 + 2 * (ref & 1);
                float te;
                return box_hit(Q, xy[0], xy[1], xy[2], xy[3], zz[0], zz[1], __builtin_inff(), te);
            };
            uint32_t c0w = (uint32_t)cand, c1w = (uint32_t)(cand >> 32);
            while (c0w) {
                const int k = __builtin_ctz(c0w);
                c0w &= c0w - 1u;
                if (meet(k)) mask.x |= 1u << k;
            }
            while (c1w) {
                const int k = __builtin_ctz(c1w);
                c1w &= c1w - 1u;
                if (meet(32 + k)) mask.y |= 1u << k;
            }
            if (i < nrays) masks[i] = j >= 0 ? mask : v2u{0u, 0u};
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
    }
}

// Tiles of a scene: ceil(min(count, cap) / tile texels).
__device__ __forceinline__ int scene_tiles(const TraceScene &P, int cap)
{
    const int total = min(*P.count, P.queue_cap);
    const int tt = tile_texels_for(P.rays, cap);
    return total > 0 ? (total + tt - 1) / tt : 0;
}

// Global tile prefix of a batch: tile_offset[s] = sum of tiles of scenes < s.
__global__ void trace_tile_prefix(const TraceScene *scenes, int n, int cap, int32_t *tile_offset)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    int acc = 0;
    for (int s = 0; s < n; ++s) {
        tile_offset[s] = acc;
        acc += scene_tiles(scenes[s], cap);
    }
    tile_offset[n] = acc;
}

// Persistent tracer.  Each wavefront repeatedly takes a tile of up to 64
// consecutive queue texels of one scene (Morton order: a compact block of the
// fine grid), draws all their rays' directions, sorts the rays by direction
// bin, and traces them in that order, so the lanes of a wavefront follow rays
// that start close together and point the same way.  Results are folded per
// texel with LDS atomics (a 64-bit min keeps the smallest distance, ties to
// the lowest ray index, together with its triangle; an add counts front and
// back hits), which makes them independent of the order rays complete in.  A
// wavefront holds two tile contexts: once its tile has handed out its last
// ray, it sorts the next tile's rays into the other context and refills its
// lanes from there while the first tile's last rays are still traced (a
// tile's Eq. (1) epilogue runs once its last ray is done), so lanes do not
// wait for the slowest ray of each tile.  A next tile of another scene in a
// batch starts only once every lane is done (the traversal takes the scene's
// hierarchy as a wave-uniform value).
// Loop shapes (LOOP): 0 = phases per iteration
// (after Aila and Laine's "while-while" loop with postponed leaves: every lane
// walks internal nodes until it holds a leaf, then all held leaves are
// tested); 1 = one unit of work per lane per iteration (a triangle of the
// current leaf, else a node, else opening a popped leaf), which keeps more
// lanes busy on wave64; 2 = as 1, but each lane only requests its stack
// push/pop and one shared copy of the stack code runs after the work; 3 =
// as 2, but every lane fetches its node or its triangle's map into the same
// registers with one shared load sequence, so an iteration waits for memory
// once instead of once per kind of work; 4 = queued triangle tests (below),
// rays starting at their tile's entry points; 5 = the same with rays starting
// at the root (single scenes of few rays, in place of 4: see kFewRays).
// BATCHED launches serve many scenes: a global tile
// index is mapped to its scene through the tile prefix.  Instrumented runs
// (STATS) also count into 64-bit counters at workspace offsets 8, 16, ...:
// node visits, triangle tests, rays, traversal-loop iterations x 64, refill
// rounds x 64, lane-iterations with work (LOOP 1 and 2), tiles x 64, node
// visits that entered neither child box (LOOP 3), tiles started while lanes
// were still busy x 64, traversal rounds that waited for every lane before a
// next tile x 64.
template <int STACK, int REFILL, int LOOP, bool STATS, bool BATCHED, bool INST = false, bool WIDE = false>
__global__ void __launch_bounds__(kTraceWaves * kWave) __attribute__((amdgpu_waves_per_eu(6, 8)))
trace_persistent(TraceArgs A)
{
    uint32_t st_nodes = 0, st_tris = 0, st_rays = 0, st_iters = 0, st_refills = 0, st_busy = 0, st_tiles = 0;
    uint32_t st_empty = 0, st_early = 0, st_drains = 0;
    constexpr bool QUEUED = LOOP >= 4, ENTRIES = LOOP == 4;
    constexpr int SL = ENTRIES ? STACK - kEntryStack : STACK;  // stack entries per lane in LDS
    __shared__ int stack_mem[kTraceWaves * SL * kWave];
    __shared__ WaveTile<ENTRIES> tiles[kTraceWaves];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds_int *stk = (lds_int *)(stack_mem + wave * SL * kWave + lane);
    WaveTile<ENTRIES> &T = tiles[wave];
    int32_t *spill = A.spill + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // the wavefront's two direction buffers: by ray id (slot * R + ray), and the same rays in bin order as
    // (direction, ray id) records
    float4 *dirs = A.dirs + ((int64_t)blockIdx.x * kTraceWaves + wave) * (2 * kTileRays);
    float4 *recs = dirs + kTileRays;
    gv2u *masks = (gv2u *)(uintptr_t)dirs;  // the records' entry points (the drawn directions are read by then)
    const int stride = A.spill_stride;
    const uint32_t frame = A.frame_ptr ? *A.frame_ptr : A.frame;
    if (frame >= kMaxFrame) {
        // a device frame counter past the argmin record's range: trace nothing (the state keeps the
        // previous frame's values) and report it
        if (blockIdx.x == 0 && threadIdx.x == 0) raise_error(RTSDF_ERR_FRAME);
        return;
    }
    const int one_total = BATCHED ? 0 : max(0, min(*A.one.count, A.one.queue_cap));
    const int one_tt = BATCHED ? 1 : tile_texels_auto(A.one.rays, A.tile_cap, one_total, (int)gridDim.x * kTraceWaves);
    const int single_tiles = BATCHED ? 0 : (one_total + one_tt - 1) / one_tt;
    const int all_tiles = BATCHED ? A.tile_offset[A.nscenes] : single_tiles;
    const auto scene_of = [&](int g) {  // last scene whose first tile is <= g
        int lo = 0, hi = A.nscenes - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (A.tile_offset[mid] <= g) lo = mid;
            else hi = mid - 1;
        }
        return __builtin_amdgcn_readfirstlane(lo);
    };

    // A scene's record for one round of the loop below, read anew by scalar loads: kept over the traversal, its fields
    // would be spilled to vector registers' lanes, an instruction for each word on every way.
    const auto record = [&](int sn) {
        scene_ptr p = BATCHED ? (scene_ptr)(uintptr_t)uniform64((uint64_t)(uintptr_t)(A.scenes + sn))
                              : (scene_ptr)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return p;
    };

    // wave-uniform context state: -1 free, else rays not yet finished | texels << 16; and the scene (batches).  Two of
    // them in two-level scenes too, where a ray keeps its world direction in LDS: a room of 120 objects with rigid parts,
    // 256^3, 5 rays: 8,980 -> 8,300 us (lanes with work 0.69 -> 0.79 of lane-iterations).  There a launch of few tiles
    // uses one: asking for a next tile with rays in flight, when there is mostly none, and handing tiles of one
    // wavefront of rays out in pieces cost more than lanes that wait (traces of rigid parts at 128^3, 1 ray, 0.7 tiles
    // per wavefront: 176 us with two, 161 with one; at 64^3 in tiles of 16 texels 174 and 145; 2 rays, 0.7 tiles: 232
    // and 222; with 1 ray and 2.25 or 3.5 tiles per wavefront of a room's parts two are faster, 386 against 389 and 630
    // against 656, at 2.7 of the lone parts one, 394 against 377).
    // (kept as the sign of the number of tiles: one more scalar over the traversal costs 0.4 %)
    const int ntiles = INST && all_tiles <= (int)gridDim.x * kTraceWaves * (one_tt * A.one.rays <= kWave ? 2 : 1)
                           ? -all_tiles
                           : all_tiles;
    int cstate[2] = {-1, -1}, cscene[2] = {0, 0};
    int cur = 0, pool = 0, nrays = 0;  // the context rays are handed out from
    uint32_t rdiv = 0;                 // its q / R multiplier (below)
    int gnext = -2;                    // the next tile: -2 not taken yet, -1 none left
    // lane state
    bool busy = false;
    int rid = 0;  // the lane's ray: (context * kTileTexels + texel slot) << 6 | ray index
    RaySetup Rs;
    float tbest = __builtin_inff();
    int ibest = -1, node = kDone, leaf = kDone, sp = 0;
    int tri_cur = 0, tri_end = 0;
    // queued loop: the pending triangles, the stack's next entry and the end of the wavefront's part of it in LDS
    uint32_t pend = 0;
    lds_int *top = stk, *const stk_end = (lds_int *)(stack_mem + (wave + 1) * SL * kWave);
    bool front = false;
    EntryCursor E{0u, 0u, nullptr};  // queued loop: the entry points not yet visited (bit kEntryEnd: none left)

    while (true) {
        // ---- start the next tile once the current one has handed out its last ray
        const bool any_busy = __builtin_amdgcn_ballot_w64(busy) != 0;
        if (pool >= nrays && cstate[cur ^ 1] < 0 && gnext != -1) {
            if (gnext == -2) {
                int g = 0;
                if (lane == 0) g = atomicAdd(A.cursor, 1);
                g = __builtin_amdgcn_readlane(g, 0);  // a wave-uniform (scalar) value
                gnext = g < (INST ? abs(ntiles) : ntiles) ? g : -1;
            }
            const int sn = gnext >= 0 && BATCHED ? scene_of(gnext) : 0;
            if (gnext >= 0 && (!any_busy || ((!INST || ntiles > 0) && (!BATCHED || sn == cscene[cur])))) {
                const int c = cur ^ 1, g = gnext;
                gnext = -2;
                const TraceScene &P = BATCHED ? A.scenes[sn] : A.one;
                if (STATS) {
                    ++st_tiles;
                    st_early += any_busy;
                }
                const int R = P.rays;
                // q / R as a multiply-high: exact for q < kTileRays and R <= 64 (the error of the rounded-up
                // reciprocal, q / 2^32, stays below the distance 1/R of q / R from the next integer)
                rdiv = R > 1 ? (uint32_t)(((1ull << 32) + (uint64_t)R - 1) / (uint64_t)R) : 0u;
                const int tile_texels = BATCHED ? tile_texels_for(R, A.tile_cap) : one_tt;
                const int total = min(*P.count, P.queue_cap);
                const int base = (g - (BATCHED ? A.tile_offset[sn] : 0)) * tile_texels;
                const int nt = min(tile_texels, total - base);
                const scene_ptr sp4 = BATCHED ? (scene_ptr)(uintptr_t)(A.scenes + sn)
                                              : (scene_ptr)__builtin_amdgcn_kernarg_segment_ptr();
                nrays = nt * R;
                tile_setup<ENTRIES>(sp4, (lds_tile<ENTRIES> *)&T, (gv4f *)(uintptr_t)dirs, base, nt, c, A.seed, frame,
                                      A.bin_directions);
                cstate[c] = nrays | nt << 16;
                cscene[c] = sn;
                cur = c;
                pool = 0;
            }
        }

        // ---- refill idle lanes from the current tile, in bin order
        const scene_ptr Pp = record(cscene[cur]);
        const auto &P = *Pp;
        const int R = P.rays;
        const int nfm = P.nf - 1;
        const BvhView S{P.bvh.nodes, P.bvh.tris, P.bvh.tmap};
        const int scene_nt = P.nt;
        {
            const uint64_t need = __builtin_amdgcn_ballot_w64(!busy);
            if (need != 0 && pool < nrays) {
                if (STATS) ++st_refills;
                const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(need >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)need, 0u));
                const int take = min(__popcll(need), nrays - pool);
                if (!busy && rank < take) {
                    const float4 d = recs[pool + rank];
                    const int q = __float_as_int(d.w);
                    const int qs = R > 1 ? (int)__umulhi((uint32_t)q, rdiv) : q;
                    rid = (cur * kTileTexels + qs) << 6 | (q - qs * R);
                    const int j = T.tex[cur * kTileTexels + qs];
                    if (j >= 0) {
                        const float ox = texel_coord(P.lox, j & nfm, P.hf);
                        const float oy = texel_coord(P.loy, (j >> P.lognf) & nfm, P.hf);
                        const float oz = texel_coord(P.loz, j >> (2 * P.lognf), P.hf);
                        ray_setup(ox, oy, oz, d.x, d.y, d.z, Rs);
                        node = scene_nt > 0 ? 0 : kDone;
                    } else {
                        node = kDone;
                    }
                    tbest = __builtin_inff();
                    if (ENTRIES) {
                        const v2u m = masks[pool + rank];
                        E.m0 = m.x;
                        E.m1 = m.y | 1u << (kEntryEnd - 32);
                        E.tab = ((lds_tile<ENTRIES> *)&T)->entry + cur * (kEntryEnd + 1);
                        node = entry_pop(E, tbest);
                    }
                    ibest = -1;
                    front = false;
                    if (QUEUED) T.best[lane] = kBestInit;
                    if (INST) {  // the world direction, for the way back from a part (in words of the queued loop's:
                        // the tile's own direction buffer is the next tile's by then)
                        T.best[lane] = (unsigned long long)__float_as_uint(d.y) << 32 | __float_as_uint(d.x);
                        T.q[kBins + lane] = __float_as_uint(d.z);
                    }
                    leaf = kDone;
                    tri_cur = tri_end = 0;
                    sp = 0;
                    top = stk;
                    busy = true;
                }
                pool += take;
            }
        }
        if (__builtin_amdgcn_ballot_w64(busy) == 0) {
            // every context is finished (a context's epilogue runs when its last ray is done)
            if (pool >= nrays && gnext == -1) break;
            continue;
        }
        {
            // refill rounds go on while this tile has rays or the next one can start before every lane is
            // done; otherwise every lane finishes first
            const bool early = (!INST || ntiles > 0) && cstate[cur ^ 1] < 0 &&
                               (gnext == -2 || (gnext >= 0 && (!BATCHED || scene_of(gnext) == cscene[cur])));
            const int refill_at = __builtin_amdgcn_readfirstlane(pool < nrays || early ? REFILL : kWave);
            if (STATS) st_drains += refill_at == kWave && gnext != -1;  // every lane finishes before the next tile
            if (LOOP == 0) {
                while (true) {
                    if (busy && leaf == kDone && node < 0 && node != kDone) {
                        leaf = node;
                        node = stack_pop<SL>(stride, sp, stk, spill);
                    }
                    // phase 1: internal nodes until every busy lane holds a leaf or is done
                    while (__ballot(busy && node >= 0 && leaf == kDone)) {
                        if (busy && node >= 0) {
                            inner_step<SL, STATS>(S, stride, Rs, node, sp, stk, spill, tbest, st_nodes);
                            if (node < 0 && node != kDone && leaf == kDone) {
                                leaf = node;
                                node = stack_pop<SL>(stride, sp, stk, spill);
                            }
                        }
                    }
                    // phase 2: triangles of the held leaves
                    if (busy && leaf != kDone) {
                        const int first = leaf_first(leaf), cnt = leaf_count(leaf);
                        if (STATS) st_tris += (uint32_t)cnt;
                        for (int i = first; i < first + cnt; ++i) {
                            tri_test(Rs, S.tmap, S.tris, i, tbest, ibest, front);
                        }
                        leaf = kDone;
                    }
                    const uint64_t done = __ballot(!busy || (node == kDone && leaf == kDone));
                    if (__popcll(done) >= refill_at) break;
                }
            } else if (LOOP == 3) {
                while (true) {
                    if (STATS) {
                        ++st_iters;
                        st_busy += busy && (node != kDone || tri_cur < tri_end);
                    }
                    // one fetch per lane and iteration: the triangle's map or the node, into the same
                    // registers, so the wavefront waits for memory once whichever work its lanes do
                    const bool do_tri = busy && tri_cur < tri_end;
                    const bool do_node = busy && !do_tri && node >= 0;
                    // (lanes with neither load the root node, which every scene allocates, and ignore it)
                    const char *base =
                        do_tri ? reinterpret_cast<const char *>(S.tmap) + rec48(tri_cur)
                               : WIDE ? reinterpret_cast<const char *>(P.nodes4) + (uint32_t)(do_node ? node : 0) * 128u
                                      : reinterpret_cast<const char *>(S.nodes) + (uint32_t)(do_node ? node : 0) * 64u;
                    const float4 *q = reinterpret_cast<const float4 *>(base);
                    const float4 w0 = q[0], w1 = q[1], w2 = q[2];
                    const int2 w3 = *reinterpret_cast<const int2 *>(q + 3);  // the map array has 16 B of padding
                    // a wide node's second record (other lanes re-read their first 64 bytes)
                    float4 w4, w5, w6;
                    int2 w7;
                    if (WIDE) {
                        const float4 *q2 = do_node ? q + 4 : q;
                        w4 = q2[0];
                        w5 = q2[1];
                        w6 = q2[2];
                        w7 = *reinterpret_cast<const int2 *>(q2 + 3);
                    }
                    bool push = false, pop = false;
                    int push_val = 0;
                    bool p1 = false, p2 = false, p3 = false;
                    int v1 = 0, v2 = 0, v3 = 0;
                    if (do_tri) {
                        if (STATS) ++st_tris;
                        tri_test_rows(Rs, w0, w1, w2, S.tris, tri_cur, tbest, ibest, front);
                        ++tri_cur;
                    } else if (do_node) {
                        if (STATS) ++st_nodes;
                        if (INST && w3.y == kInstTag) {
                            // instance node of a two-level scene: its rows take the (world) ray into the
                            // part's object space; the return marker restores it
                            const float ox = w0.x * Rs.ox + w0.y * Rs.oy + w0.z * Rs.oz + w0.w;
                            const float oy = w1.x * Rs.ox + w1.y * Rs.oy + w1.z * Rs.oz + w1.w;
                            const float oz = w2.x * Rs.ox + w2.y * Rs.oy + w2.z * Rs.oz + w2.w;
                            const float dx = w0.x * Rs.dx + w0.y * Rs.dy + w0.z * Rs.dz;
                            const float dy = w1.x * Rs.dx + w1.y * Rs.dy + w1.z * Rs.dz;
                            const float dz = w2.x * Rs.dx + w2.y * Rs.dy + w2.z * Rs.dz;
                            ray_setup(ox, oy, oz, dx, dy, dz, Rs);
                            push = true;
                            push_val = kReturn;
                            node = w3.x;
                        } else if (WIDE) {
                            node4_step_regs(Rs, w0, w1, w2, w3, w4, w5, w6, w7, node, tbest, tri_cur, tri_end, p1, p2,
                                            p3, v1, v2, v3, pop);
                            if (STATS) st_empty += pop && tri_cur >= tri_end;  // no child box was entered
                        } else {
                            const int4 m = make_int4(w3.x, w3.y, 0, 0);
                            node_step_regs(Rs, w0, w1, w2, m, node, tbest, tri_cur, tri_end, push, push_val, pop);
                            if (STATS) st_empty += pop && tri_cur >= tri_end;  // neither child box was entered
                        }
                    } else if (INST && busy && node == kReturn) {
                        // the part is done (its last leaf's triangles too): the world ray again, as drawn
                        const int j = T.tex[rid >> 6];
                        const unsigned long long dxy = T.best[lane];
                        ray_setup(texel_coord(P.lox, j & nfm, P.hf), texel_coord(P.loy, (j >> P.lognf) & nfm, P.hf),
                                  texel_coord(P.loz, j >> (2 * P.lognf), P.hf), __uint_as_float((uint32_t)dxy),
                                  __uint_as_float((uint32_t)(dxy >> 32)), __uint_as_float(T.q[kBins + lane]), Rs);
                        pop = true;
                    } else if (busy && node != kDone) {
                        tri_cur = leaf_first(node);
                        tri_end = tri_cur + leaf_count(node);
                        pop = true;
                    }
                    if (WIDE) {  // farthest first, so the nearest is popped first
                        if (p3) stack_push<SL>(stride, sp, stk, spill, v3);
                        if (p2) stack_push<SL>(stride, sp, stk, spill, v2);
                        if (p1) stack_push<SL>(stride, sp, stk, spill, v1);
                    }
                    if (push) stack_push<SL>(stride, sp, stk, spill, push_val);
                    if (pop) node = stack_pop<SL>(stride, sp, stk, spill);
                    const uint64_t done = wave_done(busy, node, tri_cur, tri_end);
                    if (__popcll(done) >= refill_at) break;
                }
            } else if (QUEUED) {
                // Queued loop: a lane that reaches a leaf appends its triangles to the wavefront's queue
                // in LDS (two per iteration at most) and goes on with its traversal; once a wavefront's
                // worth of tests is queued, every lane takes one, whichever ray it belongs to, so the
                // triangle code runs at full width instead of in nearly every iteration for a few lanes.
                // The loop is bound by vector instructions and, nearly as much, by the data return of its loads: an
                // iteration is 90 instructions and 56 bytes a lane (106 and 64 before the pending word, the queue
                // without wrap-around, the stack by address and the shorter node step; with the scenes' records read
                // anew each round, 28 registers' worth of spilled scalars less per round).  Whole updates: a room of
                // 216k triangles, 128^3 / 256^3, 16 rays: 21.0 -> 20.35 ms; 12 scenes in one launch: 17.2 -> 16.5 ms.
                // Between flushes a lane culls boxes against its ray's best distance as of the last flush
                // (a larger bound only enters more boxes); the closest hit is the minimum of the
                // (t, triangle id, facing) keys of all tests, as in the other loops.
                int qn = 0;  // tests queued (wave-uniform)
                const auto flush = [&](int nf) {
                    const bool act = lane < nf;
                    const uint32_t e = act ? T.q[lane] : (uint32_t)lane;
                    if (qn > kWave) T.q[lane] = T.q[kWave + lane];  // the later ones move up
                    const int owner = (int)(e & 63u), addr = owner << 2;
                    // the owner's ray, from its registers (every lane takes part in the permutes)
                    const float ox = __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(Rs.ox)));
                    const float oy = __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(Rs.oy)));
                    const float oz = __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(Rs.oz)));
                    const float dx = __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(Rs.dx)));
                    const float dy = __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(Rs.dy)));
                    const float dz = __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(Rs.dz)));
                    const float tb = __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(tbest)));
                    if (act) {
                        if (STATS) ++st_tris;
                        const int i = (int)(e >> 6);
                        const float4 *mp = tri_ptr(S.tmap, i);
                        float t;
                        bool fr;
                        if (tri_hit_rows(ox, oy, oz, dx, dy, dz, mp[0], mp[1], mp[2], S.tris, i, tb, t, fr)) {
                            const unsigned long long key = ((unsigned long long)__float_as_uint(t) << 32) |
                                                           ((uint32_t)tri_id(S.tris, i) << 1) | (fr ? 1u : 0u);
                            atomicMin(&T.best[owner], key);
                        }
                    }
                    qn -= nf;
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    tbest = __uint_as_float((uint32_t)(T.best[lane] >> 32));
                };
                // (lanes without a ray hold kDone and no pending triangles)
                while (true) {
                    if (STATS) {
                        ++st_iters;
                        st_busy += node != kDone || pend >= kPendOne;
                    }
                    // ---- append up to two of the lane's pending triangles, as far as the queue has room
                    bool g1 = pend >= kPendOne, g2 = pend >= 2 * kPendOne;
                    const uint64_t b1 = __builtin_amdgcn_ballot_w64(g1), b2 = __builtin_amdgcn_ballot_w64(g2);
                    // the lane's position: the requests of the lanes below it
                    const int pos = (int)__builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(b2 >> 32),
                        __builtin_amdgcn_mbcnt_lo(
                            (uint32_t)b2, __builtin_amdgcn_mbcnt_hi((uint32_t)(b1 >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)b1, 0u))));
                    int total = (int)(__popcll(b1) + __popcll(b2));
                    if (qn + total > kQueueCap) {  // rare: grant a prefix of the lanes
                        const bool fit = pos + (g2 ? 2 : 1) <= kQueueCap - qn;
                        g1 = g1 && fit;
                        g2 = g2 && fit;
                        total = (int)(__popcll(__builtin_amdgcn_ballot_w64(g1)) +
                                      __popcll(__builtin_amdgcn_ballot_w64(g2)));
                    }
                    if (g1) {
                        uint32_t *q = T.q + qn + pos;
                        const uint32_t e = (pend << 6) | (uint32_t)lane;
                        q[0] = e;
                        pend -= kPendOne - 1u;
                        if (g2) {
                            q[1] = e + 64u;
                            pend -= kPendOne - 1u;
                        }
                    }
                    qn += total;
                    // ---- the lane's traversal step: a node, or opening a popped leaf
                    const bool idle = pend < kPendOne;
                    const bool do_node = idle && node >= 0;
                    const float4 *q = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(S.nodes) +
                                                                       (uint32_t)(do_node ? node : 0) * 64u);
                    const float4 w0 = q[0], w1 = q[1], w2 = q[2];
                    const v2i w3 = *reinterpret_cast<const v2i *>(q + 3);
                    bool push = false, pop = false;
                    int push_val = 0;
                    if (do_node) {
                        if (STATS) ++st_nodes;
                        node_step_queued(Rs, w0, w1, w2, make_int2(w3.x, w3.y), node, tbest, pend, push, push_val, pop);
                        if (STATS) st_empty += pop && pend < kPendOne;
                    } else if (idle && node != kDone) {
                        pend = leaf_pending(node);
                        pop = true;
                    }
                    if (push) stack_push_at(stride, top, stk_end, spill, push_val);
                    if (pop) {
                        // (formed anew in each iteration: a scalar register less to keep and to spill)
                        int room = SL - 1;
                        asm volatile("" : "+s"(room));
                        if (top >= stk_end - room * kWave) node = stack_pop_at(stride, top, stk_end, spill);
                        else node = ENTRIES ? entry_pop(E, tbest) : kDone;
                    }
                    // ---- a wavefront's worth of tests
                    if (qn >= kWave) flush(kWave);
                    const uint64_t done = __builtin_amdgcn_ballot_w64(node == kDone) &
                                          __builtin_amdgcn_ballot_w64(pend < kPendOne);
                    if (__popcll(done) >= refill_at) break;
                }
                // the rest of the queue (the finished rays' tests among them)
                while (qn > 0) flush(min(qn, kWave));
            } else if (LOOP == 2) {
                while (true) {
                    if (STATS) {
                        ++st_iters;
                        st_busy += busy && (node != kDone || tri_cur < tri_end);
                    }
                    bool push = false, pop = false;
                    int push_val = 0;
                    if (busy) {
                        if (tri_cur < tri_end) {
                            if (STATS) ++st_tris;
                            tri_test(Rs, S.tmap, S.tris, tri_cur, tbest, ibest, front);
                            ++tri_cur;
                        } else if (node >= 0) {
                            if (STATS) ++st_nodes;
                            node_step_flat(S, Rs, node, tbest, tri_cur, tri_end, push, push_val, pop);
                        } else if (node != kDone) {
                            tri_cur = leaf_first(node);
                            tri_end = tri_cur + leaf_count(node);
                            pop = true;
                        }
                    }
                    if (push) stack_push<SL>(stride, sp, stk, spill, push_val);
                    if (pop) node = stack_pop<SL>(stride, sp, stk, spill);
                    const uint64_t done = wave_done(busy, node, tri_cur, tri_end);
                    if (__popcll(done) >= refill_at) break;
                }
            } else {
                while (true) {
                    if (STATS) {
                        ++st_iters;
                        st_busy += busy && (node != kDone || tri_cur < tri_end);
                    }
                    if (busy) {
                        if (tri_cur < tri_end) {
                            if (STATS) ++st_tris;
                            tri_test(Rs, S.tmap, S.tris, tri_cur, tbest, ibest, front);
                            ++tri_cur;
                        } else if (node >= 0) {
                            node_step<SL, STATS>(S, stride, Rs, node, sp, stk, spill, tbest, tri_cur, tri_end,
                                                 st_nodes);
                        } else if (node != kDone) {
                            tri_cur = leaf_first(node);
                            tri_end = tri_cur + leaf_count(node);
                            node = stack_pop<SL>(stride, sp, stk, spill);
                        }
                    }
                    const uint64_t done = wave_done(busy, node, tri_cur, tri_end);
                    if (__popcll(done) >= refill_at) break;
                }
            }
            const bool fin = busy && node == kDone && (QUEUED ? pend < kPendOne : leaf == kDone && tri_cur >= tri_end);
            if (fin) {
                if (STATS) ++st_rays;
                int id = -1;
                if (QUEUED) {
                    const unsigned long long kb = T.best[lane];
                    if (kb != kBestInit) {
                        tbest = __uint_as_float((uint32_t)(kb >> 32));
                        id = (int)((uint32_t)kb >> 1);
                        front = (kb & 1u) != 0u;
                    }
                } else if (ibest >= 0) {
                    id = tri_id(S.tris, ibest);
                }
                if (id >= 0) {
                    const float dist = tbest * ray_len(Rs);
                    const unsigned long long key = ((unsigned long long)__float_as_uint(dist) << 32) |
                                                   ((unsigned long long)(rid & 63) << 26) | (unsigned long long)id;
                    atomicMin(&T.key[rid >> 6], key);
                    atomicAdd(&T.cnt[rid >> 6], front ? 1u : 0x10000u);
                }
                busy = false;
            }
            const uint64_t fin1 = __builtin_amdgcn_ballot_w64(fin && rid >= (kTileTexels << 6));
            cstate[0] -= (int)__popcll(__builtin_amdgcn_ballot_w64(fin) & ~fin1);
            cstate[1] -= (int)__popcll(fin1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        // ---- Eq. (1) on the unsigned state, then the sign vote, for each tile whose last ray is done
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (cstate[c] < 0 || (cstate[c] & 0xFFFF) > 0) continue;
            const int nt = cstate[c] >> 16, e = c * kTileTexels + lane;
            cstate[c] = -1;
            const scene_ptr Qp = record(cscene[c]);
            const auto &Q = *Qp;
            if (lane < nt && T.tex[e] >= 0) {
                const int j = T.tex[e];
                const unsigned long long key = T.key[e];
                const uint32_t fc = T.cnt[e];
                const float rmin = key == ~0ull ? __builtin_inff() : __uint_as_float((uint32_t)(key >> 32));
                const int argray = (int)((key >> 26) & 63u), argtri = (int)(key & ((1u << 26) - 1u));
                const int qm = Q.nf - 1;
                const int x = j & qm, y = (j >> Q.lognf) & qm, z = j >> (2 * Q.lognf);
                const float cs = Q.coarse_sdf[(x >> Q.logr) + Q.nc * ((y >> Q.logr) + Q.nc * (z >> Q.logr))];
                const float uprev = Q.u[j];
                const uint32_t h = Q.hits[j];
                const uint32_t F = min((h & 0xFFFFu) + (fc & 0xFFFFu), 0xFFFFu);
                const uint32_t B = min((h >> 16) + (fc >> 16), 0xFFFFu);
                float uu;
                if (Q.alpha == 1.0f) {
                    uu = uprev;
                } else {
                    // alpha = 0: no memory, the alpha u term is 0 even before the first hit (u = +inf)
                    uu = Q.alpha == 0.0f ? fmaxf(cs, 0.0f) : Q.alpha * uprev + (1.0f - Q.alpha) * fmaxf(cs, 0.0f);
                }
                if (rmin < uu) {
                    uu = rmin;
                    Q.arg_tri[j] = argtri;
                    Q.arg_ray[j] = (int32_t)((frame << 8) | (uint32_t)argray);
                } else if (Q.alpha != 1.0f) {
                    Q.arg_tri[j] = -1;
                    Q.arg_ray[j] = -1;
                }
                Q.u[j] = uu;
                Q.hits[j] = F | (B << 16);
                if (isinf(uu)) Q.fine[j] = cs;
                else if (Q.sign_policy == RTSDF_SIGN_SHELL) Q.fine[j] = uu - Q.shell;
                else Q.fine[j] = B > F ? -uu : uu;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (STATS) {
        unsigned long long *ctr = reinterpret_cast<unsigned long long *>(A.cursor + 2);
        atomicAdd(&ctr[0], (unsigned long long)st_nodes);
        atomicAdd(&ctr[1], (unsigned long long)st_tris);
        atomicAdd(&ctr[2], (unsigned long long)st_rays);
        atomicAdd(&ctr[3], (unsigned long long)st_iters);
        atomicAdd(&ctr[4], (unsigned long long)st_refills);
        atomicAdd(&ctr[5], (unsigned long long)st_busy);
        atomicAdd(&ctr[6], (unsigned long long)st_tiles);
        atomicAdd(&ctr[7], (unsigned long long)st_empty);
        atomicAdd(&ctr[8], (unsigned long long)st_early);
        atomicAdd(&ctr[9], (unsigned long long)st_drains);
    }
}

// Unselected texels: fine = coarse value, state reset (Eq. (1), case c > d).
__device__ __forceinline__ void fill_unselected_body(const uint8_t *__restrict__ mask,
                                                     const float *__restrict__ coarse_sdf, int nc, int logr, int lognf,
                                                     int64_t ntex, float *__restrict__ u, uint32_t *__restrict__ hits,
                                                     int32_t *__restrict__ arg_tri, int32_t *__restrict__ arg_ray,
                                                     float *__restrict__ fine, int64_t j)
{
    if (j >= ntex || mask[j]) return;
    const int nfm = (1 << lognf) - 1;
    const int x = (int)(j & nfm), y = (int)((j >> lognf) & nfm), z = (int)(j >> (2 * lognf));
    fine[j] = coarse_sdf[(x >> logr) + nc * ((y >> logr) + nc * (z >> logr))];
    if (u[j] != __builtin_inff() || hits[j] != 0u || arg_tri[j] != -1) {
        u[j] = __builtin_inff();
        hits[j] = 0u;
        arg_tri[j] = -1;
        arg_ray[j] = -1;
    }
}

__global__ void __launch_bounds__(256) trace_fill_unselected(const uint8_t *__restrict__ mask,
                                                             const float *__restrict__ coarse_sdf, int nc, int logr,
                                                             int lognf, int64_t ntex, float *__restrict__ u,
                                                             uint32_t *__restrict__ hits, int32_t *__restrict__ arg_tri,
                                                             int32_t *__restrict__ arg_ray, float *__restrict__ fine)
{
    fill_unselected_body(mask, coarse_sdf, nc, logr, lognf, ntex, u, hits, arg_tri, arg_ray, fine,
                         (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

__global__ void __launch_bounds__(256) accum_reset_kernel(int64_t n, float *u, uint32_t *hits, int32_t *at, int32_t *ar)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        u[i] = __builtin_inff();
        hits[i] = 0u;
        at[i] = -1;
        ar[i] = -1;
    }
}

// ---------------------------------------------------------- helpers ----

__global__ void directions_kernel(const int32_t *texel, const uint32_t *frame, const int32_t *ray, int n, uint64_t seed,
                                  uint32_t scene, float *out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float3 d = sphere_dir(seed, (uint32_t)texel[i], frame[i], (uint32_t)ray[i], scene);
    out[3 * i] = d.x;
    out[3 * i + 1] = d.y;
    out[3 * i + 2] = d.z;
}

// Closest hits, a ray per lane.  Bound by latency (dependent node loads) at the occupancy that the stacks leave: 32
// entries allow 16 wavefronts per compute unit, the 64 of a rebuilt hierarchy 8.  kHitsShort: the first of two launches,
// with 20 entries (32 wavefronts); a ray whose stack fills leaves kRayTodo as its distance, and the second launch, with
// the full stack, takes those rays only.  300,007 rays after a rebuild, with the rebuild, in three rooms of 200,000 to
// 226,000 triangles: the full stack alone 850 / 846 / 861 us, 12 entries 713 / 703 / 720 and 16 entries 610 / 636 / 640
// (more rays left over), 20 entries 554 / 578 / 577, 24 entries 555 / 578 / 577.
constexpr uint32_t kRayTodo = 0x7FA5A5A5u;  // a NaN that no hit distance is
constexpr int kShortHitStack = 20;

enum HitsPass { kHitsAll, kHitsShort, kHitsRest };  // (one launch of all rays has no test for those left over)

template <int SD, HitsPass PASS>
__global__ void __launch_bounds__(256) closest_hits_kernel(BvhView S, int nt, const float *__restrict__ o,
                                                           const float *__restrict__ d, int n, float *t_out,
                                                           int32_t *tri_out, int32_t *front_out)
{
    __shared__ int stack_mem[4 * SD * kWave];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int *stk = stack_mem + wave * SD * kWave + lane;
    if (i >= n || (PASS == kHitsRest && __float_as_uint(t_out[i]) != kRayTodo)) return;
    RaySetup R;
    ray_setup(o[3 * i], o[3 * i + 1], o[3 * i + 2], d[3 * i], d[3 * i + 1], d[3 * i + 2], R);
    float tbest = __builtin_inff();
    int ibest = -1, node = nt > 0 ? 0 : kDone, sp = 0;
    bool front = false;
    while (node != kDone) {
        trav_step(S, R, node, sp, stk, kWave, tbest, ibest, front);
        if (PASS == kHitsShort && sp >= SD) {
            t_out[i] = __uint_as_float(kRayTodo);
            return;
        }
    }
    t_out[i] = ibest >= 0 ? tbest : __builtin_inff();
    tri_out[i] = ibest >= 0 ? tri_id(S.tris, ibest) : -1;
    front_out[i] = ibest >= 0 && front;
}

// Gradient scatter: dL/dv_i += dL/df * sign * |w| * b_i * n / (n . w).
__global__ void __launch_bounds__(256) trace_backward_kernel(const float *__restrict__ v, const int32_t *__restrict__ f,
                                                             int nt, int lognf, float lox, float loy, float loz,
                                                             float hf, const int32_t *__restrict__ arg_tri,
                                                             const int32_t *__restrict__ arg_ray,
                                                             const float *__restrict__ fine,
                                                             const float *__restrict__ grad, uint64_t seed,
                                                             uint32_t scene, float *grad_v, int64_t ntex, bool vote)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= ntex) return;
    const int tri = arg_tri[j];
    const float g = grad[j];
    if (tri < 0 || tri >= nt || g == 0.0f) return;
    const uint32_t key = (uint32_t)arg_ray[j];
    const int nfm = (1 << lognf) - 1;
    const float ox = texel_coord(lox, (int)(j & nfm), hf), oy = texel_coord(loy, (int)((j >> lognf) & nfm), hf),
                oz = texel_coord(loz, (int)(j >> (2 * lognf)), hf);
    const float3 w = sphere_dir(seed, (uint32_t)j, key >> 8, key & 0xFFu, scene);
    const int i0 = f[3 * tri], i1 = f[3 * tri + 1], i2 = f[3 * tri + 2];
    const float3 p0 = make_float3(v[3 * i0], v[3 * i0 + 1], v[3 * i0 + 2]);
    const float3 p1 = make_float3(v[3 * i1], v[3 * i1 + 1], v[3 * i1 + 2]);
    const float3 p2 = make_float3(v[3 * i2], v[3 * i2 + 1], v[3 * i2 + 2]);
    const float3 e1 = make_float3(p1.x - p0.x, p1.y - p0.y, p1.z - p0.z);
    const float3 e2 = make_float3(p2.x - p0.x, p2.y - p0.y, p2.z - p0.z);
    // Moller-Trumbore barycentrics of the recorded hit
    const float3 pv = make_float3(w.y * e2.z - w.z * e2.y, w.z * e2.x - w.x * e2.z, w.x * e2.y - w.y * e2.x);
    const float det = e1.x * pv.x + e1.y * pv.y + e1.z * pv.z;
    if (det == 0.0f) return;
    const float inv = 1.0f / det;
    const float3 s = make_float3(ox - p0.x, oy - p0.y, oz - p0.z);
    const float bu = (s.x * pv.x + s.y * pv.y + s.z * pv.z) * inv;
    const float3 q = make_float3(s.y * e1.z - s.z * e1.y, s.z * e1.x - s.x * e1.z, s.x * e1.y - s.y * e1.x);
    const float bv = (w.x * q.x + w.y * q.y + w.z * q.z) * inv;
    const float3 nrm = make_float3(e1.y * e2.z - e1.z * e2.y, e1.z * e2.x - e1.x * e2.z, e1.x * e2.y - e1.y * e2.x);
    const float nw = nrm.x * w.x + nrm.y * w.y + nrm.z * w.z;
    if (nw == 0.0f) return;
    const float len = sqrtf(w.x * w.x + w.y * w.y + w.z * w.z);
    const float sgn = !vote || fine[j] >= 0.0f ? 1.0f : -1.0f;  // a shell value is the distance minus a constant
    const float scale = g * sgn * len / nw;
    const float b[3] = {1.0f - bu - bv, bu, bv};
    const int vid[3] = {i0, i1, i2};
    for (int k = 0; k < 3; ++k) {
        atomicAdd(&grad_v[3 * vid[k]], scale * b[k] * nrm.x);
        atomicAdd(&grad_v[3 * vid[k] + 1], scale * b[k] * nrm.y);
        atomicAdd(&grad_v[3 * vid[k] + 2], scale * b[k] * nrm.z);
    }
}

// ------------------------------------------------------------- launch ----

static rtsdf_trace_tuning g_tuning = {28, 0, 0, 4, 1, 12, 64, 2};
constexpr int kMaxBlocksPerCu = 8;  // persistent workgroups per CU (direction buffers and spill area sized for this)
constexpr int kMinShortStack = 12 - kEntryStack;  // smallest LDS stack part (spill area sized for this)
constexpr int kMaxStackDepth = 64;  // deepest hierarchy the tracer takes

static bool tuning_ok(const rtsdf_trace_tuning &t)
{
    if (t.refill != 16 && t.refill != 28) return false;
    if (t.blocks_per_cu < 0 || t.blocks_per_cu > kMaxBlocksPerCu) return false;
    if (t.stats < 0 || t.stats > 1 || t.loop < 0 || t.loop > 4) return false;
    if (t.bin_directions < 0 || t.bin_directions > 1) return false;
    if (t.stack_lds != 12 && t.stack_lds != 16 && t.stack_lds != 24) return false;
    if (t.tile_texels != 16 && t.tile_texels != 32 && t.tile_texels != 64) return false;
    if (t.bvh_width != 2 && t.bvh_width != 4) return false;
    return true;
}

template <int SL, int REFILL, int LOOP, bool STATS, bool BATCHED, bool INST = false, bool WIDE = false>
static int launch_trace5(TraceArgs A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    int per_cu = T.blocks_per_cu;
    if (per_cu <= 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, trace_persistent<SL, REFILL, LOOP, STATS, BATCHED>,
                                                         kTraceWaves * kWave, 0) != hipSuccess ||
            per_cu <= 0)
            per_cu = 2;
    }
    per_cu = std::min(per_cu, kMaxBlocksPerCu);
    const int blocks = num_cus() * per_cu;
    A.spill_stride = blocks * kTraceWaves * kWave;
    A.bin_directions = T.bin_directions;
    A.tile_cap = T.tile_texels;
    trace_persistent<SL, REFILL, LOOP, STATS, BATCHED, INST, WIDE><<<dim3(blocks), dim3(kTraceWaves * kWave), 0, s>>>(A);
    RTSDF_CHECK_LAUNCH();
    return RTSDF_OK;
}

template <int SL, int REFILL, int LOOP, bool BATCHED>
static int launch_trace4(const TraceArgs &A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    return T.stats ? launch_trace5<SL, REFILL, LOOP, true, BATCHED>(A, T, s)
                   : launch_trace5<SL, REFILL, LOOP, false, BATCHED>(A, T, s);
}

template <int SL, int REFILL, bool BATCHED>
static int launch_trace3(const TraceArgs &A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    switch (T.loop) {
    case 0: return launch_trace4<SL, REFILL, 0, BATCHED>(A, T, s);
    case 1: return launch_trace4<SL, REFILL, 1, BATCHED>(A, T, s);
    case 2: return launch_trace4<SL, REFILL, 2, BATCHED>(A, T, s);
    case 4:
        if constexpr (!BATCHED)  // (see kFewRays)
            if (A.few_rays) return launch_trace4<SL, REFILL, 5, false>(A, T, s);
        return launch_trace4<SL, REFILL, 4, BATCHED>(A, T, s);
    default: return launch_trace4<SL, REFILL, 3, BATCHED>(A, T, s);
    }
}

template <int SL, bool BATCHED>
static int launch_trace2(const TraceArgs &A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    return T.refill == 16 ? launch_trace3<SL, 16, BATCHED>(A, T, s) : launch_trace3<SL, 28, BATCHED>(A, T, s);
}

// two-level scenes: the one-fetch loop only
template <int SL, int REFILL>
static int launch_trace_inst2(const TraceArgs &A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    return T.stats ? launch_trace5<SL, REFILL, 3, true, false, true>(A, T, s)
                   : launch_trace5<SL, REFILL, 3, false, false, true>(A, T, s);
}

template <int SL>
static int launch_trace_inst1(const TraceArgs &A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    return T.refill == 16 ? launch_trace_inst2<SL, 16>(A, T, s) : launch_trace_inst2<SL, 28>(A, T, s);
}

static int launch_trace_inst(const TraceArgs &A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    switch (T.stack_lds) {
    case 12: return launch_trace_inst1<12>(A, T, s);
    case 24: return launch_trace_inst1<24>(A, T, s);
    default: return launch_trace_inst1<16>(A, T, s);
    }
}

// 4-wide single-scene launches: the one-fetch loop only
template <int SL, int REFILL>
static int launch_trace_wide2(const TraceArgs &A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    return T.stats ? launch_trace5<SL, REFILL, 3, true, false, false, true>(A, T, s)
                   : launch_trace5<SL, REFILL, 3, false, false, false, true>(A, T, s);
}

static int launch_trace_wide(const TraceArgs &A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    switch (T.stack_lds) {
    case 12: return T.refill == 16 ? launch_trace_wide2<12, 16>(A, T, s) : launch_trace_wide2<12, 28>(A, T, s);
    case 24: return T.refill == 16 ? launch_trace_wide2<24, 16>(A, T, s) : launch_trace_wide2<24, 28>(A, T, s);
    default: return T.refill == 16 ? launch_trace_wide2<16, 16>(A, T, s) : launch_trace_wide2<16, 28>(A, T, s);
    }
}

template <bool BATCHED>
static int launch_trace(const TraceArgs &A, const rtsdf_trace_tuning &T, hipStream_t s)
{
    switch (T.stack_lds) {
    case 12: return launch_trace2<12, BATCHED>(A, T, s);
    case 24: return launch_trace2<24, BATCHED>(A, T, s);
    default: return launch_trace2<16, BATCHED>(A, T, s);
    }
}

static int stack_depth_for(const rtsdf_scene *sc) { return sc->max_depth + 1; }

// stack entries a 4-wide traversal can hold at once: up to three pushed at each wide level on the path
// (levels 0 .. depth4), plus one
static int wide_stack_depth(const rtsdf_scene *sc) { return 3 * (sc->depth4 + 1) + 1; }

// whether a trace of this scene with tuning T runs the 4-wide loop
static bool trace_wide(const rtsdf_scene *sc, const rtsdf_trace_tuning &T)
{
    return T.bvh_width == 4 && sc->nodes4 && sc->ninst == 0 && wide_stack_depth(sc) <= kMaxStackDepth;
}

// the tuning a trace of this scene uses: its own if set, else the process default
static const rtsdf_trace_tuning &tuning_for(const rtsdf_scene *sc)
{
    return sc->has_tuning ? sc->tuning : g_tuning;
}

// Trace workspace: 256 B of counters, the wavefronts' direction buffers, then
// the spill area for stack entries deeper than the LDS part (per lane of the
// largest launch, for the deepest hierarchy the tracer takes).  Everything a
// launch writes besides its outputs lives here, so launches with separate
// workspaces can run concurrently, on one scene too.
static size_t trace_lanes_max() { return (size_t)num_cus() * kMaxBlocksPerCu * kTraceWaves * kWave; }
static size_t dirs_bytes() { return (size_t)num_cus() * kMaxBlocksPerCu * kTraceWaves * 2 * kTileRays * sizeof(float4); }
static size_t spill_bytes() { return trace_lanes_max() * (kMaxStackDepth - kMinShortStack) * sizeof(int32_t); }
static size_t trace_ws_bytes() { return 256 + dirs_bytes() + spill_bytes(); }
static float4 *ws_dirs(void *ws) { return reinterpret_cast<float4 *>(static_cast<char *>(ws) + 256); }
static int32_t *ws_spill(void *ws) { return reinterpret_cast<int32_t *>(static_cast<char *>(ws) + 256 + dirs_bytes()); }

}  // namespace rtsdf

extern "C" int rtsdf_trace_config(const rtsdf_trace_tuning *t)
{
    if (!t || !rtsdf::tuning_ok(*t)) return RTSDF_EINVAL;
    rtsdf::g_tuning = *t;
    return RTSDF_OK;
}

extern "C" int rtsdf_scene_set_tuning(rtsdf_scene *scene, const rtsdf_trace_tuning *t)
{
    if (!scene || (t && !rtsdf::tuning_ok(*t))) return RTSDF_EINVAL;
    if (t && t->bvh_width == 4 && !scene->nodes4) {  // the 4-wide copy is built on first use
        const int rc = rtsdf::wide_build(scene, nullptr);
        if (rc != RTSDF_OK) return rc;
        if (rtsdf::wide_stack_depth(scene) > rtsdf::kMaxStackDepth) return RTSDF_EINVAL;
    }
    scene->has_tuning = t != nullptr;
    if (t) scene->tuning = *t;
    return RTSDF_OK;
}

extern "C" int rtsdf_scene_get_tuning(const rtsdf_scene *scene, rtsdf_trace_tuning *t)
{
    if (!scene || !t) return RTSDF_EINVAL;
    *t = rtsdf::tuning_for(scene);
    return RTSDF_OK;
}

extern "C" int rtsdf_trace_config_get(rtsdf_trace_tuning *t)
{
    if (!t) return RTSDF_EINVAL;
    *t = rtsdf::g_tuning;
    return RTSDF_OK;
}

extern "C" int rtsdf_accum_reset(rtsdf_grid fine, rtsdf_accum st, rtsdf_stream stream)
{
    using namespace rtsdf;
    if (!grid_ok(fine) || !st.u || !st.hits || !st.arg_tri || !st.arg_ray) return RTSDF_EINVAL;
    const int64_t n = (int64_t)fine.n * fine.n * fine.n;
    int64_t blocks = std::min<int64_t>((n + 255) / 256, 8192);
    accum_reset_kernel<<<dim3((unsigned)blocks), dim3(256), 0, as_stream(stream)>>>(n, st.u, st.hits, st.arg_tri, st.arg_ray);
    RTSDF_CHECK_LAUNCH();
    return RTSDF_OK;
}

extern "C" size_t rtsdf_trace_workspace_size(void) { return rtsdf::trace_ws_bytes(); }

extern "C" int rtsdf_trace_accumulate(const rtsdf_scene *scene, rtsdf_grid coarse, const float *coarse_sdf,
                                      rtsdf_grid fine, const uint8_t *mask, const int32_t *queue, const int32_t *count,
                                      int32_t queue_cap, int32_t rays_per_texel, uint32_t frame,
                                      const uint32_t *frame_ptr, uint64_t seed, uint32_t scene_id, float alpha,
                                      rtsdf_accum st, float *fine_sdf, void *workspace, rtsdf_stream stream)
{
    using namespace rtsdf;
    if (!scene || !grid_ok(coarse) || !grid_ok(fine) || !coarse_sdf || !mask || !count || !fine_sdf || !workspace)
        return RTSDF_EINVAL;
    if (!st.u || !st.hits || !st.arg_tri || !st.arg_ray) return RTSDF_EINVAL;
    if (!is_pow2(coarse.n) || !is_pow2(fine.n) || fine.n < coarse.n || fine.n > 1024) return RTSDF_EINVAL;
    if (queue_cap < 0 || (queue_cap > 0 && !queue)) return RTSDF_EINVAL;
    if (rays_per_texel < 1 || rays_per_texel > 64) return RTSDF_EINVAL;
    if (!(alpha >= 0.0f && alpha <= 1.0f)) return RTSDF_EINVAL;
    if (frame >= kMaxFrame && !frame_ptr) return RTSDF_EINVAL;
    const int sd = stack_depth_for(scene);
    if (sd > kMaxStackDepth) return RTSDF_EINVAL;
    rtsdf_trace_tuning T = tuning_for(scene);
    if (scene->nt >= (1 << 26)) return RTSDF_EINVAL;  // triangle ids share a 64-bit key with the distance
    if (T.loop == 4 && scene->nref >= kMaxQueuedRefs) T.loop = 3;  // queue entries hold 26-bit indices
    hipStream_t s = as_stream(stream);
    const int lognf = ilog2(fine.n), logr = ilog2(fine.n / coarse.n);
    const int64_t ntex = (int64_t)fine.n * fine.n * fine.n;
    trace_fill_unselected<<<dim3((unsigned)((ntex + 255) / 256)), dim3(256), 0, s>>>(
        mask, coarse_sdf, coarse.n, logr, lognf, ntex, st.u, st.hits, st.arg_tri, st.arg_ray, fine_sdf);
    RTSDF_CHECK_LAUNCH();
    int32_t *cursor = static_cast<int32_t *>(workspace);
    int rc = launch_fill<int32_t>(cursor, 0, T.stats ? 32 : 1, s);
    if (rc != RTSDF_OK) return rc;
    TraceArgs A{};
    TraceScene &P = A.one;
    P.bvh.nodes = scene->nodes;
    P.bvh.tris = scene->tris;
    P.bvh.tmap = scene->tmap;
    P.nodes4 = scene->nodes4;
    P.nt = scene->nt;
    P.queue = queue;
    P.count = count;
    P.queue_cap = queue_cap;
    P.coarse_sdf = coarse_sdf;
    P.nc = coarse.n;
    P.logr = logr;
    P.nf = fine.n;
    P.lognf = lognf;
    P.lox = fine.lo[0];
    P.loy = fine.lo[1];
    P.loz = fine.lo[2];
    P.hf = fine.h;
    P.rays = rays_per_texel;
    P.scene_id = scene_id;
    P.alpha = alpha;
    P.sign_policy = scene->sign_policy;
    P.shell = scene->shell;
    P.u = st.u;
    P.hits = st.hits;
    P.arg_tri = st.arg_tri;
    P.arg_ray = st.arg_ray;
    P.fine = fine_sdf;
    A.scenes = nullptr;
    A.tile_offset = nullptr;
    A.nscenes = 1;
    A.cursor = cursor;
    A.frame = frame;
    A.frame_ptr = frame_ptr;
    A.seed = seed;
    A.spill = ws_spill(workspace);
    A.spill_stride = 0;
    A.dirs = ws_dirs(workspace);
    A.few_rays = tile_texels_for(rays_per_texel, T.tile_texels) * rays_per_texel <= kFewRays;
    if (scene->ninst > 0) return launch_trace_inst(A, T, s);
    return trace_wide(scene, T) ? launch_trace_wide(A, T, s) : launch_trace<false>(A, T, s);
}

extern "C" int rtsdf_directions(const int32_t *texel, const uint32_t *frame, const int32_t *ray, int32_t n,
                                uint64_t seed, uint32_t scene_id, float *out, rtsdf_stream stream)
{
    using namespace rtsdf;
    if (n < 0 || (n > 0 && (!texel || !frame || !ray || !out))) return RTSDF_EINVAL;
    if (n == 0) return RTSDF_OK;
    directions_kernel<<<dim3((n + 255) / 256), dim3(256), 0, as_stream(stream)>>>(texel, frame, ray, n, seed, scene_id, out);
    RTSDF_CHECK_LAUNCH();
    return RTSDF_OK;
}

extern "C" int rtsdf_closest_hits(const rtsdf_scene *scene, const float *origins, const float *dirs, int32_t n,
                                  float *t_out, int32_t *tri_out, int32_t *front_out, rtsdf_stream stream)
{
    using namespace rtsdf;
    if (!scene || n < 0 || (n > 0 && (!origins || !dirs || !t_out || !tri_out || !front_out))) return RTSDF_EINVAL;
    if (scene->ninst > 0) return RTSDF_EINVAL;  // single-level scenes only
    if (n == 0) return RTSDF_OK;
    const int sd = stack_depth_for(scene);
    if (sd > kMaxStackDepth) return RTSDF_EINVAL;
    BvhView S{scene->nodes, scene->tris, scene->tmap};
    hipStream_t s = as_stream(stream);
    const dim3 g((n + 255) / 256), b(256);
    const int full = sd <= 32 ? 32 : 64;
    // short stacks first where the full ones leave no room for all rays at once (64 entries, 140,000 rays: 382 -> 265
    // us; 100,000: 248 -> 267; 32 entries, 320,000 rays: 357 -> 258; 250,000: 223 -> 236)
    const bool two = (int64_t)n * full * 4 > kChipLds && sd > kShortHitStack;
    const auto launch = [&](auto kernel) {
        kernel<<<g, b, 0, s>>>(S, scene->nt, origins, dirs, n, t_out, tri_out, front_out);
    };
    if (two) {
        launch(closest_hits_kernel<kShortHitStack, kHitsShort>);
        RTSDF_CHECK_LAUNCH();
        if (full == 32) launch(closest_hits_kernel<32, kHitsRest>);
        else launch(closest_hits_kernel<64, kHitsRest>);
    } else if (full == 32) {
        launch(closest_hits_kernel<32, kHitsAll>);
    } else {
        launch(closest_hits_kernel<64, kHitsAll>);
    }
    RTSDF_CHECK_LAUNCH();
    return RTSDF_OK;
}

extern "C" int rtsdf_trace_backward(const rtsdf_scene *scene, rtsdf_grid fine, rtsdf_accum st, const float *fine_sdf,
                                    const float *grad_fine, uint64_t seed, uint32_t scene_id, float *grad_v,
                                    rtsdf_stream stream)
{
    using namespace rtsdf;
    if (!scene || !grid_ok(fine) || !is_pow2(fine.n) || !st.arg_tri || !st.arg_ray || !fine_sdf || !grad_fine || !grad_v)
        return RTSDF_EINVAL;
    const int64_t ntex = (int64_t)fine.n * fine.n * fine.n;
    trace_backward_kernel<<<dim3((unsigned)((ntex + 255) / 256)), dim3(256), 0, as_stream(stream)>>>(
        scene->vertices, scene->faces, scene->nt, ilog2(fine.n), fine.lo[0], fine.lo[1], fine.lo[2], fine.h, st.arg_tri,
        st.arg_ray, fine_sdf, grad_fine, seed, scene_id, grad_v, ntex, scene->sign_policy == RTSDF_SIGN_VOTE);
    RTSDF_CHECK_LAUNCH();
    return RTSDF_OK;
}
