// Selection of the fine texels to ray trace (paper Sec. 2.2; the case
// c <= d of Eq. (1)), as a stream compaction.
//
// A fine texel is selected when the coarse voxel containing its centre has
// D^2 <= K, K = floor(((d + beta) / h_c)^2), which is c <= d in exact
// arithmetic.  Since the fine size is a power-of-two multiple r of the coarse
// size, the r^3 fine children of a coarse voxel are consecutive in fine Morton
// order (their codes are (coarse code) * r^3 + child), so the queue is built by
// compacting the coarse voxels in Morton order and expanding each selected one
// into its r^3 children.
//
//   select_count   one coarse voxel per lane in Morton order; wavefront ballot
//                  + popcount, per-block totals
//   select_scan    one workgroup: exclusive prefix of the block totals
//   select_scatter ballot + mbcnt rank inside the wavefront, wave offsets
//                  through LDS, block offset from the scan; writes r^3 queue
//                  entries per selected voxel
//   select_mask    the linear uint8 mask, four texels per lane
// Batches run these over all their scenes.  Single grids of 64^3 cells and more
// take wider kernels of the same steps:
//   select_rows    counts and mask in one read of the predicate, four cells
//                  (16 bytes) per lane in rows of 64
//   select_scan, or select_chunks + select_chunk_scan above 4096 blocks
//   select_expand  one Morton block of 1024 cells per workgroup, its selected
//                  cells listed in LDS and written out coalesced
// No workgroup ever waits on another, and the queue order is deterministic.
#include <mutex>

#include "common.hpp"

namespace rtsdf {

constexpr int kSelBlock = 256;
constexpr int kSelItems = 4;  // coarse voxels per lane per block
constexpr int kSelPerBlock = kSelBlock * kSelItems;

// What is compared: D^2 against the integer threshold K (point sampling of
// the coarse voxel), or a float field at the selection grid's own resolution
// against d (trilinear sampling, see rtsdf_coarse_trilinear).
struct SelPred {
    const int32_t *d2;
    int K;
    const float *field;
    float d;
};

template <bool FIELD>
__device__ __forceinline__ bool pred_at(const SelPred &p, int64_t idx)
{
    if (FIELD) return p.field[idx] <= p.d;
    return p.d2[idx] <= p.K;
}

template <bool FIELD>
__device__ __forceinline__ bool coarse_selected(const SelPred &p, uint32_t m, int logn)
{
    const uint32_t x = compact1by2(m), y = compact1by2(m >> 1), z = compact1by2(m >> 2);
    const int64_t idx = x + ((int64_t)y << logn) + ((int64_t)z << (2 * logn));
    return pred_at<FIELD>(p, idx);
}

__device__ __forceinline__ uint32_t wave_prefix(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

template <bool FIELD = false>
__device__ __forceinline__ void select_count_body(const SelPred &pr, int logn, uint32_t total,
                                                  uint32_t *__restrict__ block_sums, uint32_t blk)
{
    __shared__ uint32_t wsum[kSelBlock / kWave];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t cnt = 0;
    for (int it = 0; it < kSelItems; ++it) {
        const uint32_t m = blk * kSelPerBlock + it * kSelBlock + threadIdx.x;
        const bool sel = m < total && coarse_selected<FIELD>(pr, m, logn);
        cnt += (uint32_t)__popcll(__ballot(sel));
    }
    if (lane == 0) wsum[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t s = 0;
        for (int w = 0; w < kSelBlock / kWave; ++w) s += wsum[w];
        block_sums[blk] = s;
    }
}

template <bool FIELD>
__global__ void __launch_bounds__(kSelBlock) select_count(SelPred pr, int logn, uint32_t total,
                                                          uint32_t *__restrict__ block_sums)
{
    select_count_body<FIELD>(pr, logn, total, block_sums, blockIdx.x);
}

// count and the overflow check from the number of selected coarse voxels
__device__ __forceinline__ void select_total(uint64_t coarse, uint32_t r3, int32_t *__restrict__ count, int32_t cap)
{
    const uint64_t texels = coarse * r3;
    *count = texels > (uint64_t)INT32_MAX ? INT32_MAX : (int32_t)texels;
    if (texels > (uint64_t)cap) raise_error(RTSDF_ERR_QUEUE_FULL);
}

// Inclusive scan of one value per lane over a workgroup of W wavefronts; `before` excludes the lane's own, the sum of
// all is returned.  wsum: W words of LDS, free again after the next barrier.
template <int W>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *wsum, uint32_t &before)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == kWave - 1) wsum[wave] = x;
    __syncthreads();
    uint32_t base = 0, all = 0;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        base += k < wave ? wsum[k] : 0u;
        all += wsum[k];
    }
    before = base + x - v;
    return all;
}

// Exclusive scan of nblocks totals in one workgroup of 1024 lanes, in rounds
// of 4096 consecutive totals, four per lane (131,072 totals read 128 apart per
// lane took 230 us; above 4096 the chunks below take 10); also the grand total -> count
// (texels = coarse * r3) and the overflow check.
__device__ __forceinline__ void select_scan_body(uint32_t *__restrict__ sums, uint32_t nblocks, uint32_t r3,
                                                 int32_t *__restrict__ count, int32_t cap)
{
    __shared__ uint32_t wsum[1024 / kWave];
    uint64_t carry = 0;
    for (uint32_t b0 = 0; b0 < nblocks; b0 += 4096) {
        const uint32_t i0 = b0 + 4 * threadIdx.x;
        uint32_t v[4];
        for (int k = 0; k < 4; ++k) v[k] = i0 + k < nblocks ? sums[i0 + k] : 0u;
        uint32_t e;
        const uint32_t all = block_scan<1024 / kWave>(v[0] + v[1] + v[2] + v[3], wsum, e);
        e += (uint32_t)carry;
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < nblocks) sums[i0 + k] = e;
            e += v[k];
        }
        carry += all;
        __syncthreads();  // wsum is rewritten next round
    }
    if (threadIdx.x == 0) select_total(carry, r3, count, cap);
}

__global__ void __launch_bounds__(1024) select_scan(uint32_t *__restrict__ sums, uint32_t nblocks, uint32_t r3,
                                                    int32_t *__restrict__ count, int32_t cap)
{
    select_scan_body(sums, nblocks, r3, count, cap);
}

template <bool FIELD = false>
__device__ __forceinline__ void select_scatter_body(const SelPred &pr, int logn, uint32_t total,
                                                    const uint32_t *__restrict__ offsets, int logr, int nf,
                                                    int32_t *__restrict__ queue, int32_t cap, uint32_t blk)
{
    __shared__ uint32_t wsum[kSelItems][kSelBlock / kWave];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bool sel[kSelItems];
    uint32_t rank[kSelItems];
    for (int it = 0; it < kSelItems; ++it) {
        const uint32_t m = blk * kSelPerBlock + it * kSelBlock + threadIdx.x;
        sel[it] = m < total && coarse_selected<FIELD>(pr, m, logn);
        const uint64_t bal = __ballot(sel[it]);
        rank[it] = wave_prefix(bal);
        if (lane == 0) wsum[it][wave] = (uint32_t)__popcll(bal);
    }
    __syncthreads();
    const uint32_t r3 = 1u << (3 * logr);
    uint32_t base = offsets[blk];
    for (int it = 0; it < kSelItems; ++it) {
        uint32_t before = 0;
        for (int w = 0; w < wave; ++w) before += wsum[it][w];
        if (sel[it]) {
            const uint32_t m = blk * kSelPerBlock + it * kSelBlock + threadIdx.x;
            const uint64_t pos = ((uint64_t)(base + before + rank[it])) * r3;
            const uint32_t cx = compact1by2(m), cy = compact1by2(m >> 1), cz = compact1by2(m >> 2);
            for (uint32_t c = 0; c < r3; ++c) {
                if (pos + c >= (uint64_t)cap) break;
                const uint32_t fx = (cx << logr) | compact1by2(c), fy = (cy << logr) | compact1by2(c >> 1),
                               fz = (cz << logr) | compact1by2(c >> 2);
                queue[pos + c] = (int32_t)(fx + (uint32_t)nf * (fy + (uint32_t)nf * fz));
            }
        }
        for (int w = 0; w < kSelBlock / kWave; ++w) base += wsum[it][w];
    }
}

template <bool FIELD>
__global__ void __launch_bounds__(kSelBlock) select_scatter(SelPred pr, int logn, uint32_t total,
                                                            const uint32_t *__restrict__ offsets, int logr, int nf,
                                                            int32_t *__restrict__ queue, int32_t cap)
{
    select_scatter_body<FIELD>(pr, logn, total, offsets, logr, nf, queue, cap, blockIdx.x);
}

template <bool FIELD = false>
__device__ __forceinline__ void select_mask_body(const SelPred &pr, int logn, int logr, int nf, int64_t nquads,
                                                 uint32_t *__restrict__ mask4, int64_t q)
{
    if (q >= nquads) return;
    const int64_t j = q * 4;
    const int x = (int)(j % nf), y = (int)((j / nf) % nf), z = (int)(j / ((int64_t)nf * nf));
    const int cy = y >> logr, cz = z >> logr;
    const int64_t row = ((int64_t)cy << logn) + ((int64_t)cz << (2 * logn));
    uint32_t w = 0;
    for (int i = 0; i < 4; ++i) w |= (uint32_t)pred_at<FIELD>(pr, row + ((x + i) >> logr)) << (8 * i);
    mask4[q] = w;
}

template <bool FIELD>
__global__ void __launch_bounds__(256) select_mask(SelPred pr, int logn, int logr, int nf, int64_t nquads,
                                                   uint32_t *__restrict__ mask4)
{
    select_mask_body<FIELD>(pr, logn, logr, nf, nquads, mask4, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// ------------------------------------------------ grids of 64^3 and more ----

// Block totals and the mask, from one read of the predicate.  A workgroup takes 64 x 8 x 8 cells, four Morton blocks of
// 16 x 8 x 8 next to each other: 64 rows of 256 bytes, 16 bytes per lane, and writes each row's mask (64 bytes times
// r, r^2 rows) whole.  Bound by memory: a 512^3 field, 671 MB, in 158 us (4.2 TB/s, a large copy's 4.8); counting in
// Morton order, a lane per cell, and the mask in a pass of its own took 255 + 141 us.
template <bool FIELD>
__global__ void __launch_bounds__(256) select_rows(SelPred pr, int logn, int logr, int nf, uint32_t *__restrict__ mask4,
                                                   uint32_t *__restrict__ block_sums)
{
    __shared__ uint32_t cnts[4];
    const int t = threadIdx.x, quad = t & 15;
    const uint32_t logx = (uint32_t)logn - 6, logy = (uint32_t)logn - 3;
    const uint32_t X = (blockIdx.x & ((1u << logx) - 1)) * 64, Y = ((blockIdx.x >> logx) & ((1u << logy) - 1)) * 8,
                   Z = (blockIdx.x >> (logx + logy)) * 8;
    if (t < 4) cnts[t] = 0u;
    __syncthreads();
    const uint32_t x = X + 4 * quad;
    uint32_t nib[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const uint32_t row = it * 16 + (t >> 4), y = Y + (row & 7), z = Z + (row >> 3);
        const size_t idx = x + ((size_t)y << logn) + ((size_t)z << (2 * logn));
        if (FIELD) {
            const float4 v = *reinterpret_cast<const float4 *>(pr.field + idx);
            nib[it] = (v.x <= pr.d ? 1u : 0u) | (v.y <= pr.d ? 2u : 0u) | (v.z <= pr.d ? 4u : 0u) |
                      (v.w <= pr.d ? 8u : 0u);
        } else {
            const int4 v = *reinterpret_cast<const int4 *>(pr.d2 + idx);
            nib[it] = (v.x <= pr.K ? 1u : 0u) | (v.y <= pr.K ? 2u : 0u) | (v.z <= pr.K ? 4u : 0u) |
                      (v.w <= pr.K ? 8u : 0u);
        }
    }
    uint32_t c = 0;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const uint32_t row = it * 16 + (t >> 4), y = Y + (row & 7), z = Z + (row >> 3), b = nib[it];
        c += (uint32_t)__popc(b);
        if (logr == 0) {
            mask4[((size_t)x + ((size_t)y << logn) + ((size_t)z << (2 * logn))) >> 2] =
                (b & 1u) | (b & 2u) << 7 | (b & 4u) << 14 | (b & 8u) << 21;
            continue;
        }
        const int r = 1 << logr;
        for (int zz = 0; zz < r; ++zz)
            for (int yy = 0; yy < r; ++yy) {
                const size_t frow = (size_t)((z << logr) + zz) * nf + ((y << logr) + yy);
                uint32_t *m = mask4 + (frow * nf >> 2) + (x >> 2 << logr);
                if (logr == 1) {
                    *reinterpret_cast<uint2 *>(m) = make_uint2((b & 1u) * 0x0101u | (b >> 1 & 1u) * 0x01010000u,
                                                               (b >> 2 & 1u) * 0x0101u | (b >> 3 & 1u) * 0x01010000u);
                } else {
                    for (int w = 0; w < r; w += 4) {
                        const auto word = [&](int i) { return (b >> ((w + i) >> (logr - 2)) & 1u) * 0x01010101u; };
                        *reinterpret_cast<uint4 *>(m + w) = make_uint4(word(0), word(1), word(2), word(3));
                    }
                }
            }
    }
    // totals of the four Morton blocks: lanes with the same bits 2 and 3
    c += (uint32_t)__shfl_xor((int)c, 1);
    c += (uint32_t)__shfl_xor((int)c, 2);
    c += (uint32_t)__shfl_xor((int)c, 16);
    c += (uint32_t)__shfl_xor((int)c, 32);
    if ((t & 0x33) == 0) atomicAdd(&cnts[quad >> 2], c);
    __syncthreads();
    if (t < 4) block_sums[morton3(X + 16 * t, Y, Z) >> 10] = cnts[t];
}

// Exclusive scan of each 1024 consecutive totals (one workgroup each); the first of them, whose own prefix is 0, takes
// the chunk's total instead.
__global__ void __launch_bounds__(256) select_chunks(uint32_t *__restrict__ sums)
{
    __shared__ uint32_t wsum[256 / kWave];
    uint4 *p = reinterpret_cast<uint4 *>(sums + (size_t)blockIdx.x * 1024) + threadIdx.x;
    const uint4 v = *p;
    uint32_t e;
    const uint32_t all = block_scan<256 / kWave>(v.x + v.y + v.z + v.w, wsum, e);
    *p = make_uint4(threadIdx.x == 0 ? all : e, e + v.x, e + v.x + v.y, e + v.x + v.y + v.z);
}

// Exclusive scan of the chunks' totals (at most 1024 chunks) in their places, and the grand total.
__global__ void __launch_bounds__(1024) select_chunk_scan(uint32_t *__restrict__ sums, uint32_t nchunks, uint32_t r3,
                                                          int32_t *__restrict__ count, int32_t cap)
{
    __shared__ uint32_t wsum[1024 / kWave];
    const uint32_t t = threadIdx.x;
    uint32_t e;
    const uint32_t all = block_scan<1024 / kWave>(t < nchunks ? sums[(size_t)t * 1024] : 0u, wsum, e);
    if (t < nchunks) sums[(size_t)t * 1024] = e;
    if (t == 0) select_total(all, r3, count, cap);
}

// Queue entries of Morton block blockIdx.x (16 x 8 x 8 cells): the selected cells' Morton indices are listed in LDS in
// order, then all lanes write the list's r^3 children with consecutive stores.  A field's predicate is read back from
// the mask (a byte a cell instead of four).  A 512^3 field: 292 -> 118 us against a lane per cell in Morton order,
// 131,072 workgroups of mostly latency; 256^3 cells with 61 M texels selected: 171 -> 72 us (3.4 TB/s).
template <bool FIELD>
__global__ void __launch_bounds__(256) select_expand(SelPred pr, int logn, const uint32_t *__restrict__ sums,
                                                     int chunked, const uint32_t *__restrict__ mask4, int logr, int nf,
                                                     int32_t *__restrict__ queue, int32_t cap)
{
    __shared__ __align__(16) uint8_t sel[1024];
    __shared__ uint32_t list[1024];  // first child's texel index
    __shared__ uint32_t wsum[4];
    const uint32_t t = threadIdx.x, blk = blockIdx.x, m0 = blk << 10;
    const uint32_t X = compact1by2(m0), Y = compact1by2(m0 >> 1), Z = compact1by2(m0 >> 2);
    const uint32_t lx = (t & 3) * 4, ly = (t >> 2) & 7, lz = t >> 5;
    const size_t idx = X + lx + ((size_t)(Y + ly) << logn) + ((size_t)(Z + lz) << (2 * logn));
    uint32_t bytes;
    if (FIELD) {
        bytes = mask4[idx >> 2];
    } else {
        const int4 v = *reinterpret_cast<const int4 *>(pr.d2 + idx);
        bytes = (v.x <= pr.K ? 1u : 0u) | (v.y <= pr.K ? 0x100u : 0u) | (v.z <= pr.K ? 0x10000u : 0u) |
                (v.w <= pr.K ? 0x1000000u : 0u);
    }
    if (!__syncthreads_or(bytes != 0u)) return;
    const uint32_t m = morton3(lx, ly, lz);  // cells lx + 0 .. 3: Morton offsets 0, 1, 8, 9
    *reinterpret_cast<uint16_t *>(sel + m) = (uint16_t)bytes;
    *reinterpret_cast<uint16_t *>(sel + m + 8) = (uint16_t)(bytes >> 16);
    __syncthreads();
    const uint32_t four = *reinterpret_cast<const uint32_t *>(sel + 4 * t);  // Morton indices 4 t .. 4 t + 3
    uint32_t at;
    const uint32_t n = block_scan<4>((uint32_t)__popc(four), wsum, at);
    for (uint32_t k = 0; k < 4; ++k) {
        if (!(four >> (8 * k) & 1u)) continue;
        const uint32_t l = 4 * t + k;
        const uint32_t row = (Y + compact1by2(l >> 1)) + (uint32_t)nf * (Z + compact1by2(l >> 2));
        list[at++] = ((X + compact1by2(l)) + (uint32_t)nf * row) << logr;
    }
    __syncthreads();
    const uint32_t base = chunked ? sums[blk & ~1023u] + ((blk & 1023u) ? sums[blk] : 0u) : sums[blk];
    const uint64_t first = (uint64_t)base << (3 * logr);
    const uint32_t log3 = 3 * (uint32_t)logr, r3 = 1u << log3;
    const auto child = [&](uint32_t c) {
        return compact1by2(c) + (uint32_t)nf * (compact1by2(c >> 1) + (uint32_t)nf * compact1by2(c >> 2));
    };
    // a lane's entries are 256 apart: the same child of every 256 / r^3-th cell (r > 6: of one cell, child by child)
    const uint32_t end = (uint32_t)min((uint64_t)n << log3, (uint64_t)cap > first ? (uint64_t)cap - first : 0ull);
    if (r3 <= 256) {
        const uint32_t c = child(t & (r3 - 1));
        for (uint32_t e = t; e < end; e += 256) queue[first + e] = (int32_t)(list[e >> log3] + c);
    } else {
        for (uint32_t e = t; e < end; e += 256) queue[first + e] = (int32_t)(list[e >> log3] + child(e & (r3 - 1)));
    }
}

// Trilinear value of the coarse SDF at fine texel centres.  Coarse values sit
// at voxel centres; a fine centre at coarse coordinate u = (j + 1/2) / r - 1/2
// (r = fine / coarse size) is clamped to [0, n - 1], split into the cell
// i0 = floor(u), i1 = min(i0 + 1, n - 1) and the weight t = u - i0 (all exact
// for power-of-two r), and interpolated along x, then y, then z with
// lerp(a, b, t) = a + t (b - a), each float operation rounded once.  A cell
// with an infinite corner (no seed anywhere) gives +inf.
__device__ __forceinline__ void tri_axis(int j, float inv_r, int nc, int &i0, int &i1, float &t)
{
    float u = rn_sub(rn_mul(rn_add((float)j, 0.5f), inv_r), 0.5f);
    u = fminf(fmaxf(u, 0.0f), (float)(nc - 1));
    i0 = (int)u;  // u >= 0: truncation is the floor
    i1 = min(i0 + 1, nc - 1);
    t = rn_sub(u, (float)i0);
}

__device__ __forceinline__ float lerp_c(float a, float b, float t) { return rn_add(a, rn_mul(t, rn_sub(b, a))); }

__global__ void __launch_bounds__(256) coarse_trilinear_kernel(const float *__restrict__ c, int nc, int lognf, int logr,
                                                               float *__restrict__ out, int64_t ntex)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= ntex) return;
    const int nfm = (1 << lognf) - 1;
    const int jx = (int)(j & nfm), jy = (int)((j >> lognf) & nfm), jz = (int)(j >> (2 * lognf));
    const float inv_r = 1.0f / (float)(1 << logr);  // exact
    int x0, x1, y0, y1, z0, z1;
    float tx, ty, tz;
    tri_axis(jx, inv_r, nc, x0, x1, tx);
    tri_axis(jy, inv_r, nc, y0, y1, ty);
    tri_axis(jz, inv_r, nc, z0, z1, tz);
    auto at = [&](int x, int y, int z) { return c[x + (int64_t)nc * (y + (int64_t)nc * z)]; };
    const float c000 = at(x0, y0, z0), c100 = at(x1, y0, z0), c010 = at(x0, y1, z0), c110 = at(x1, y1, z0);
    const float c001 = at(x0, y0, z1), c101 = at(x1, y0, z1), c011 = at(x0, y1, z1), c111 = at(x1, y1, z1);
    const float m = fmaxf(fmaxf(fmaxf(c000, c100), fmaxf(c010, c110)), fmaxf(fmaxf(c001, c101), fmaxf(c011, c111)));
    if (isinf(m)) {
        out[j] = __builtin_inff();
        return;
    }
    const float c00 = lerp_c(c000, c100, tx), c10 = lerp_c(c010, c110, tx);
    const float c01 = lerp_c(c001, c101, tx), c11 = lerp_c(c011, c111, tx);
    const float c0 = lerp_c(c00, c10, ty), c1 = lerp_c(c01, c11, ty);
    out[j] = lerp_c(c0, c1, tz);
}

// The same for fine sizes of 2, 4, ... times the coarse size (r = 2^LOGR; LOGR = 3: 8 and more), four texels along x by
// two rows along y and z per lane.  Two neighbouring rows chosen not to straddle a coarse centre read the same two
// coarse rows (r = 2: rows 2 p - 1 and 2 p; r >= 4: rows 2 p and 2 p + 1), so interpolation along x serves four rows
// and that along y two, and the texels' 2 to 4 distinct columns are read once: 1 read and 9 roundings per texel instead
// of 8 and 21.  Bound by its writes: 512^3 from 256^3 376 -> 162 us (3.7 TB/s).  The operations of each texel are the
// ones above in the same order.
template <int LOGR>
__global__ void __launch_bounds__(256) coarse_trilinear_quads(const float *__restrict__ c, int nc, int lognf,
                                                              float inv_r, int pairs, float *__restrict__ out,
                                                              int64_t items)
{
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= items) return;
    const int nf = 1 << lognf, logq = lognf - 2;
    const int k = (int)(id & ((1 << logq) - 1)), rows = (int)(id >> logq), py = rows % pairs, pz = rows / pairs;
    constexpr int S = LOGR == 1 ? 1 : 0;  // first row of pair p: 2 p - S
    int y0, y1, z0, z1, i0, i1;
    float ty[2], tz[2], tx[4];
    // the pair's rows share their coarse rows; a row outside the grid (r = 2: the first and last pair) is not written
    tri_axis(min(max(2 * py - S, 0), nf - 1), inv_r, nc, y0, y1, ty[0]);
    tri_axis(min(2 * py - S + 1, nf - 1), inv_r, nc, y0, y1, ty[1]);
    tri_axis(min(max(2 * pz - S, 0), nf - 1), inv_r, nc, z0, z1, tz[0]);
    tri_axis(min(2 * pz - S + 1, nf - 1), inv_r, nc, z0, z1, tz[1]);
    // columns: texel q reads columns lo[q] and lo[q] + 1 of `col`, the coarse columns cb, cb + 1, ... (clamped)
    constexpr int NC = LOGR == 1 ? 4 : LOGR == 2 ? 3 : 2;
    int cb;
#pragma unroll
    for (int q = 0; q < 4; ++q) tri_axis(4 * k + q, inv_r, nc, i0, i1, tx[q]);
    if (LOGR == 1) cb = 2 * k - 1;
    else if (LOGR == 2) cb = k - 1;
    else cb = i0;
    const int64_t row[4] = {(int64_t)nc * (y0 + (int64_t)nc * z0), (int64_t)nc * (y1 + (int64_t)nc * z0),
                            (int64_t)nc * (y0 + (int64_t)nc * z1), (int64_t)nc * (y1 + (int64_t)nc * z1)};
    float col[4][NC];
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int q = 0; q < NC; ++q) col[w][q] = c[row[w] + min(max(cb + q, 0), nc - 1)];
    float res[2][2][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        // left of the first coarse centre the cell is that of columns 0 and 1 (weight 0)
        const int lo = LOGR == 1 ? (q + 1) / 2 : LOGR == 2 ? q / 2 : 0;
        const bool first = LOGR <= 2 && k == 0 && (LOGR == 1 ? q == 0 : q < 2);
        float xl[4], m = __builtin_nanf("");  // the largest corner that is a number, as above: NaN if there is none
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float a = first ? col[w][1] : col[w][lo], b = first ? col[w][NC > 2 ? 2 : 1] : col[w][lo + 1];
            m = fmaxf(m, fmaxf(a, b));
            xl[w] = lerp_c(a, b, tx[q]);
        }
        const bool inf = isinf(m);
#pragma unroll
        for (int yy = 0; yy < 2; ++yy) {
            const float a = lerp_c(xl[0], xl[1], ty[yy]), b = lerp_c(xl[2], xl[3], ty[yy]);
#pragma unroll
            for (int zz = 0; zz < 2; ++zz) res[zz][yy][q] = inf ? __builtin_inff() : lerp_c(a, b, tz[zz]);
        }
    }
#pragma unroll
    for (int zz = 0; zz < 2; ++zz)
#pragma unroll
        for (int yy = 0; yy < 2; ++yy) {
            const int jy = 2 * py - S + yy, jz = 2 * pz - S + zz;
            if (jy >= 0 && jy < nf && jz >= 0 && jz < nf)
                *reinterpret_cast<float4 *>(out + 4 * k + ((int64_t)jy << lognf) + ((int64_t)jz << (2 * lognf))) =
                    make_float4(res[zz][yy][0], res[zz][yy][1], res[zz][yy][2], res[zz][yy][3]);
        }
}

// K = floor(((d + beta) / h_c)^2), -1 if d + beta < 0
inline int select_threshold(float hc, float beta, float d)
{
    const double q = ((double)d + (double)beta) / (double)hc;
    if (q < 0) return -1;
    const double k = floor(q * q);
    return k > (double)INT32_MAX ? INT32_MAX : (int)k;
}


// The launches of a selection: cells of side 2^logn, r = 2^logr texels per cell and axis, with the block sums in `sums`
// (at least rtsdf_select_workspace_size bytes of the cells' grid, less the alignment).  Every sum the launches read is
// written earlier in the same sequence (counts, then scan), so `sums` needs no clearing.  The kernels of 64^3 and more
// move 16 bytes per lane and take 16-byte aligned arrays; smaller grids (whose time is the launches') and other arrays
// keep a lane per cell.
template <bool FIELD>
static int select_launch(const SelPred &pr, int logn, int logr, uint8_t *mask, int32_t *queue, int32_t cap,
                         int32_t *count, uint32_t *sums, hipStream_t s)
{
    const int n = 1 << logn, nf = n << logr;
    const uint32_t total = (uint32_t)((int64_t)n * n * n), r3 = 1u << (3 * logr);
    const uint32_t nblocks = (total + kSelPerBlock - 1) / kSelPerBlock;
    uint32_t *mask4 = reinterpret_cast<uint32_t *>(mask);
    sums = reinterpret_cast<uint32_t *>((reinterpret_cast<uintptr_t>(sums) + 15) & ~(uintptr_t)15);
    const uintptr_t align = reinterpret_cast<uintptr_t>(FIELD ? (const void *)pr.field : (const void *)pr.d2) |
                            reinterpret_cast<uintptr_t>(mask);
    if (logn >= 6 && (align & 15) == 0) {
        select_rows<FIELD><<<dim3(nblocks / 4), dim3(256), 0, s>>>(pr, logn, logr, nf, mask4, sums);
        RTSDF_CHECK_LAUNCH();
        const int chunked = nblocks > 4096;  // 128^3 cells: 2048 blocks, one round of the one-workgroup scan
        if (chunked) {
            select_chunks<<<dim3(nblocks / 1024), dim3(256), 0, s>>>(sums);
            RTSDF_CHECK_LAUNCH();
            select_chunk_scan<<<dim3(1), dim3(1024), 0, s>>>(sums, nblocks / 1024, r3, count, cap);
        } else {
            select_scan<<<dim3(1), dim3(1024), 0, s>>>(sums, nblocks, r3, count, cap);
        }
        RTSDF_CHECK_LAUNCH();
        select_expand<FIELD><<<dim3(nblocks), dim3(256), 0, s>>>(pr, logn, sums, chunked, mask4, logr, nf, queue, cap);
        RTSDF_CHECK_LAUNCH();
        return RTSDF_OK;
    }
    select_count<FIELD><<<dim3(nblocks), dim3(kSelBlock), 0, s>>>(pr, logn, total, sums);
    RTSDF_CHECK_LAUNCH();
    select_scan<<<dim3(1), dim3(1024), 0, s>>>(sums, nblocks, r3, count, cap);
    RTSDF_CHECK_LAUNCH();
    select_scatter<FIELD><<<dim3(nblocks), dim3(kSelBlock), 0, s>>>(pr, logn, total, sums, logr, nf, queue, cap);
    RTSDF_CHECK_LAUNCH();
    const int64_t nquads = (int64_t)nf * nf * nf / 4;
    select_mask<FIELD><<<dim3((unsigned)((nquads + 255) / 256)), dim3(256), 0, s>>>(pr, logn, logr, nf, nquads, mask4);
    RTSDF_CHECK_LAUNCH();
    return RTSDF_OK;
}

// Point-sampled selection.
static int select_run(rtsdf_grid coarse, const int32_t *dist2, rtsdf_grid fine, float beta, float d, uint8_t *mask,
                      int32_t *queue, int32_t queue_cap, int32_t *count, uint32_t *sums, hipStream_t s)
{
    const SelPred pr{dist2, select_threshold(coarse.h, beta, d), nullptr, 0.0f};
    return select_launch<false>(pr, ilog2(coarse.n), ilog2(fine.n / coarse.n), mask, queue, queue_cap, count, sums, s);
}

static bool select_args_ok(rtsdf_grid coarse, const int32_t *dist2, rtsdf_grid fine, float beta, float d,
                           const uint8_t *mask, const int32_t *queue, int32_t queue_cap, const int32_t *count)
{
    if (!grid_ok(coarse) || !grid_ok(fine) || !is_pow2(coarse.n) || coarse.n > 512) return false;
    if (!is_pow2(fine.n) || fine.n < coarse.n || fine.n > 1024 || fine.n < 4) return false;
    if ((double)fine.h * fine.n != (double)coarse.h * coarse.n) return false;
    if (fine.lo[0] != coarse.lo[0] || fine.lo[1] != coarse.lo[1] || fine.lo[2] != coarse.lo[2]) return false;
    if (!dist2 || !mask || !count || queue_cap < 0 || (queue_cap > 0 && !queue)) return false;
    if (!(beta == beta) || !(d == d)) return false;
    return true;
}

// Scratch of the allocation-free selection: the block sums of the largest
// coarse grid rtsdf_select takes (512^3 voxels -> 131,072 blocks), 512 KiB per
// device, held until the process ends.  Host code never passes `scratch`
// itself to a kernel (on the host it is only a stand-in for the symbol); it
// uses the device address hipGetSymbolAddress returns for each device.
constexpr size_t kSelScratchWords = ((size_t)512 * 512 * 512 + kSelPerBlock - 1) / kSelPerBlock + 64;
__device__ __align__(256) uint32_t scratch[kSelScratchWords];

constexpr int kMaxDevices = 64;
static uint32_t *g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mu;

// The current device's address of `scratch`, looked up once per device.
static uint32_t *scratch_for_current_device()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        g_scratch_ptr[dev] = static_cast<uint32_t *>(ptr);
    }
    return g_scratch_ptr[dev];
}

}  // namespace rtsdf

extern "C" size_t rtsdf_select_workspace_size(int32_t coarse_n)
{
    using namespace rtsdf;
    if (coarse_n <= 0) return 0;
    const int64_t total = (int64_t)coarse_n * coarse_n * coarse_n;
    return (size_t)(((total + kSelPerBlock - 1) / kSelPerBlock) * sizeof(uint32_t) + 256);
}

extern "C" int rtsdf_select(rtsdf_grid coarse, const int32_t *dist2, rtsdf_grid fine, float beta, float d,
                            uint8_t *mask, int32_t *queue, int32_t queue_cap, int32_t *count, void *workspace,
                            rtsdf_stream stream)
{
    using namespace rtsdf;
    if (!select_args_ok(coarse, dist2, fine, beta, d, mask, queue, queue_cap, count) || !workspace)
        return RTSDF_EINVAL;
    return select_run(coarse, dist2, fine, beta, d, mask, queue, queue_cap, count, static_cast<uint32_t *>(workspace),
                      as_stream(stream));
}

extern "C" size_t rtsdf_select_noalloc_max_bytes(void) { return rtsdf::kSelScratchWords * sizeof(uint32_t); }

extern "C" int rtsdf_select_noalloc(rtsdf_grid coarse, const int32_t *dist2, rtsdf_grid fine, float beta, float d,
                                    uint8_t *mask, int32_t *queue, int32_t queue_cap, int32_t *count,
                                    rtsdf_stream stream)
{
    using namespace rtsdf;
    if (!select_args_ok(coarse, dist2, fine, beta, d, mask, queue, queue_cap, count)) return RTSDF_EINVAL;
    if (rtsdf_select_workspace_size(coarse.n) > kSelScratchWords * sizeof(uint32_t)) return RTSDF_EINVAL;
    uint32_t *sums = scratch_for_current_device();
    if (!sums) return RTSDF_EHIP;
    return select_run(coarse, dist2, fine, beta, d, mask, queue, queue_cap, count, sums, as_stream(stream));
}

extern "C" int rtsdf_coarse_trilinear(rtsdf_grid coarse, const float *coarse_sdf, rtsdf_grid fine, float *fine_c,
                                      rtsdf_stream stream)
{
    using namespace rtsdf;
    if (!grid_ok(coarse) || !grid_ok(fine) || !is_pow2(coarse.n) || !is_pow2(fine.n)) return RTSDF_EINVAL;
    if (fine.n < coarse.n || fine.n > 1024 || coarse.n > 512) return RTSDF_EINVAL;
    if ((double)fine.h * fine.n != (double)coarse.h * coarse.n) return RTSDF_EINVAL;
    if (fine.lo[0] != coarse.lo[0] || fine.lo[1] != coarse.lo[1] || fine.lo[2] != coarse.lo[2]) return RTSDF_EINVAL;
    if (!coarse_sdf || !fine_c) return RTSDF_EINVAL;
    const int64_t ntex = (int64_t)fine.n * fine.n * fine.n;
    const int lognf = ilog2(fine.n), logr = ilog2(fine.n / coarse.n);
    hipStream_t s = as_stream(stream);
    if (logr >= 1 && fine.n >= 16 && (reinterpret_cast<uintptr_t>(fine_c) & 15) == 0) {
        const int pairs = fine.n / 2 + (logr == 1 ? 1 : 0);
        const int64_t items = (int64_t)(fine.n / 4) * pairs * pairs;
        const dim3 grid((unsigned)((items + 255) / 256)), block(256);
        const float inv_r = 1.0f / (float)(1 << logr);  // exact
        if (logr == 1)
            coarse_trilinear_quads<1><<<grid, block, 0, s>>>(coarse_sdf, coarse.n, lognf, inv_r, pairs, fine_c, items);
        else if (logr == 2)
            coarse_trilinear_quads<2><<<grid, block, 0, s>>>(coarse_sdf, coarse.n, lognf, inv_r, pairs, fine_c, items);
        else
            coarse_trilinear_quads<3><<<grid, block, 0, s>>>(coarse_sdf, coarse.n, lognf, inv_r, pairs, fine_c, items);
    } else {
        coarse_trilinear_kernel<<<dim3((unsigned)((ntex + 255) / 256)), dim3(256), 0, s>>>(coarse_sdf, coarse.n, lognf,
                                                                                           logr, fine_c, ntex);
    }
    RTSDF_CHECK_LAUNCH();
    return RTSDF_OK;
}

extern "C" int rtsdf_select_field(rtsdf_grid grid, const float *field, float d, uint8_t *mask, int32_t *queue,
                                  int32_t queue_cap, int32_t *count, void *workspace, rtsdf_stream stream)
{
    using namespace rtsdf;
    if (!grid_ok(grid) || !is_pow2(grid.n) || grid.n < 4 || grid.n > 1024) return RTSDF_EINVAL;
    if (!field || !mask || !count || !workspace || queue_cap < 0 || (queue_cap > 0 && !queue)) return RTSDF_EINVAL;
    if (!(d == d)) return RTSDF_EINVAL;
    const SelPred pr{nullptr, 0, field, d};
    return select_launch<true>(pr, ilog2(grid.n), 0, mask, queue, queue_cap, count, static_cast<uint32_t *>(workspace),
                               as_stream(stream));
}
