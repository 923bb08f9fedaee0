// Pillarization and point-feature canvas for gfx950.
//
// Deterministic sort of points by cell (LDS, no order-dependent result), over
// a group of agents released together (the blocks of the group's agents are
// interleaved, see group_block; a single release is a group of one).
// Small inputs (pillars_small_fits) take one launch before the point-feature
// net, one block per agent:
//   pillars_small LDS counts of every cell (16 bits each), each point's rank in
//                its cell from the LDS atomic, a block scan over the cells ->
//                the pillar lists and each point's place in cell order
// Larger ones three.  Cells are cut into tiles of PillarGroup::tile_cells,
// points into blocks of kPtsPerBlock:
//   bin_count    cell id per point; per point block, an LDS histogram of its
//                points over the tiles, the point's rank in its (block,
//                tile) bin from the LDS atomic; every non-empty bin
//                reserves its run in its tile (one global atomic per
//                non-empty bin, not one per point)
//   bin_scatter  the tiles' first points (each block scans the tiles'
//                totals itself), point indices and cells in tile order
//   tile_sort    one block per tile: LDS counts of the tile's cells, their
//                scan -> the tile's pillars in ascending cell order and
//                each point's place in cell order (member, sorted); the
//                block publishes its pillar count, adds up those of the
//                tiles before it and writes its part of the global lists
// Then for both:
//   pfn_canvas   one lane per (two pillars, 8 channels): linear 4 -> C,
//                ReLU, max over the pillar's points into its cell.  Extra
//                blocks take the crowded pillars, one wavefront each, and
//                move the cap lowest point indices (found by bisection on
//                the index value) of those over the cap to the front of the
//                segment
// The canvas is zero outside the pillars: canvas_clear zeroes the last
// frame's pillar cells again (off the encoder's path: the executor runs it
// when the next frame begins, before any branch input has arrived).
// The only order-dependent intermediate is the order of members inside a
// segment, and every consumer of it is order-independent (max, set
// selection), so every output is bitwise reproducible.
#include <climits>

#include "kernels.hpp"

namespace rtcc {
namespace kern {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ inline int2 add2(int2 a, int2 b) { return make_int2(a.x + b.x, a.y + b.y); }

// Inclusive scan across the 64 lanes of a wavefront.
__device__ inline int2 wave_incl_scan(int2 v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int ax = __shfl_up(v.x, d, 64);
        int ay = __shfl_up(v.y, d, 64);
        if (lane >= d) {
            v.x += ax;
            v.y += ay;
        }
    }
    return v;
}

// Exclusive scan of one int2 per thread over a 256-thread block.
__device__ inline int2 block_excl_scan256(int2 v, int2 *total) {
    __shared__ int2 wsum[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int2 inc = wave_incl_scan(v);
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int2 base = make_int2(0, 0), tot = make_int2(0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i < w) base = add2(base, wsum[i]);
        tot = add2(tot, wsum[i]);
    }
    __syncthreads();
    *total = tot;
    return make_int2(base.x + inc.x - v.x, base.y + inc.y - v.y);
}

// One point per lane, so that a whole input is in flight over the bus at once.
// Bound by the bus; six agents with 4,027 points (387 KB) cost the frame 100 us
// less than a DMA copy, an event and a wait each (461 -> 361).
__global__ __launch_bounds__(256) void k_points_upload(const PointsUpload u) {
    const int j = blockIdx.x % u.m, i = int(blockIdx.x / u.m) * 256 + int(threadIdx.x);
    if (i < u.n[j]) u.dst[j][i] = u.src[j][i];
}

__global__ __launch_bounds__(256) void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256)
        p[i] = v;
}

// 16 bytes with the non-temporal hint: the canvas is read by the backbone,
// not by the pillar kernels.
__device__ inline void nt_store16(void *p, uint4 v) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, static_cast<u32x4 *>(p));
}

// Block -> (agent row j of the group, block index b within that agent's
// grid): the agents' blocks are interleaved.  The dispatcher hands
// consecutive blocks to the XCDs in turn, so in a group of 8 every agent's
// blocks run on one XCD, and the random accesses of its pillar stage (cell
// counts, offsets, member lists) stay in that XCD's L2.
struct GroupBlock {
    int j, b, nb;  // agent row, block within the agent, blocks per agent
};
__device__ inline GroupBlock group_block(const PillarGroup &grp) {
    const int m = grp.m;
    return GroupBlock{int(blockIdx.x) % m, int(blockIdx.x) / m, int(gridDim.x) / m};
}
__device__ inline PillarBufs group_bufs(const PillarGroup &grp, int j) { return grp.bufs[grp.agent[j]]; }

__device__ inline int cell_of(const float4 p, const PillarGeom &g) {
    int c = -1;
    if (__builtin_isfinite(p.x) && __builtin_isfinite(p.y) && __builtin_isfinite(p.z) &&
        __builtin_isfinite(p.w) && p.x >= g.x0 && p.x < g.x1 && p.y >= g.y0 && p.y < g.y1 &&
        p.z >= g.z0 && p.z < g.z1) {
        // float32, round-to-nearest subtract and divide, then floor
        const float fx = floorf(__fdiv_rn(__fsub_rn(p.x, g.x0), g.v));
        const float fy = floorf(__fdiv_rn(__fsub_rn(p.y, g.y0), g.v));
        if (fx >= 0.f && fx < float(g.W) && fy >= 0.f && fy < float(g.H)) c = int(fy) * g.W + int(fx);
    }
    return c;
}

inline __device__ int blocks_of(int n) { return (n + kPtsPerBlock - 1) / kPtsPerBlock; }

// K1: cell ids, per-(block, tile) counts and the block's run in every
// tile; two points per thread.
__global__ __launch_bounds__(256) void k_bin_count(const PillarGroup grp, const PillarGeom g) {
    extern __shared__ int lds[];  // [grp.tiles] counts, then [grp.tiles] bases
    int *hist = lds, *base = lds + grp.tiles;
    const GroupBlock gb = group_block(grp);
    const int j = gb.j;
    const int n = grp.n[j];
    if (gb.b >= blocks_of(n)) return;  // the whole block: past this agent's points
    const PillarBufs B = group_bufs(grp, j);
    const float4 *pts = grp.pts[j];
    for (int t = threadIdx.x; t < grp.tiles; t += 256) hist[t] = 0;
    __syncthreads();
    int tile[2], rank[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = gb.b * kPtsPerBlock + u * 256 + int(threadIdx.x);
        tile[u] = -1;
        if (i < n) {
            const int c = cell_of(pts[i], g);
            B.cell[i] = c;
            if (c >= 0) {
                tile[u] = c / grp.tile_cells;
                rank[u] = atomicAdd(&hist[tile[u]], 1);
            }
        }
    }
    __syncthreads();
    // the block's run in every tile it touches: one global atomic per
    // non-empty (block, tile) bin
    for (int t = threadIdx.x; t < grp.tiles; t += 256) {
        const int h = hist[t];
        if (h > 0) base[t] = atomicAdd(&B.ttotal[t], h);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (tile[u] >= 0) B.slot[gb.b * kPtsPerBlock + u * 256 + int(threadIdx.x)] = base[tile[u]] + rank[u];
}

// K2: every point to its place in tile order.  Each block scans the tiles'
// totals in LDS into the tiles' first points; the agent's first block also
// stores them (tstart) and the point count.
__global__ __launch_bounds__(256) void k_bin_scatter(const PillarGroup grp) {
    extern __shared__ int ts[];  // [grp.tiles + 1]
    const GroupBlock gb = group_block(grp);
    const int j = gb.j;
    const int n = grp.n[j];
    const PillarBufs B = group_bufs(grp, j);
    const int T = grp.tiles;
    const int per = (T + 255) / 256;
    int s = 0;
    for (int r = 0; r < per; ++r) {
        const int t = int(threadIdx.x) * per + r;
        if (t < T) s += B.ttotal[t];
    }
    int2 tot;
    int acc = block_excl_scan256(make_int2(s, 0), &tot).x;
    for (int r = 0; r < per; ++r) {
        const int t = int(threadIdx.x) * per + r;
        if (t < T) {
            ts[t] = acc;
            acc += B.ttotal[t];
        }
    }
    if (threadIdx.x == 0) ts[T] = tot.x;
    __syncthreads();
    if (gb.b == 0) {
        for (int t = threadIdx.x; t <= T; t += 256) {
            B.tstart[t] = ts[t];
            if (t < T) B.npil[t] = 0;  // not published yet
        }
        if (threadIdx.x == 0) {
            B.meta[0] = tot.x;
            B.meta[1] = 0;  // the last tile writes the pillar count
            B.meta[2] = 0;  // crowded pillars, appended to by the tile sort
            B.meta[3] = 0;  // tiles taken
        }
    }
    if (gb.b >= blocks_of(n)) return;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = gb.b * kPtsPerBlock + u * 256 + int(threadIdx.x);
        if (i < n) {
            const int c = B.cell[i];
            if (c >= 0) {
                const int d = ts[c / grp.tile_cells] + B.slot[i];
                B.binned[d] = i;
                B.cellb[d] = c;
            }
        }
    }
}

// K3: one block per tile of cells; 256 threads, CPT cells each.  A block takes
// its tile by a ticket, so the blocks of all earlier tiles have started when
// it waits for their pillar counts (each is published before its block waits
// for anything): the wait always ends.
constexpr int kSortCache = 8;
template <int CPT>
__global__ __launch_bounds__(256) void k_tile_sort(const PillarGroup grp, int32_t crowd) {
    constexpr int CELLS = 256 * CPT;
    __shared__ int cnt[CELLS];
    __shared__ int loff[CELLS];
    __shared__ int ticket, first_crowded;
    const int j = group_block(grp).j;
    const PillarBufs B = group_bufs(grp, j);
    const float4 *pts = grp.pts[j];
    if (threadIdx.x == 0) ticket = atomicAdd(&B.meta[3], 1);
    for (int q = threadIdx.x; q < CELLS; q += 256) cnt[q] = 0;
    __syncthreads();
    const int t = ticket;
    const int lo = B.tstart[t], hi = B.tstart[t + 1];
    const int c0 = t * CELLS;
    // the tile's first kSortCache * 256 points keep their cell and rank in
    // registers between the passes; any further ones go through `rank`
    int lcell[kSortCache], rk[kSortCache];
#pragma unroll
    for (int u = 0; u < kSortCache; ++u) {
        const int e = lo + int(threadIdx.x) + u * 256;
        lcell[u] = e < hi ? B.cellb[e] - c0 : 0;
    }
#pragma unroll
    for (int u = 0; u < kSortCache; ++u)
        if (lo + int(threadIdx.x) + u * 256 < hi) rk[u] = atomicAdd(&cnt[lcell[u]], 1);
    for (int e = lo + int(threadIdx.x) + kSortCache * 256; e < hi; e += 256)
        B.rank[e] = atomicAdd(&cnt[B.cellb[e] - c0], 1);
    __syncthreads();
    int v[CPT];
    int s = 0, f = 0;  // points; pillars, and the crowded ones above 16 bits
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        v[i] = cnt[threadIdx.x * CPT + i];
        s += v[i];
        f += int(v[i] > 0) + (int(v[i] > crowd) << 16);
    }
    int2 tot;
    const int2 ex = block_excl_scan256(make_int2(s, f), &tot);
    if (threadIdx.x == 0) {
        __hip_atomic_store(&B.npil[t], (tot.y & 0xffff) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        first_crowded = tot.y >> 16 ? atomicAdd(&B.meta[2], tot.y >> 16) : 0;
    }
    int off = ex.x;
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        loff[threadIdx.x * CPT + i] = off;
        off += v[i];
    }
    __syncthreads();
    int idx[kSortCache];
#pragma unroll
    for (int u = 0; u < kSortCache; ++u) {
        const int e = lo + int(threadIdx.x) + u * 256;
        idx[u] = e < hi ? B.binned[e] : 0;
    }
#pragma unroll
    for (int u = 0; u < kSortCache; ++u) {
        const int e = lo + int(threadIdx.x) + u * 256;
        if (e < hi) {
            const int d = lo + loff[lcell[u]] + rk[u];
            B.member[d] = idx[u];
            B.sorted[d] = pts[idx[u]];
        }
    }
    for (int e = lo + int(threadIdx.x) + kSortCache * 256; e < hi; e += 256) {
        const int d = lo + loff[B.cellb[e] - c0] + B.rank[e];
        const int i = B.binned[e];
        B.member[d] = i;
        B.sorted[d] = pts[i];
    }
    // the tile's pillars to their place in the global lists, behind those of
    // the tiles before it
    int before = 0;
    for (int q = threadIdx.x; q < t; q += 256) {
        int np;
        while ((np = __hip_atomic_load(&B.npil[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) __builtin_amdgcn_s_sleep(1);
        before += np - 1;
    }
    int2 all;
    block_excl_scan256(make_int2(before, 0), &all);
    int p = all.x + (ex.y & 0xffff), k = first_crowded + (ex.y >> 16);
    off = ex.x;
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        if (v[i] > 0) {
            B.pcells[p] = c0 + int(threadIdx.x) * CPT + i;
            B.pcounts[p] = v[i];
            B.poffs[p] = lo + off;
            if (v[i] > crowd) B.crowded[k++] = p;
            ++p;
        }
        off += v[i];
    }
    if (threadIdx.x == 0) {
        if (t == grp.tiles - 1) B.meta[1] = all.x + (tot.y & 0xffff);
        // the tile's point total back to zero, the state the next frame's
        // bin count starts from (every reader of it has finished)
        B.ttotal[t] = 0;
    }
}

// The whole sort of one agent in one block: at most PER x 1024 points and
// CELLS cells, two 16-bit counts (then offsets) per LDS word; the points stay
// in registers.  Bound by latency and by what one CU can issue (16 wavefronts).
template <int CELLS, int PER>
__global__ __launch_bounds__(1024) void k_pillars_small(const PillarGroup grp, const PillarGeom g, int32_t crowd) {
    __shared__ uint32_t cnt[CELLS / 2];
    __shared__ int2 wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = blockIdx.x;
    const int n = grp.n[j];
    const PillarBufs B = group_bufs(grp, j);
    const f32x4_t *pv = reinterpret_cast<const f32x4_t *>(grp.pts[j]);
    const int words = (grp.n_cells + 1) / 2;
    for (int w = tid; w < words; w += 1024) cnt[w] = 0u;
    __syncthreads();
    f32x4_t q[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = u * 1024 + tid;
        q[u] = i < n ? pv[i] : f32x4_t{INFINITY, 0.f, 0.f, 0.f};  // no cell
    }
    int at[PER];  // cell + (rank in the cell << 16); -1: dropped
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int c = cell_of(make_float4(q[u].x, q[u].y, q[u].z, q[u].w), g);
        at[u] = -1;
        if (c >= 0) {
            const int sh = (c & 1) * 16;
            at[u] = c | int(((atomicAdd(&cnt[c >> 1], 1u << sh) >> sh) & 0xffffu) << 16);
        }
    }
    __syncthreads();
    // an odd number of consecutive words per thread: no bank conflicts
    const int per = ((words + 1023) / 1024) | 1;
    const int w0 = tid * per < words ? tid * per : words, w1 = w0 + per < words ? w0 + per : words;
    int2 v = make_int2(0, 0);  // points; pillars, and the crowded ones above 16 bits
#pragma unroll 4
    for (int w = w0; w < w1; ++w) {
        const int a = cnt[w] & 0xffffu, b = cnt[w] >> 16;
        v.x += a + b;
        v.y += int(a > 0) + int(b > 0) + ((int(a > crowd) + int(b > crowd)) << 16);
    }
    const int2 inc = wave_incl_scan(v);
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int2 base = make_int2(0, 0), tot = make_int2(0, 0);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        if (q < wave) base = add2(base, wsum[q]);
        tot = add2(tot, wsum[q]);
    }
    const int before = base.y + inc.y - v.y;
    int off = base.x + inc.x - v.x, p = before & 0xffff, k = before >> 16;
    for (int w = w0; w < w1; ++w) {
        const uint32_t both = cnt[w];
        cnt[w] = uint32_t(off) | (uint32_t(off + int(both & 0xffffu)) << 16);
        auto list = [&](int c, int count) {
            if (count == 0) return;
            B.pcells[p] = c;
            B.pcounts[p] = count;
            B.poffs[p] = off;
            if (count > crowd) B.crowded[k++] = p;
            off += count;
            ++p;
        };
        list(2 * w, int(both & 0xffffu));
        list(2 * w + 1, int(both >> 16));
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (at[u] < 0) continue;
        const int c = at[u] & 0xffff;
        const int d = int((cnt[c >> 1] >> ((c & 1) * 16)) & 0xffffu) + (at[u] >> 16);
        B.member[d] = u * 1024 + tid;
        reinterpret_cast<f32x4_t *>(B.sorted)[d] = q[u];
    }
    if (tid == 0) {
        B.meta[0] = tot.x;
        B.meta[1] = tot.y & 0xffff;
        B.meta[2] = tot.y >> 16;
    }
}

__device__ inline uint32_t pack_bf16x2(float a, float b) {
    uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    ua += 0x7fffu + ((ua >> 16) & 1u);
    ub += 0x7fffu + ((ub >> 16) & 1u);
    return (ua >> 16) | (ub & 0xffff0000u);
}

// One point's contribution to 8 channels of its pillar: ReLU(b + W^T f),
// f = (x / hx, y / hy, (z - z0) / dz, r), maxed into mx.  The same code for
// pillars under and over the cap.
__device__ inline void pfn_point(const PfnArgs &a, const float4 pt, const float (&w0)[8], const float (&w1)[8],
                                 const float (&w2)[8], const float (&w3)[8], const float (&bb)[8], float (&mx)[8]) {
    const float f0 = pt.x * a.inv_hx;
    const float f1 = pt.y * a.inv_hy;
    const float f2 = (pt.z - a.z0) * a.inv_dz;
    const float f3 = pt.w;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float h = bb[i] + w0[i] * f0 + w1[i] * f1 + w2[i] * f2 + w3[i] * f3;
        h = h > 0.f ? h : 0.f;  // +0 for every non-positive value
        mx[i] = fmaxf(mx[i], h);
    }
}

template <bool BF16>
__device__ inline void store_canvas8(const PfnArgs &a, void *canvas, int cell, int ch, const float (&mx)[8]) {
    if (BF16) {
        uint4 o;
        o.x = pack_bf16x2(mx[0], mx[1]);
        o.y = pack_bf16x2(mx[2], mx[3]);
        o.z = pack_bf16x2(mx[4], mx[5]);
        o.w = pack_bf16x2(mx[6], mx[7]);
        nt_store16(static_cast<uint16_t *>(canvas) + size_t(cell) * a.C + ch, o);
    } else {
        float *dst = static_cast<float *>(canvas) + size_t(cell) * a.C + ch;
        nt_store16(dst, make_uint4(__float_as_uint(mx[0]), __float_as_uint(mx[1]), __float_as_uint(mx[2]),
                                   __float_as_uint(mx[3])));
        nt_store16(dst + 4, make_uint4(__float_as_uint(mx[4]), __float_as_uint(mx[5]), __float_as_uint(mx[6]),
                                       __float_as_uint(mx[7])));
    }
}

// Blocks from a.crowd_blocks on: a lane per (two pillars, 8 channels) of the
// global pillar list takes ReLU(W^T f + b) maxed over the pillar's points,
// read in segment order from `sorted`, into the pillar's cell.  Crowded
// pillars (more than a.crowd points) are left to the blocks before them, one
// wavefront each: a lane that walked a pillar of 20 or 30 points held up its
// wavefront, and the kernel, for as many loads and 8 times as many
// multiply-adds in a row.  Of a pillar over the cap that wavefront first moves
// the cap lowest point indices to the front of its segment (member indices
// and points).  The other cells of the canvas already hold zeros.  One agent with 40,000 points 16.6 -> 7.3 us, 6,000
// on 2,640 cells 13.5 -> 5.1, 100,000 on 512 x 512 cells 12.8 -> 10.8.
template <bool BF16>
__global__ __launch_bounds__(256) void k_pfn_canvas(const PfnArgs a, const PillarGroup grp) {
    // PFN weights and bias, read once per block into LDS (C <= 512)
    __shared__ float sw[5 * 512];
    for (int q = threadIdx.x; q < 5 * a.C; q += 256) sw[q] = q < 4 * a.C ? a.w[q] : a.b[q - 4 * a.C];
    __syncthreads();
    const GroupBlock gb = group_block(grp);
    const int j = gb.j;
    const PillarBufs B = group_bufs(grp, j);
    void *const canvas = a.canvas ? a.canvas : B.canvas;
    if (gb.b < a.crowd_blocks) {
        // crowded pillars, one wavefront each: 8 channels per lane, and where
        // the channel groups divide the wavefront its lanes share the points
        // (a maximum does not depend on the order)
        const int lane = threadIdx.x & 63;
        const int wave = (gb.b * 256 + int(threadIdx.x)) >> 6;
        const int n_waves = (a.crowd_blocks * 256) >> 6;
        const int n_crowded = B.meta[2];
        const float4 *pts = grp.pts[j];
        const int groups = a.C >> 3;
        const bool share = groups <= 64 && (64 % groups) == 0;
        const int pg = share ? lane / groups : 0, npg = share ? 64 / groups : 1;
        float w0[8], w1[8], w2[8], w3[8], bb[8];
        auto weights = [&](int ch) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                w0[i] = sw[0 * a.C + ch + i];
                w1[i] = sw[1 * a.C + ch + i];
                w2[i] = sw[2 * a.C + ch + i];
                w3[i] = sw[3 * a.C + ch + i];
                bb[i] = sw[4 * a.C + ch + i];
            }
        };
        if (share) weights((lane % groups) * 8);
        for (int w = wave; w < n_crowded; w += n_waves) {
            const int p = B.crowded[w];
            const int c = B.pcells[p];
            const int cnt = B.pcounts[p];
            int32_t *seg = B.member + B.poffs[p];
            float4 *sseg = B.sorted + B.poffs[p];
            if (cnt > a.max_pts && !a.replay) {
                // the first 256 members stay in registers
                int e[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) e[u] = u * 64 + lane < cnt ? seg[u * 64 + lane] : INT_MAX;
                // Smallest T with #{members < T} >= max_pts.  Members are
                // distinct point indices in [0, n), so exactly max_pts members
                // lie below T.
                int lo = 1, hi = grp.n[j];
                while (lo < hi) {
                    const int mid = lo + (hi - lo) / 2;
                    int below = 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u) below += __popcll(__ballot(e[u] < mid));
                    for (int q0 = 256; q0 < cnt; q0 += 64)
                        below += __popcll(__ballot(q0 + lane < cnt && seg[q0 + lane] < mid));
                    if (below >= a.max_pts) hi = mid;
                    else lo = mid + 1;
                }
                const int T = lo;
                // Stable in-place compaction of the selected members to the
                // front: a chunk is read completely before any of it is
                // overwritten, and writes never pass the chunk being read.
                int pos = 0;
                auto move = [&](int m) {
                    const unsigned long long sel = __ballot(m < T);
                    if (m < T) {
                        const int my = pos + __popcll(sel & ((1ull << lane) - 1ull));
                        seg[my] = m;
                        sseg[my] = pts[m];
                    }
                    pos += __popcll(sel);
                };
#pragma unroll
                for (int u = 0; u < 4; ++u) move(e[u]);
                for (int q0 = 256; q0 < cnt && pos < a.max_pts; q0 += 64)
                    move(q0 + lane < cnt ? seg[q0 + lane] : INT_MAX);
                // the wave's own writes above are read back by other lanes
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            const int used = cnt < a.max_pts ? cnt : a.max_pts;
            for (int ch = (share ? lane % groups : lane) * 8; ch < a.C; ch += 64 * 8) {
                if (!share) weights(ch);
                float mx[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) mx[i] = 0.f;
#pragma unroll 2
                for (int t = pg; t < used; t += npg) pfn_point(a, sseg[t], w0, w1, w2, w3, bb, mx);
                if (share)
                    for (int d = groups; d < 64; d <<= 1)
#pragma unroll
                        for (int i = 0; i < 8; ++i) mx[i] = fmaxf(mx[i], __shfl_xor(mx[i], d, 64));
                if (pg == 0) store_canvas8<BF16>(a, canvas, c, ch, mx);
            }
        }
        return;
    }
    // two pillars per lane (8 channels of each): their loads are in flight
    // together
    const int lanes_per_cell = a.C >> 3;
    const int gid = (gb.b - a.crowd_blocks) * 256 + int(threadIdx.x);
    const int pp = gid / lanes_per_cell;
    const int ch = (gid - pp * lanes_per_cell) * 8;
    const int P = B.meta[1];
    const int p0 = 2 * pp;
    if (p0 >= P) return;
    const bool has1 = p0 + 1 < P;
    const int cell0 = B.pcells[p0], cnt0 = B.pcounts[p0], off0 = B.poffs[p0];
    const int cell1 = has1 ? B.pcells[p0 + 1] : 0;
    const int cnt1 = has1 ? B.pcounts[p0 + 1] : 0;
    const int off1 = has1 ? B.poffs[p0 + 1] : off0;
    // crowded pillars are left to the blocks above
    const int n0 = cnt0 <= a.crowd ? cnt0 : 0;
    const int n1 = cnt1 <= a.crowd ? cnt1 : 0;
    float w0[8], w1[8], w2[8], w3[8], bb[8], m0[8], m1[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        w0[i] = sw[0 * a.C + ch + i];
        w1[i] = sw[1 * a.C + ch + i];
        w2[i] = sw[2 * a.C + ch + i];
        w3[i] = sw[3 * a.C + ch + i];
        bb[i] = sw[4 * a.C + ch + i];
        m0[i] = 0.f;
        m1[i] = 0.f;
    }
    // the last point of a pillar stands in for the points past its end (the
    // max is unchanged by a repeat); every index stays inside its segment
    const int l0 = n0 > 0 ? n0 - 1 : 0, l1 = n1 > 0 ? n1 - 1 : 0;
    const int tmax = n0 > n1 ? n0 : n1;
    for (int t = 0; t < tmax; ++t) {
        const float4 q0 = B.sorted[off0 + (t < l0 ? t : l0)];
        const float4 q1 = B.sorted[off1 + (t < l1 ? t : l1)];
        if (n0 > 0) pfn_point(a, q0, w0, w1, w2, w3, bb, m0);
        if (n1 > 0) pfn_point(a, q1, w0, w1, w2, w3, bb, m1);
    }
    if (n0 > 0) store_canvas8<BF16>(a, canvas, cell0, ch, m0);
    if (n1 > 0) store_canvas8<BF16>(a, canvas, cell1, ch, m1);
}

// The canvas cells of the last frame's pillars back to zero, one lane per
// (pillar, 8 channels), for every agent of the group (its pillar list and
// count are those of its last encoder); the rest of each canvas holds zeros
// already.
template <bool BF16>
__global__ __launch_bounds__(256) void k_canvas_clear(const PillarGroup grp, int32_t C) {
    const GroupBlock gb = group_block(grp);
    const PillarBufs B = group_bufs(grp, gb.j);
    const int lanes = C >> 3;
    const int gid = gb.b * 256 + int(threadIdx.x);
    const int p = gid / lanes;
    if (p >= B.meta[1]) return;
    const size_t off = size_t(B.pcells[p]) * C + (gid - p * lanes) * 8;
    if (BF16) {
        nt_store16(static_cast<uint16_t *>(B.canvas) + off, make_uint4(0u, 0u, 0u, 0u));
    } else {
        nt_store16(static_cast<float *>(B.canvas) + off, make_uint4(0u, 0u, 0u, 0u));
        nt_store16(static_cast<float *>(B.canvas) + off + 4, make_uint4(0u, 0u, 0u, 0u));
    }
}

inline unsigned blocks_for(int64_t n, int per) { return unsigned((n + per - 1) / per); }

}  // namespace

hipError_t fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    unsigned g = blocks_for(n, 256);
    if (g > 4096) g = 4096;
    k_fill_i32<<<g, 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

hipError_t points_upload(const PointsUpload &u, hipStream_t s) {
    int32_t n_max = 0;
    for (int j = 0; j < u.m; ++j) n_max = u.n[j] > n_max ? u.n[j] : n_max;
    if (n_max <= 0) return hipSuccess;
    k_points_upload<<<blocks_for(n_max, 256) * unsigned(u.m), 256, 0, s>>>(u);
    return hipGetLastError();
}

hipError_t bin_count(const PillarGroup &grp, const PillarGeom &g, hipStream_t s) {
    if (grp.n_max <= 0) return hipSuccess;
    k_bin_count<<<blocks_for(grp.n_max, kPtsPerBlock) * unsigned(grp.m), 256, size_t(grp.tiles) * 8, s>>>(grp, g);
    return hipGetLastError();
}

hipError_t bin_scatter(const PillarGroup &grp, hipStream_t s) {
    // at least one block per agent: the first one stores the tile starts
    const unsigned nb = grp.n_max > 0 ? blocks_for(grp.n_max, kPtsPerBlock) : 1u;
    k_bin_scatter<<<nb * unsigned(grp.m), 256, size_t(grp.tiles + 1) * 4, s>>>(grp);
    return hipGetLastError();
}

hipError_t tile_sort(const PillarGroup &grp, int32_t crowd, hipStream_t s) {
    const unsigned g = unsigned(grp.tiles) * unsigned(grp.m);
    if (grp.tile_cells == kTileCellsFine) k_tile_sort<kTileCellsFine / 256><<<g, 256, 0, s>>>(grp, crowd);
    else if (grp.tile_cells == kTileCells) k_tile_sort<kTileCells / 256><<<g, 256, 0, s>>>(grp, crowd);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t pillars_small(const PillarGroup &grp, const PillarGeom &g, int32_t crowd, hipStream_t s) {
    if (!pillars_small_fits(grp.n_cells, grp.n_max, true)) return hipErrorInvalidValue;
    const unsigned blocks = unsigned(grp.m);
    if (grp.n_cells <= kSmallCells) k_pillars_small<kSmallCells, kSmallPoints / 1024><<<blocks, 1024, 0, s>>>(grp, g, crowd);
    else k_pillars_small<kSmallCells * 4, kSmallPoints / 2048><<<blocks, 1024, 0, s>>>(grp, g, crowd);
    return hipGetLastError();
}

hipError_t pfn_canvas(bool bf16, PfnArgs a, const PillarGroup &grp, int32_t max_pillars, hipStream_t s) {
    // blocks for the crowded pillars (four at a time each), which take the
    // longest, then the others.  At most one per CU over all agents: more hold the
    // others up (eight agents with 100,000 points, 256 for each -> for all, us:
    // clustered on 512 x 512 cells 43.8 -> 41.0, spread evenly 41.0 -> 39.2, on 352
    // x 100 cells 32.3 -> 29.8; over the cap only 53, 39, 29.6)
    const unsigned crowds = blocks_for(grp.n_max / (a.crowd + 1), 4), most = 256u / unsigned(grp.m);
    a.crowd_blocks = int32_t(crowds < most ? crowds : most);
    const unsigned blocks = unsigned(a.crowd_blocks) + blocks_for(int64_t((max_pillars + 1) / 2) * (a.C / 8), 256);
    if (blocks == 0) return hipSuccess;
    const unsigned grid = blocks * unsigned(grp.m);
    if (bf16) k_pfn_canvas<true><<<grid, 256, 0, s>>>(a, grp);
    else k_pfn_canvas<false><<<grid, 256, 0, s>>>(a, grp);
    return hipGetLastError();
}

hipError_t canvas_clear(bool bf16, const PillarGroup &grp, int32_t C, int32_t max_pillars, hipStream_t s) {
    const unsigned blocks = blocks_for(int64_t(max_pillars) * (C / 8), 256);
    if (blocks == 0) return hipSuccess;
    const unsigned grid = blocks * unsigned(grp.m);
    if (bf16) k_canvas_clear<true><<<grid, 256, 0, s>>>(grp, C);
    else k_canvas_clear<false><<<grid, 256, 0, s>>>(grp, C);
    return hipGetLastError();
}

}  // namespace kern
}  // namespace rtcc
