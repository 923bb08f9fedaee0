// Host launchers of the gfx950 kernels.  Every launcher checks nothing but
// enqueues on the given stream and returns hipGetLastError(); the executor
// validates shapes before calling.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "conv_plan.hpp"

namespace rtcc {
namespace kern {

// ------------------------------------------------------------ pillarization
struct PillarGeom {
    float x0, x1, y0, y1, z0, z1, v;
    int H, W;
};

// Cells per tile of the pillar sort (PillarGroup::tile_cells): fine tiles up to
// kFineCells cells, for enough blocks on small grids (352 x 100 cells: 69
// blocks instead of 18 per agent); above, coarse ones, as every 512-point
// block reserves a run in each tile it touches (at 512 x 512 cells fine tiles
// would take an atomic per point).
constexpr int kTileCells = 2048, kTileCellsFine = 512, kFineCells = 131072;
inline int pillar_tile_cells(int n_cells) { return n_cells <= kFineCells ? kTileCellsFine : kTileCells; }

hipError_t fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s);

// One agent's pillar-stage buffers (device pointers, fixed for a context).
// With tiles = ceil(H*W / tile_cells) tiles of cells, the sizes are: cell,
// slot, binned, cellb, rank, member [n_max]; sorted [n_max] points; ttotal
// [tiles] (zero between frames); tstart [tiles + 1]; npil [tiles]; pcells,
// pcounts, poffs [min(n_max, H*W)]; crowded [n_max / (pfn_crowd(max_pts) + 1)
// + 1]; meta [4] (valid points, pillars, crowded pillars, tiles taken); canvas
// [H*W][C].
struct PillarBufs {
    int32_t *cell, *slot, *ttotal, *tstart, *binned, *cellb, *rank, *npil;
    int32_t *pcells, *pcounts, *poffs, *crowded, *member, *meta;
    float4 *sorted;
    void *canvas;
};

constexpr int kPtsPerBlock = 512;  // points per block of the per-point kernels

// The agents whose pillar stage one launch chain runs: agent row j is agent
// agent[j] (its buffers bufs[agent[j]], its n[j] points at pts[j]).  One
// agent is a group of one.
constexpr int kMaxGroup = 16;
struct PillarGroup {
    const PillarBufs *bufs;  // device array, indexed by agent
    const float4 *pts[kMaxGroup];
    int32_t n[kMaxGroup];
    int32_t agent[kMaxGroup];
    int32_t m;       // agents in the group, 1..kMaxGroup
    int32_t n_max;   // max over the group of n[j]
    int32_t n_cells; // H * W
    int32_t tiles;   // ceil(n_cells / tile_cells)
    int32_t tile_cells; // kTileCells or kTileCellsFine
};

// The points of m agents from pinned host memory to device memory, one launch.
struct PointsUpload {
    const float4 *src[kMaxGroup];
    float4 *dst[kMaxGroup];
    int32_t n[kMaxGroup];
    int32_t m;
};
hipError_t points_upload(const PointsUpload &u, hipStream_t s);

// A pillar of more points is crowded: above the cap, or above a few, where a
// lane's walk over the points costs more than a wavefront for the pillar.  Six,
// so that a cloud spread over its cells evenly, three points in each, has few of
// them (pfn_canvas, us, more than four / six / eight / twelve points):
//   clustered  100,000 on 512 x 512 cells      13.6 / 12.1 / 12.7 / 13.4
//              6,000 on 352 x 100               7.6 /  8.0 /  8.6 / 11.3
//   even       100,000 on 352 x 100            16.6 / 10.9 / 11.3 / 11.7
inline int32_t pfn_crowd(int32_t max_pts) { return max_pts < 6 ? max_pts : 6; }

// The sort of points by cell (counting in LDS):
// K1 bin_count: cell id per point (-1 if dropped); per block of
//    kPtsPerBlock points, its points' count in every tile of cells, one
//    atomic ttotal[tile] += count per non-empty tile (ttotal starts at
//    zero) reserving the block's run in the tile, and each point's
//    position within its tile (slot).
// K2 bin_scatter: tstart[t] = first point of tile t in tile order,
//    tstart[tiles] = meta[0] = valid points, meta[2] (crowded count), meta[3]
//    and npil = 0; binned / cellb = point index / cell in tile order.
// K3 tile_sort: per tile, LDS counts of its cells: the tile's pillars in
//    ascending cell order at their place in the global lists pcells / pcounts
//    / poffs (npil[tile] - 1 of them), the pillars of more than `crowd` points
//    listed in crowded (by that place, meta[2] of them), member / sorted = the points in
//    cell order (rank within a cell: an arbitrary order); meta[1] = P pillars;
//    ttotal back to zero.
hipError_t bin_count(const PillarGroup &grp, const PillarGeom &g, hipStream_t s);
hipError_t bin_scatter(const PillarGroup &grp, hipStream_t s);
hipError_t tile_sort(const PillarGroup &grp, int32_t crowd, hipStream_t s);
// K1 to K3 in one launch, one block per agent, for small inputs: the same
// lists, member and sorted points.  Two launches fewer, about 10 us of the host
// where branches are released apart, against a kernel that grows with the
// points and cells of one agent: such releases take it as far as it reaches, a
// group and a lone agent, where the stage is all that runs, up to half of that.
// A frame, us, one block -> three launches:
//                          points per agent
//                              2,000        4,000        6,000        8,000
//   64 x 64, float32, apart, 8 196 -> 215   199 -> 217   200 -> 220   206 -> 219
//     a group of 8              90 -> 95     94 -> 96     97 -> 97    101 -> 99
//     a group of 8, graphs     118 -> 115   119 -> 116   122 -> 117   125 -> 119
//   128 x 128, bf16, apart, 8  305 -> 342   306 -> 345   315 -> 345   328 -> 343
//     apart, 4, graphs         243 -> 258   244 -> 263   252 -> 258   272 -> 261
//     a group of 8             132 -> 137   137 -> 139   142 -> 140   147 -> 141
//     one agent, graphs        116 -> 119   119 -> 120   123 -> 119   128 -> 121
//   44 x 60, bf16, apart, 4, graphs                      331 -> 341
//   352 x 100, bf16, apart, 8  513 -> 555   509 -> 544
//     a group of 8             284 -> 285   287 -> 286
constexpr int kSmallPoints = 8192, kSmallCells = 16384;
inline bool pillars_small_fits(int n_cells, int n_max, bool apart) {
    const int points = apart ? kSmallPoints : kSmallPoints / 2;
    return n_cells <= kSmallCells ? n_max <= points : n_cells <= kSmallCells * 4 && n_max <= points / 2;
}
hipError_t pillars_small(const PillarGroup &grp, const PillarGeom &g, int32_t crowd, hipStream_t s);
// K4 pfn_canvas: the dense canvas [H*W][C]: per pillar cell, channel max over the first
// min(count, max_pts) members of ReLU(W^T f + b) (for cells over the cap,
// after moving the max_pts lowest point indices to the front of the
// segment).  Writes the pillar cells only: every other cell must already be
// zero (canvas_clear zeroes the previous frame's pillars).
struct PfnArgs {
    const float *w;  // [4][C]
    const float *b;  // [C]
    int32_t C;
    int32_t max_pts;
    int32_t crowd;  // pfn_crowd(max_pts): pillars of more points take a wavefront each
    float inv_hx, inv_hy, z0, inv_dz;
    int32_t crowd_blocks;  // set by pfn_canvas
    // replay = 1: the pillars over the cap already hold their selected points
    // first (a previous launch on the same lists chose them), so they are
    // not chosen again; the canvas cells come out bit for bit as in that
    // launch.  canvas: where the cells go (nullptr: the agent's canvas).
    int32_t replay;
    void *canvas;
};
// max_pillars bounds every agent's meta[1] (at most min(cells, points)).
hipError_t pfn_canvas(bool bf16, PfnArgs a, const PillarGroup &grp, int32_t max_pillars, hipStream_t s);
// For every agent of the group, the canvas cells of the pillars listed in its
// pcells (meta[1] of them) back to zero; max_pillars bounds meta[1].  Only
// grp.bufs, grp.agent and grp.m are read.
hipError_t canvas_clear(bool bf16, const PillarGroup &grp, int32_t C, int32_t max_pillars, hipStream_t s);

// ------------------------------------------------------------ implicit GEMM
// conv:   out[m][c_off + n] for m = output pixel, 3x3 taps, pad 1, stride.
// deconv: A rows are input pixels, phase = blockIdx.z, output pixel
//         (iy * u + py, ix * u + px), skipped outside Ho x Wo.
struct GemmArgs {
    const void *in;    // NHWC, channel stride Ci
    const void *wt;    // Bt[N][K] (conv) or u*u phases of Bt[N][Ci] (deconv)
    const float *bias; // [N]
    void *out;         // NHWC, channel stride ldo
    int32_t Hi, Wi, Ci;
    int32_t Ho, Wo;
    int32_t N;
    int32_t stride;    // conv only
    int32_t u;         // deconv only
    int32_t ldo, c_off;
    int32_t splits;    // K slices (>= 1); > 1 needs ws and a conv (no deconv)
    int32_t variant;   // conv kernel: kConvImplicit or one of the halo tilings
    const void *zero;  // >= 16 zero bytes in device memory (padding reads)
    float *ws;         // split-K partials [splits][M][N] float32
    // Several agents' maps side by side in one launch (the same layer and
    // weights): batch > 1 takes agent b's input, output and split-K partials
    // from in_b / out_b / ws_b [b] instead of in / out / ws.  Every output
    // element is computed exactly as in a launch of its own.
    int32_t batch;     // 0 or 1: one map
    const void *in_b[16];
    void *out_b[16];
    float *ws_b[16];
    const void *wfrag; // conv_slices: the weights in fragment order (conv_frag)
    int32_t n_cu;      // conv_slices: compute units of the GPU
    int32_t slices;    // halo tilings, > 1: the channel chunks in that many slices, added in order (splits = 1)
};
// With start / stop events, the first kernel of the convolution records
// `start` when it begins executing and the last one `stop` when it ends
// (kernel execution time, without the dispatch gap before it).
hipError_t conv3x3(bool bf16, const GemmArgs &a, hipStream_t s, hipEvent_t start = nullptr,
                   hipEvent_t stop = nullptr);
hipError_t deconv(bool bf16, const GemmArgs &a, hipStream_t s);
// The convolution of a plan with ConvPlan::slices, below its halo_maps: the K
// slices of a tile side by side in one block, summed there (no ws).  Needs
// wfrag and n_cu, and splits = conv_slices_of(Ci * element size).
hipError_t conv_slices(bool bf16, const GemmArgs &a, hipStream_t s, hipEvent_t start = nullptr,
                       hipEvent_t stop = nullptr);
// Bt [N][9 Ci] (N a multiple of 16) to the order conv_slices reads; as large.
hipError_t conv_frag(bool bf16, const void *wt, void *out, int32_t N, int32_t Ci, hipStream_t s);

// The upsamplings of several stages into their channels of the slot, one
// launch over the stages and over `batch` maps (upsample.hip).
struct UpsampleStage {
    const void *wfrag;   // upsample_frag of the stage's weights
    const float *bias;   // [Co]
    int32_t Hi, Wi, Ci;  // input map
    int32_t u, c_off;    // kernel = stride; first output channel in the slot
    int32_t per, blocks, run; // set by upsample: groups per block, blocks per map, blocks per XCD
};
struct UpsampleArgs {
    UpsampleStage stage[4];
    const void *in[4][16];  // per stage and map
    void *out[16];          // per map [Ho][Wo][ldo]
    int32_t n_stages, batch, Ho, Wo, Co, ldo;
};
// Whether upsample runs a stage of this shape (else: deconv).
inline bool upsample_fits(bool bf16, int Ci, int Co) {
    return bf16 && (Ci == 64 || Ci == 128 || Ci == 256) && Co % 128 == 0;
}
hipError_t upsample(UpsampleArgs a, hipStream_t s);
// u * u phases of Bt [Co][Ci] to the order upsample reads; as large.
hipError_t upsample_frag(const void *wt, void *out, int32_t u, int32_t Co, int32_t Ci, hipStream_t s);

// ------------------------------------------------------------ post-join
struct WarpArgs {
    const void *slots[16];  // per agent [H2*W2][C]
    float affine[16][6];    // per agent {M00, M01, t0, M10, M11, t1}
    void *fused;            // [H2*W2][C]
    int32_t K, H2, W2, C;
    uint32_t ident;         // bit k: agent k's affine is exactly the identity
};
// Bit k set iff affine[k] is {1, 0, 0, 0, 1, 0} (by value).
inline uint32_t identity_mask(const float (*affine)[6], int K) {
    uint32_t m = 0;
    for (int k = 0; k < K; ++k)
        if (affine[k][0] == 1.f && affine[k][1] == 0.f && affine[k][2] == 0.f && affine[k][3] == 0.f &&
            affine[k][4] == 1.f && affine[k][5] == 0.f)
            m |= 1u << k;
    return m;
}
// With start / stop events the launch records them around the kernel's own
// execution (hipExtLaunchKernelGGL).
hipError_t warp_fuse(bool bf16, bool attn, const WarpArgs &a, hipStream_t s, hipEvent_t start = nullptr,
                     hipEvent_t stop = nullptr);

// Warp as the last node of a branch: one agent's slot resampled on the ego
// grid (the sampling of warp_fuse) and stored in the activation dtype.
struct WarpSlotArgs {
    const void *slot;  // [H2*W2][C]
    float affine[6];   // {M00, M01, t0, M10, M11, t1}
    void *out;         // [H2*W2][C]
    int32_t H2, W2, C;
};
hipError_t warp_slot(bool bf16, const WarpSlotArgs &a, hipStream_t s, hipEvent_t start = nullptr,
                     hipEvent_t stop = nullptr);

// Fusion (the fold of warp_fuse) of K stored ego-frame maps.
struct FuseArgs {
    const void *maps[16];  // per agent [cells][C]
    void *fused;           // [cells][C]
    int32_t K, cells, C;
};
hipError_t fuse(bool bf16, bool attn, const FuseArgs &a, hipStream_t s, hipEvent_t start = nullptr,
                hipEvent_t stop = nullptr);

// 1x1 head: out[m][16] float32 = bias + Bt[16][C] . in[m][C].  counts[w]
// (w < ceil(M / 16)) = anchors of pixels 16 w .. 16 w + 15 whose class
// logit (output 0 or 8) is > thr: the decode's compaction offsets.
hipError_t head1x1(bool bf16, const void *in, const void *wt, const float *bias, float *out,
                   int32_t M, int32_t C, float thr, int32_t *counts, hipStream_t s);

// Threshold and decode: anchors of [M][16] head outputs (2 anchors x 8).
struct DecodeArgs {
    const float *head;
    int32_t H2, W2;
    float thr;
    float x0, y0, dx, dy;
    float aw, al, ah, az, ayaw0, ayaw1;
    const int32_t *head_counts;  // [ceil(H2 W2 / 16)] from head1x1 with the same thr; 16-byte aligned
    float *rec;            // [n_anchors][9]: box 7, score, index bits
    uint32_t *key;         // [n_anchors] or NULL: nms_key of every record's score
    int32_t *count;        // total kept
};
constexpr int kDecodeTile = 1024;
hipError_t decode(const DecodeArgs &a, hipStream_t s);
// The result of a frame without NMS into pinned host memory: word 0 of `host`
// the count (word 1: 0; with NMS, word 0 the decoded and word 1 the kept
// count), and from byte 64 the first min(*count, first) 36-byte records of
// `recs`; written with vector stores and fenced at system scope; then 1 is
// stored to word 2 with release semantics at system scope, so a host that
// cleared word 2 before enqueuing the kernel and then reads 1 there (acquire)
// also sees the counts and records, without waiting for the stream.
hipError_t export_results(const int32_t *count, const float *recs, int first, void *host, hipStream_t s);

// Rotated NMS of the decoded records (see nms.hip).
constexpr int kNmsMaxCandidates = 16384;
constexpr int kNmsFootDoubles = 8;  // per candidate: x, y, w, l, cos yaw, sin yaw, valid (0, 1, 2), circumradius
// Ranking key of a score: its order-preserving image.  Flips the sign bit of
// a non-negative float and every bit of a negative one, which orders all
// finite and infinite values like the numbers (-0 is taken as +0); a NaN, and
// nothing else, maps to 0.
__device__ inline uint32_t nms_key(float score) {
    const uint32_t bits = score == 0.f ? 0u : __float_as_uint(score);
    return score != score ? 0u : (bits >> 31) ? ~bits : (bits | 0x80000000u);
}
struct NmsArgs {
    const float *rec;             // [n][9] decoded records, ascending anchor index
    const int32_t *count;         // n, on the device
    const uint32_t *key;          // [n] nms_key of every score
    int32_t *order;               // [max_candidates]
    double *foot;                 // [max_candidates][kNmsFootDoubles]
    unsigned long long *mask_t;   // [max_candidates]: earlier rows of its own 64-row chunk that suppress it
    int32_t *colrows;             // [nms_listed]: rows listed per column chunk
    unsigned long long *colwords; // [nms_listed]: their words, bit b: the row suppresses candidate b of the chunk
    int32_t *colcount;            // [ceil(max_candidates / 64)] rows listed per column chunk
    float *out;                   // [max_candidates][9] kept records, ascending anchor index
    int32_t *out_count;           // kept, on the device
    double iou_threshold;         // suppress iff IoU > threshold
    int32_t max_candidates;       // 1 .. kNmsMaxCandidates
    int32_t *bad_score = nullptr; // optional: set to 1 if a score is NaN (the caller clears it)
    // Optional: the frame's result into pinned host memory, as export_results
    // writes it (counts n and kept, the first host_first kept records, flag).
    uint32_t *host = nullptr;
    int32_t host_first = 0;
};
// Keys of n caller-provided records; count[0] = n, count[1] = count[2] = 0.
hipError_t nms_keys(const float *rec, int32_t n, uint32_t *key, int32_t *count, hipStream_t s);
// max_records bounds n (the grid of the per-record kernels).
hipError_t rotated_nms(const NmsArgs &a, int64_t max_records, hipStream_t s);
// Elements of NmsArgs::colrows and colwords for a candidate cap.
constexpr size_t nms_listed(int32_t max_candidates) {
    const size_t w = size_t(max_candidates + 63) / 64;
    return 64 * w * (w > 0 ? w - 1 : 0) / 2 + 1;
}

}  // namespace kern
}  // namespace rtcc
