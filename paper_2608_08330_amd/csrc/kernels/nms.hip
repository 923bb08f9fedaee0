// Rotated non-maximum suppression on bird's-eye-view boxes, after decoding
// (part of the detection post-processing that ends T^det, Sec. V-A3).
//
// Input: the decoded records rec[n][9] (x, y, z, w, l, h, yaw, score,
// anchor index bits) in ascending anchor index, n = *count on the device.
//   k_nms_keys     (caller-provided records only; in the join the decode
//                  writes the keys) one 32-bit key per record, an
//                  order-preserving image of its score.
//   k_nms_rank     rank of every record: records with a higher key, plus
//                  records with the same key and a lower index (= a lower
//                  anchor index, the records being in anchor order); the
//                  ranks are a permutation, so the order is unique.  One
//                  block per 64 records, its wavefronts sharing the keys; the
//                  first m = min(n, max_candidates) records by rank go to
//                  their place at once: order[rank] = record, footprint (x,
//                  y, w, l, cos yaw, sin yaw, valid, circumradius) as f64.
//   k_nms_mask     whether candidate a suppresses candidate b > a (BEV IoU
//                  above the threshold), one block per 64 x 64 tile: the
//                  pairs whose circumcircles meet are listed in LDS and the
//                  list is evaluated by four lanes per pair.  The words of
//                  rows that suppress something in a later chunk are listed
//                  per column chunk.  IoU in float64: the intersection area
//                  is the shoelace sum over the edge pieces of each rectangle
//                  inside the other (Cyrus-Beck clipped, crossing points
//                  shared by the two pieces that meet there); pairs whose
//                  centres are farther apart than the sum of their
//                  circumradii are disjoint and skip the clipping.  A box
//                  with a non-finite parameter or w <= 0 or l <= 0 overlaps
//                  nothing.
//   k_nms_select   the greedy selection as the fixed point of "kept = no kept
//                  suppressor ranked before", a window of 64-row chunks at
//                  once: a chunk takes the rows removed by the listed words of
//                  kept rows and resolves itself; the window moves behind the
//                  first chunk that a round changes.
//                  The kept records are then compacted in ascending record
//                  (anchor) order and, at the end of a join, also written to
//                  the host.
// Everything is integer or float64 except the scores, which are compared as
// stored: the decisions do not depend on the grid or the timing.
#include "kernels.hpp"

#include <cmath>

namespace rtcc {
namespace kern {

namespace {

constexpr int kRecFloats = 9;
constexpr int kFoot = kNmsFootDoubles;  // x, y, w, l, cos, sin, valid, circumradius
// "valid" is 0 (overlaps nothing), 1, or 2 for a footprint that the float32
// evaluation of the IoU is trusted with (see kFilter).
constexpr double kValid = 1.0, kPlain = 2.0;
constexpr double kPlainAspect = 64.0, kPlainSide = 1048576.0;

// The keys of caller-provided records and the call's counters: count[0] = n,
// count[1] = kept = 0, count[2] = the NaN-score flag = 0.
__global__ __launch_bounds__(256) void k_nms_keys(const float *rec, int32_t n, uint32_t *key, int32_t *count) {
    if (blockIdx.x == 0 && threadIdx.x < 3) count[threadIdx.x] = threadIdx.x == 0 ? n : 0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256)
        key[i] = nms_key(rec[size_t(i) * kRecFloats + 7]);
}

// Keys key[b .. e) that are above k (OREQ: or equal).  b and e are uniform
// over the wavefront, so the keys come through the scalar cache, 64 in
// flight, and a comparison is two vector instructions.
template <bool OREQ, int N>
__device__ inline int count_run(const uint32_t *__restrict__ key, uint32_t k) {
    int r = 0;
#pragma unroll
    for (int q = 0; q < N; ++q) r += OREQ ? key[q] >= k : key[q] > k;
    return r;
}
template <bool OREQ>
__device__ inline int count_before(const uint32_t *__restrict__ key, int b, int e, uint32_t k) {
    int r = 0, j = b;
    for (; j + 64 <= e; j += 64) r += count_run<OREQ, 64>(key + j, k);
    for (; j + 16 <= e; j += 16) r += count_run<OREQ, 16>(key + j, k);
    for (; j < e; ++j) r += OREQ ? key[j] >= k : key[j] > k;
    return r;
}

constexpr int kRankWaves = 7;

// Footprint of record i: x, y, w, l, cos yaw, sin yaw, valid, circumradius.
__device__ inline void footprint(const NmsArgs &a, int i, double (&f)[kFoot]) {
    const float *p = a.rec + size_t(i) * kRecFloats;
    const double x = p[0], y = p[1], w = p[3], l = p[4], yaw = p[6];
    const bool ok = isfinite(x) && isfinite(y) && isfinite(w) && isfinite(l) && isfinite(yaw) && w > 0.0 && l > 0.0;
    f[0] = x;
    f[1] = y;
    f[2] = w;
    f[3] = l;
    f[4] = ok ? cos(yaw) : 1.0;
    f[5] = ok ? sin(yaw) : 0.0;
    const double lo = w < l ? w : l, hi = w < l ? l : w;
    const bool plain = hi <= kPlainAspect * lo && hi <= kPlainSide && lo >= 1.0 / kPlainSide;
    f[6] = !ok ? 0.0 : plain ? kPlain : kValid;
    f[7] = ok ? 0.5 * sqrt(w * w + l * l) : 0.0;
}

// One block per 64 records (lane = record): wavefronts 0 .. 6 count, each over
// its share of the keys, while the last one works out the footprints; it then
// adds the counts and stores the candidates.  Bound by the comparisons, O(n^2)
// (9e8 at 30,000 records), and below some thousand records by latency.  30,000
// records 80 us, 1,400 7.9 us; as 64-bit keys in LDS, one block per 256
// records, with a second kernel for the sums and footprints, 457 and 31 us.
__global__ __launch_bounds__(64 * (kRankWaves + 1)) void k_nms_rank(NmsArgs a, const uint32_t *__restrict__ key) {
    __shared__ int part[kRankWaves][64];
    if (blockIdx.x == 0)  // the mask kernel counts the listed rows per column chunk from zero
        for (int c = threadIdx.x; c < (a.max_candidates + 63) / 64; c += blockDim.x) a.colcount[c] = 0;
    const int n = *a.count;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per = ((n + kRankWaves - 1) / kRankWaves + 15) & ~15;
    const int k0 = wave * per, k1 = k0 + per < n ? k0 + per : n;
    for (int i0 = int(blockIdx.x) * 64; i0 < n; i0 += int(gridDim.x) * 64) {  // uniform over the block
        const int i = i0 + lane;
        double f[kFoot];
        if (wave < kRankWaves) {
            const uint32_t ki = i < n ? key[i] : 0xffffffffu;
            // keys before the tile win ties, keys after it lose them
            int r = count_before<true>(key, k0, k1 < i0 ? k1 : i0, ki);
            const int m0 = k0 > i0 ? k0 : i0, m1 = k1 < i0 + 64 ? k1 : i0 + 64;
            for (int j = m0; j < m1; ++j) {
                const uint32_t kj = key[j];
                r += kj > ki || (kj == ki && j < i);
            }
            r += count_before<false>(key, k0 > i0 + 64 ? k0 : i0 + 64, k1, ki);
            part[wave][lane] = r;
        } else if (i < n) {
            footprint(a, i, f);
            if (a.bad_score && key[i] == 0u) *a.bad_score = 1;
        }
        __syncthreads();
        if (wave == kRankWaves && i < n) {
            int r = 0;
#pragma unroll
            for (int v = 0; v < kRankWaves; ++v) r += part[v][lane];
            if (r < a.max_candidates) {
                a.order[r] = i;
#pragma unroll
                for (int q = 0; q < kFoot; ++q) a.foot[size_t(r) * kFoot + q] = f[q];
            }
        }
        __syncthreads();  // part is reused
    }
}

struct Foot {
    double x, y, w, l, c, s, rad;
    bool ok;
};

__device__ inline Foot load_foot(const double *f) {
    return Foot{f[0], f[1], f[2], f[3], f[4], f[5], f[7], f[6] != 0.0};
}

// corners counter-clockwise: (+l/2, +w/2), (-l/2, +w/2), (-l/2, -w/2),
// (+l/2, -w/2) in the box frame (l along the heading), relative to (ox, oy)
__device__ inline void foot_corners(const Foot &b, double ox, double oy, double *px, double *py) {
#pragma clang fp contract(off)
    const double hl = 0.5 * b.l, hw = 0.5 * b.w;
    const double sa[4] = {hl, -hl, -hl, hl}, sb[4] = {hw, hw, -hw, -hw};
    const double cx = b.x - ox, cy = b.y - oy;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        px[k] = cx + (sa[k] * b.c - sb[k] * b.s);
        py[k] = cy + (sa[k] * b.s + sb[k] * b.c);
    }
}

// The value x of lane K of this lane's quad.
template <int K>
__device__ inline float quad_lane(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), K * 0x55, 0xf, 0xf, false));
}
template <int K>
__device__ inline double quad_lane(double x) {
    const uint2 u = __builtin_bit_cast(uint2, x);
    return __builtin_bit_cast(double, make_uint2(__builtin_amdgcn_update_dpp(0u, u.x, K * 0x55, 0xf, 0xf, false),
                                                 __builtin_amdgcn_update_dpp(0u, u.y, K * 0x55, 0xf, 0xf, false)));
}
// The value x of the next lane of this lane's quad (the first one's for the last).
__device__ inline float quad_next(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x39, 0xf, 0xf, false));
}
__device__ __forceinline__ double pick(const double (&v)[4], int k) {
    const double v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];  // all read: selects, no indexing
    const double a = k & 1 ? v1 : v0, b = k & 1 ? v3 : v2;
    return k & 2 ? b : a;
}

// Twice the area of the intersection of two counter-clockwise rectangles P
// and Q.  The boundary of the intersection consists of the pieces of P's
// edges inside Q and of Q's edges inside P; its shoelace sum (Green's
// theorem) is twice the area.  Each piece is the part of an edge inside the
// other rectangle's four half-planes cross(e_j, p - q_j) >= 0 (Cyrus-Beck
// clipping; the bounds are kept as fractions and compared crosswise, one
// division per end).  Where a piece of P ends on an edge of Q, the piece of
// Q begins at the same point: both take it from P's parametrisation, so the
// boundary closes even for nearly parallel edges.  An edge of P lying on an
// edge of Q counts once, for P, if both run the same way; an edge of Q on
// an edge of P never counts.  No fused multiply-add: these collinearity
// tests need exact zeros.  Fixed trip counts: registers only.
//
// The four lanes of a quad evaluate one pair: lane e clips edge e of P and
// edge e of Q, and every lane adds the eight pieces in the same order (P's
// edges, then Q's), so all four hold the same sum.  One lane per pair made
// the clip a chain of thousands of instructions in a few busy lanes.
__device__ __forceinline__ double inter_twice(const double (&px)[4], const double (&py)[4], const double (&qx)[4],
                                              const double (&qy)[4], int e) {
#pragma clang fp contract(off)
    double pdx[4], pdy[4], qdx[4], qdy[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        pdx[k] = px[(k + 1) & 3] - px[k];
        pdy[k] = py[(k + 1) & 3] - py[k];
        qdx[k] = qx[(k + 1) & 3] - qx[k];
        qdy[k] = qy[(k + 1) & 3] - qy[k];
    }
    const double pxe = pick(px, e), pye = pick(py, e), pdxe = pick(pdx, e), pdye = pick(pdy, e);
    const double qxe = pick(qx, e), qye = pick(qy, e), qdxe = pick(qdx, e), qdye = pick(qdy, e);
    double piece_p = 0.0, piece_q = 0.0;
    {
        double n0 = 0.0, d0 = 1.0, n1 = 1.0, d1 = 1.0;
        bool empty = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // P's edge against Q's edge line j
            const double al = qdx[j] * (pye - qy[j]) - qdy[j] * (pxe - qx[j]);
            const double be = qdx[j] * pdye - qdy[j] * pdxe;
            if (be > 0.0) {
                if (-al * d0 > n0 * be) {
                    n0 = -al;
                    d0 = be;
                }
            } else if (be < 0.0) {
                if (al * d1 < n1 * -be) {
                    n1 = al;
                    d1 = -be;
                }
            } else if (al < 0.0 || (al == 0.0 && !(qdx[j] * pdxe + qdy[j] * pdye > 0.0))) {
                empty = true;
            }
        }
        const double t0 = n0 / d0, t1 = n1 / d1;
        if (!empty && t0 < t1) {
            const double x0 = pxe + t0 * pdxe, y0 = pye + t0 * pdye;
            const double x1 = pxe + t1 * pdxe, y1 = pye + t1 * pdye;
            piece_p = x0 * y1 - x1 * y0;
        }
    }
    {
        double n0 = 0.0, d0 = 1.0, n1 = 1.0, d1 = 1.0;
        bool empty = false;
        // the chosen bounds: P's edge (corner, direction) that cuts there
        double cx0 = 0.0, cy0 = 0.0, ex0 = 0.0, ey0 = 0.0, cx1 = 0.0, cy1 = 0.0, ex1 = 0.0, ey1 = 0.0;
        bool b0 = false, b1 = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // Q's edge against P's edge line i
            const double al = pdx[i] * (qye - py[i]) - pdy[i] * (qxe - px[i]);
            const double be = pdx[i] * qdye - pdy[i] * qdxe;
            if (be > 0.0) {
                if (-al * d0 > n0 * be) {
                    n0 = -al;
                    d0 = be;
                    b0 = true;
                    cx0 = px[i];
                    cy0 = py[i];
                    ex0 = pdx[i];
                    ey0 = pdy[i];
                }
            } else if (be < 0.0) {
                if (al * d1 < n1 * -be) {
                    n1 = al;
                    d1 = -be;
                    b1 = true;
                    cx1 = px[i];
                    cy1 = py[i];
                    ex1 = pdx[i];
                    ey1 = pdy[i];
                }
            } else if (al <= 0.0) {
                empty = true;
            }
        }
        if (!empty && n0 / d0 < n1 / d1) {
            double ax0 = qxe, ay0 = qye;
            double ax1 = pick(qx, (e + 1) & 3), ay1 = pick(qy, (e + 1) & 3);
            if (b0) {  // P's parametrisation of its crossing with this edge's line
                const double al = qdxe * (cy0 - qye) - qdye * (cx0 - qxe), be = qdxe * ey0 - qdye * ex0;
                const double t = -al / be;
                ax0 = cx0 + t * ex0;
                ay0 = cy0 + t * ey0;
            }
            if (b1) {
                const double al = qdxe * (cy1 - qye) - qdye * (cx1 - qxe), be = qdxe * ey1 - qdye * ex1;
                const double t = -al / be;
                ax1 = cx1 + t * ex1;
                ay1 = cy1 + t * ey1;
            }
            piece_q = ax0 * ay1 - ax1 * ay0;
        }
    }
    double twice = 0.0;
    twice += quad_lane<0>(piece_p);
    twice += quad_lane<1>(piece_p);
    twice += quad_lane<2>(piece_p);
    twice += quad_lane<3>(piece_p);
    twice += quad_lane<0>(piece_q);
    twice += quad_lane<1>(piece_q);
    twice += quad_lane<2>(piece_q);
    twice += quad_lane<3>(piece_q);
    return twice;
}

// BEV IoU of two footprints (0 if either is invalid or they are farther
// apart than the sum of their circumradii), coordinates relative to A's
// centre; evaluated by the four lanes e of a quad, which all return it.
__device__ __forceinline__ double foot_iou(const Foot &A, const Foot &B, int e) {
#pragma clang fp contract(off)
    if (!A.ok || !B.ok) return 0.0;
    const double dx = A.x - B.x, dy = A.y - B.y;
    if (dx * dx + dy * dy > (A.rad + B.rad) * (A.rad + B.rad)) return 0.0;
    double px[4], py[4], qx[4], qy[4];
    foot_corners(A, A.x, A.y, px, py);
    foot_corners(B, A.x, A.y, qx, qy);
    const double twice = inter_twice(px, py, qx, qy, e);
    const double inter = twice > 0.0 ? 0.5 * twice : 0.0;
    const double uni = A.w * A.l + B.w * B.l - inter;
    return uni > 0.0 ? inter / uni : 0.0;
}

// Whether two footprints' circumcircles meet, the comparison foot_iou makes
// before clipping: a pair for which it fails has IoU 0.
__device__ __forceinline__ bool circles_meet(double ax, double ay, double ar, double bx, double by, double br) {
#pragma clang fp contract(off)
    const double dx = ax - bx, dy = ay - by, rd = ar + br;
    return !(dx * dx + dy * dy > rd * rd);
}

// The decision IoU > threshold, taken in float64.  For two plain footprints a
// float32 evaluation decides first, where it lies more than kFilter from the
// threshold.  It does not clip edge against edge: with collinear edges (boxes
// of equal heading and width, one ahead of the other) rounded signs can count
// a stretch of border twice or not at all, whole tenths of the IoU.  It adds up, over
// the edges of B in A's frame, the integral of -clamp(y) dx over the part with
// |x| <= l / 2 (Green's theorem), which is continuous in the corners, so its
// error is bounded.  With u = 2^-24 and r the larger circumradius: a corner is
// off by at most 12 u * 2 r, which moves the area by that times a perimeter of at
// most 5.7 r, and the integrals round by less than 3 u r^2: 140 u r^2, that is 35 u
// (w^2 + l^2) of the larger footprint.  The union is at least that footprint's
// w l, and the intersection enters the quotient twice: 70 u (l / w + w / l),
// 2.7e-4 at the aspect ratio of 64 up to which a footprint is plain.  (Seen over 200,000 pairs of
// a kind: 9e-7 at 1.6 x 3.9, 4e-6 at 0.1 x 6.4, 3e-4 at 0.01 x 50.)  Products
// of two lengths stay inside the float32 range for sides from 2^-20 to 2^20.
constexpr float kFilter = 1e-3f, kTiny = 0x1p-60f;
__device__ __forceinline__ float clampf(float v, float m) { return fminf(fmaxf(v, -m), m); }
__device__ __forceinline__ float plain_iou(const double *A, const double *B, int e) {
    const float aw = float(A[2]), al = float(A[3]), ac = float(A[4]), as = float(A[5]);
    const float bw = float(B[2]), bl = float(B[3]), bc = float(B[4]), bs = float(B[5]);
    const float dx = float(B[0]) - float(A[0]), dy = float(B[1]) - float(A[1]);
    const float cd = bc * ac + bs * as, sd = bs * ac - bc * as;  // B's heading in A's frame
    const float sa = 0.5f * (e == 0 || e == 3 ? bl : -bl), sb = 0.5f * (e < 2 ? bw : -bw);
    // edge e of B runs from its corner e to the next lane's
    const float x0 = dx * ac + dy * as + (sa * cd - sb * sd), y0 = dy * ac - dx * as + (sa * sd + sb * cd);
    const float x1 = quad_next(x0), y1 = quad_next(y0);
    const float hl = 0.5f * al, hw = 0.5f * aw;
    // (below kTiny the integral, or its variation, is nothing next to an area)
    const float slope = fabsf(x1 - x0) > kTiny ? (y1 - y0) / (x1 - x0) : 0.f;
    const float c0 = clampf(x0, hl), c1 = clampf(x1, hl);
    const float e0 = y0 + (c0 - x0) * slope, e1 = y1 + (c1 - x1) * slope;  // the edge at c0 and c1
    const float lo = fminf(e0, e1), hi = fmaxf(e0, e1), inv = hi - lo > kTiny ? 1.f / (hi - lo) : 0.f;
    // the parts of [lo, hi] below -w / 2 and up to w / 2
    const float t1 = fminf(fmaxf((-hw - lo) * inv, 0.f), 1.f), t2 = fminf(fmaxf((hw - lo) * inv, 0.f), 1.f);
    const float mean = hi - lo > kTiny ? hw * (1.f - t2 - t1) + (t2 - t1) * 0.5f * (clampf(lo, hw) + clampf(hi, hw))
                                       : clampf(lo, hw);
    const float piece = (c0 - c1) * mean;
    const float area = quad_lane<0>(piece) + quad_lane<1>(piece) + quad_lane<2>(piece) + quad_lane<3>(piece);
    const float inter = fmaxf(area, 0.f), uni = aw * al + bw * bl - inter;
    return uni > 0.f ? inter / uni : 0.f;
}

// Column chunk c: the rows of earlier chunks that suppress something there
// are listed, with their words, from col_base(c), at most 64 c.
__host__ __device__ inline int64_t col_base(int c) { return int64_t(64) * c * (c - 1) / 2; }

// One 64 x 64 tile (row chunk rb, column chunk cb >= rb) of the suppression
// matrix, or, where the tiles are few, a quarter of its rows per block: a
// crowded tile is thousands of clips.  The pairs whose footprints'
// circumcircles meet are first compacted into an LDS list (lane = column, one
// ballot per row); the list is then evaluated in float32, four lanes per pair,
// and the pairs that float32 leaves undecided, or is not trusted with, in float64.  Lists
// the rows with a nonzero word of an off-diagonal tile, and on the diagonal
// the transposed words: for every column, the earlier rows of its own chunk
// that suppress it (a quarter writes its 16 bits of them).  90 records 6.5 us,
// 1,400 12.0, 4,096 candidates 40; one lane per pair, whole tiles, and the
// words of a full matrix: 13.3, 19.2 and 119 us.  Quarters for every size
// would take 17 and 86 us at 1,400 and 4,096 (the footprints are staged four
// times), whole tiles 30 against 18 us for a frame's 80 crowded boxes.
constexpr int kQuarterTiles = 64;  // quarters up to this many tiles (10 chunks, 640 candidates)
__global__ __launch_bounds__(256) void k_nms_mask(NmsArgs a) {
    __shared__ double fr[64 * kFoot], fc[64 * kFoot];
    __shared__ unsigned short list[64 * 64], open[64 * 64];
    __shared__ unsigned long long rowbits[64], tq[64];
    __shared__ int nlist, nopen;
    const int n = *a.count;
    const int m = n < a.max_candidates ? n : a.max_candidates;
    const int T = (m + 63) / 64, tiles = T * (T + 1) / 2;
    const int parts = tiles <= kQuarterTiles ? 4 : 1, rows = 64 / parts;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int item = blockIdx.x; item < tiles * parts; item += gridDim.x) {  // uniform over the block
        const int part = item % parts;
        int tri = item / parts, rb = 0;
        while (tri >= T - rb) {
            tri -= T - rb;
            ++rb;
        }
        const int cb = rb + tri;
        const int r0 = rb * 64 + part * rows, c0 = cb * 64;
        for (int q = tid; q < 64 * kFoot; q += 256) {
            const int k = q / kFoot;
            fc[q] = c0 + k < m ? a.foot[size_t(c0) * kFoot + q] : 0.0;
            if (k < rows) fr[q] = r0 + k < m ? a.foot[size_t(r0) * kFoot + q] : 0.0;
        }
        if (tid < 64) {
            rowbits[tid] = 0ull;
            tq[tid] = 0ull;
        }
        if (tid == 0) nlist = nopen = 0;
        __syncthreads();
        // close pairs (row i, column j), j > i on the diagonal tile (a
        // footprint past the last candidate is not valid); four rows of a
        // wavefront at a time
        const double *B = fc + lane * kFoot;
        const double bx = B[0], by = B[1], brad = B[7];
        const bool bok = B[6] != 0.0;
        for (int i0 = wave * 4; i0 < rows; i0 += 16) {
            unsigned long long bal[4];
            int cnt = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double *A = fr + (i0 + u) * kFoot;
                bal[u] = __ballot(bok && A[6] != 0.0 && (cb > rb || lane > part * rows + i0 + u) &&
                                  circles_meet(A[0], A[1], A[7], bx, by, brad));
                cnt += __popcll(bal[u]);
            }
            if (cnt == 0) continue;
            int at = 0;
            if (lane == 0) at = atomicAdd(&nlist, cnt);
            at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if ((bal[u] >> lane) & 1ull)
                    list[at + __popcll(bal[u] & ((1ull << lane) - 1ull))] =
                        static_cast<unsigned short>(((i0 + u) << 6) | lane);
                at += __popcll(bal[u]);
            }
        }
        __syncthreads();
        const int e = tid & 3;
        auto suppress = [&](int i, int j) {
            atomicOr(&rowbits[i], 1ull << j);
            if (cb == rb) atomicOr(&tq[j], 1ull << i);
        };
        for (int q = tid >> 2; q < nlist; q += 64) {
            const int p = list[q], i = p >> 6, j = p & 63;
            const float thr = float(a.iou_threshold);
            float v = thr;  // undecided
            if (fr[i * kFoot + 6] == kPlain && fc[j * kFoot + 6] == kPlain)
                v = plain_iou(fr + i * kFoot, fc + j * kFoot, e);
            if (e != 0) continue;
            if (v > thr + kFilter) suppress(i, j);
            else if (!(v < thr - kFilter)) open[atomicAdd(&nopen, 1)] = static_cast<unsigned short>(p);
        }
        __syncthreads();
        for (int q = tid >> 2; q < nopen; q += 64) {
            const int p = open[q], i = p >> 6, j = p & 63;
            const double v = foot_iou(load_foot(fr + i * kFoot), load_foot(fc + j * kFoot), e);
            if (e == 0 && v > a.iou_threshold) suppress(i, j);
        }
        __syncthreads();
        if (cb != rb) {
            if (tid < rows && rowbits[tid]) {
                const int64_t at = col_base(cb) + atomicAdd(&a.colcount[cb], 1);
                a.colrows[at] = r0 + tid;
                a.colwords[at] = rowbits[tid];
            }
        } else if (tid < 64 && c0 + tid < m) {
            if (parts == 1) a.mask_t[c0 + tid] = tq[tid];
            else reinterpret_cast<unsigned short *>(a.mask_t + c0 + tid)[part] = static_cast<unsigned short>(tq[tid]);
        }
        __syncthreads();  // the tile's LDS is reused by the next item
    }
}

__device__ inline unsigned long long uniform64(unsigned long long v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(v >> 32));
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// OR over the 64 lanes of a wavefront (DPP row shifts, then row
// broadcasts; lane 63 holds the total), returned to every lane.
__device__ inline uint32_t wave_or32(uint32_t v) {
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v |= __builtin_amdgcn_update_dpp(0u, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ inline unsigned long long wave_or64(unsigned long long v) {
    return (static_cast<unsigned long long>(wave_or32(uint32_t(v >> 32))) << 32) | wave_or32(uint32_t(v));
}

// The same resolution in parallel: lane r holds `sup`, the earlier rows of
// the chunk that suppress row r.  kept = standing rows none of whose kept
// suppressors exist, iterated from kept = standing: after t rounds rows
// 0 .. t-1 are final, so the iteration stops at the unique fixed point
// within 65 rounds (usually a few).
__device__ inline unsigned long long resolve_chunk_parallel(unsigned long long rem, unsigned long long sup, int rows) {
    const unsigned long long rowmask = rows >= 64 ? ~0ull : (1ull << rows) - 1ull;
    const int lane = threadIdx.x & 63;
    const unsigned long long standing = ~uniform64(rem) & rowmask;
    unsigned long long kept = standing;
    for (int it = 0; it <= 64; ++it) {
        const bool mine = ((standing >> lane) & 1ull) && !(kept & sup);
        const unsigned long long next = __ballot(mine);
        if (next == kept) break;
        kept = next;
    }
    return kept;
}

constexpr int kSelectThreads = 1024;
constexpr int kSelectWaves = kSelectThreads / 64;
constexpr int kMaxChunks = kNmsMaxCandidates / 64;
constexpr int kSelCap = 8192;    // listed words held in LDS
constexpr int kSupLds = 4096;    // candidates whose in-chunk suppressors are held in LDS
constexpr int kWindow = 32;      // chunks in work at a time, two per wavefront
constexpr int kFlagBits = 131072;  // records compacted per pass

// Exclusive scan of one int per thread over the block; *total to everyone.
__device__ inline int select_scan(int v, int *wsum, int *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(inc, d, 64);
        if (lane >= d) inc += t;
    }
    __syncthreads();  // wsum's last use is over
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < kSelectWaves; ++q) {
        if (q < wave) base += wsum[q];
        tot += wsum[q];
    }
    *total = tot;
    return base + inc - v;
}

// The greedy selection: kept(q) = no kept(p) with p ranked before q that
// suppresses it.  A window of chunks of 64 rows iterates at once, a wavefront
// per chunk: the rows removed from outside are the OR of the words listed for
// the chunk whose row is kept in the current estimate, and the chunk then
// resolves itself exactly (resolve_chunk_parallel), in place.  A round in
// which chunk l is the first to change has read only unchanged words for every
// chunk up to l, which therefore are final, whichever of the other chunks'
// words a wavefront saw: the window moves on behind l, or, after a round that
// changes nothing, behind its end.  Every round moves it, so there are at most
// as many rounds as chunks, of two chunks per wavefront; scenes take a few per
// window.  A chunk that its suppressors leave as they did is not resolved
// again.  A walk over the chunks in order paid the same latency once per
// chunk; all chunks in every round are up to T^2 / 16 resolutions in a row.  The
// call, us, walk -> all chunks -> window:
//   a chain of boxes, each decided by the one before
//                     1,500 212 -> 261 -> 177   4,096 430 -> 1,286 -> 376   16,384 2,104 -> 17,408 -> 1,564
//   crowded           1,500 224 -> 108 -> 106   4,096 546 -> 182 -> 162     16,384 4,481 -> 1,304 -> 795
// (the last with the mask kernel's changes).  Windows of 16 and 64 chunks: 349
// and 398 for the chain of 4,096, 170 and 172 for the crowd.
// The listed words are copied into LDS when they fit, else read where they
// are.  The kept records are then compacted in ascending record order.
// 1,400 records 16.6 us, 4,096 candidates of 30,000 crowded ones 45 us; as a
// walk, with the kept records found by a scan over all records: 32.6 and 221.
__global__ __launch_bounds__(kSelectThreads) void k_nms_select(NmsArgs a) {
    __shared__ unsigned long long keep[kMaxChunks], removed[kMaxChunks];
    __shared__ __attribute__((aligned(16))) unsigned long long eword[kSelCap];
    __shared__ unsigned short erow[kSelCap];
    __shared__ int coff[kMaxChunks + 1];
    __shared__ unsigned long long supl[kSupLds];
    __shared__ uint32_t fbits[kFlagBits / 32];
    __shared__ int wsum[kSelectWaves];
    __shared__ int lowest[3];  // per round, the first chunk that changed
    static_assert(kSelCap * 8 >= kNmsMaxCandidates * 4, "the kept list reuses the words' LDS");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = *a.count;
    const int m = n < a.max_candidates ? n : a.max_candidates;
    const int T = (m + 63) / 64;
    int listed;
    const int off = select_scan(tid < T ? a.colcount[tid] : 0, wsum, &listed);
    if (tid <= T) coff[tid] = off;
    const bool fits = listed <= kSelCap;
    const bool sup_lds = m <= kSupLds;
    if (sup_lds)
        for (int q = tid; q < m; q += kSelectThreads) supl[q] = a.mask_t[q];
    for (int c = tid; c < T; c += kSelectThreads) keep[c] = ~0ull;
    if (tid == 0) lowest[0] = T;
    __syncthreads();
    if (fits)
        for (int c = wave; c < T; c += kSelectWaves)
            for (int k = lane; k < coff[c + 1] - coff[c]; k += 64) {
                erow[coff[c] + k] = static_cast<unsigned short>(a.colrows[col_base(c) + k]);
                eword[coff[c] + k] = a.colwords[col_base(c) + k];
            }
    __syncthreads();
    // the first two chunks of a wavefront keep their suppressors and up to
    // 128 listed words in registers
    constexpr int RC = 2, RE = 2;
    unsigned long long rsup[RC], rword[RC][RE];
    int rrow[RC][RE], rlen[RC];
#pragma unroll
    for (int g = 0; g < RC; ++g) {
        const int c = wave + g * kSelectWaves;
        rlen[g] = c < T ? coff[c + 1] - coff[c] : 0;
        const int row = c * 64 + lane;
        rsup[g] = c < T && row < m ? (sup_lds ? supl[row] : a.mask_t[row]) : 0ull;
#pragma unroll
        for (int x = 0; x < RE; ++x) {
            const int k = lane + 64 * x;
            rrow[g][x] = 0;
            rword[g][x] = 0ull;
            if (k < rlen[g]) {
                rrow[g][x] = fits ? int(erow[coff[c] + k]) : a.colrows[col_base(c) + k];
                rword[g][x] = fits ? eword[coff[c] + k] : a.colwords[col_base(c) + k];
            }
        }
    }
    auto kept_row = [&](int r) { return (__hip_atomic_load(&keep[r >> 6], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >> (r & 63)) & 1ull; };
    int first = 0, reached = 0;  // the first chunk not final, and not yet in work
    for (int it = 0; first < T; ++it) {
        const int end = first + kWindow < T ? first + kWindow : T;
        int low = T;  // the first chunk of this wavefront that changed
        auto settle = [&](int c, unsigned long long rem, unsigned long long sup) {
            rem = wave_or64(rem);
            if (c < reached && rem == removed[c]) return;
            if (lane == 0) removed[c] = rem;
            const unsigned long long kb = resolve_chunk_parallel(rem, sup, m - c * 64 < 64 ? m - c * 64 : 64);
            if (kb != keep[c] && c < low) low = c;
            if (lane == 0) __hip_atomic_store(&keep[c], kb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        auto listed_from = [&](int c, int k) {
            unsigned long long rem = 0ull;
            for (; k < coff[c + 1] - coff[c]; k += 64) {
                const int r = fits ? int(erow[coff[c] + k]) : a.colrows[col_base(c) + k];
                const unsigned long long w = fits ? eword[coff[c] + k] : a.colwords[col_base(c) + k];
                if (kept_row(r)) rem |= w;
            }
            return rem;
        };
#pragma unroll
        for (int g = 0; g < RC; ++g) {
            const int c = wave + g * kSelectWaves;
            if (c < first || c >= end) continue;
            unsigned long long rem = 0ull;
#pragma unroll
            for (int x = 0; x < RE; ++x)
                if (kept_row(rrow[g][x])) rem |= rword[g][x];
            if (rlen[g] > 64 * RE) rem |= listed_from(c, lane + 64 * RE);
            settle(c, rem, rsup[g]);
        }
        // this wavefront's other chunks of the window
        const int skip = first - wave > 0 ? (first - wave + kSelectWaves - 1) / kSelectWaves : 0;
        for (int c = wave + (skip > RC ? skip : RC) * kSelectWaves; c < end; c += kSelectWaves) {
            const int row = c * 64 + lane;
            settle(c, listed_from(c, lane), row < m ? (sup_lds ? supl[row] : a.mask_t[row]) : 0ull);
        }
        if (lane == 0 && low < T) atomicMin(&lowest[it % 3], low);
        if (tid == 0) lowest[(it + 1) % 3] = T;  // last read two rounds ago
        __syncthreads();
        const int l = lowest[it % 3];
        first = l < T ? l + 1 : end;
        reached = end;
    }
    // kept candidates -> their records, ascending: a bitmap of the records
    // per pass, its set bits numbered by a scan
    uint32_t *kept = reinterpret_cast<uint32_t *>(eword);
    int found = 0;
    for (int s0 = 0; s0 < n; s0 += kFlagBits) {
        const int words = (n - s0 < kFlagBits ? n - s0 + 31 : kFlagBits) / 32;
        for (int w = tid; w < words; w += kSelectThreads) fbits[w] = 0u;
        __syncthreads();
        for (int q = tid; q < m; q += kSelectThreads) {
            if (!((keep[q >> 6] >> (q & 63)) & 1ull)) continue;
            const int i = a.order[q] - s0;
            if (unsigned(i) < unsigned(kFlagBits)) atomicOr(&fbits[i >> 5], 1u << (i & 31));
        }
        __syncthreads();
        const int per = (words + kSelectThreads - 1) / kSelectThreads;
        int c = 0;
        for (int w = tid * per; w < tid * per + per && w < words; ++w) c += __popc(fbits[w]);
        int tot;
        int at = found + select_scan(c, wsum, &tot);
        for (int w = tid * per; w < tid * per + per && w < words; ++w)
            for (uint32_t b = fbits[w]; b; b &= b - 1u) kept[at++] = uint32_t(s0 + w * 32 + __ffs(b) - 1);
        found += tot;
        __syncthreads();
    }
    // the records, four words per thread: to the output, and at the end of a
    // join the first ones to the host (16-byte stores across the bus)
    const int words = found * kRecFloats;
    const int hrec = a.host ? (found < a.host_first ? found : a.host_first) : 0;
    const uint32_t *src = reinterpret_cast<const uint32_t *>(a.rec);
    uint32_t *dst = reinterpret_cast<uint32_t *>(a.out);
    for (int v = tid * 4; v < words; v += kSelectThreads * 4) {
        uint32_t x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int p = (v + q) / kRecFloats;
            if (v + q < words) x[q] = src[size_t(kept[p]) * kRecFloats + (v + q - p * kRecFloats)];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (v + q < words) dst[v + q] = x[q];
        if (v + 4 <= hrec * kRecFloats) *reinterpret_cast<uint4 *>(a.host + 16 + v) = make_uint4(x[0], x[1], x[2], x[3]);
        else
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (v + q < hrec * kRecFloats) a.host[16 + v + q] = x[q];
    }
    if (tid == 0) *a.out_count = found;
    if (!a.host) return;
    if (tid == 0) {
        a.host[0] = uint32_t(n);
        a.host[1] = uint32_t(found);
    }
    __threadfence_system();
    __syncthreads();  // every thread's stores are fenced before the flag
    if (tid == 0) __hip_atomic_store(&a.host[2], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace

hipError_t nms_keys(const float *rec, int32_t n, uint32_t *key, int32_t *count, hipStream_t s) {
    const unsigned blocks = unsigned((int64_t(n) + 255) / 256);
    k_nms_keys<<<blocks < 1024u ? blocks : 1024u, 256, 0, s>>>(rec, n, key, count);
    return hipGetLastError();
}

hipError_t rotated_nms(const NmsArgs &a, int64_t max_records, hipStream_t s) {
    if (a.max_candidates < 1 || a.max_candidates > kNmsMaxCandidates || max_records < 1)
        return hipErrorInvalidValue;
    // grids are bounded by the worst case and loop over the work of the
    // actual count read on the device; two blocks per CU fill the chip
    const int64_t blocks = (max_records + 63) / 64;
    k_nms_rank<<<unsigned(blocks < 512 ? blocks : 512), 64 * (kRankWaves + 1), 0, s>>>(a, a.key);
    const int64_t m = max_records < a.max_candidates ? max_records : a.max_candidates;
    const int64_t chunks = (m + 63) / 64, tiles = chunks * (chunks + 1) / 2;
    const int64_t items = tiles <= kQuarterTiles ? 4 * tiles : tiles < 4 * kQuarterTiles ? 4 * kQuarterTiles : tiles;
    k_nms_mask<<<unsigned(items < 1024 ? items : 1024), 256, 0, s>>>(a);
    k_nms_select<<<1, kSelectThreads, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace kern
}  // namespace rtcc
