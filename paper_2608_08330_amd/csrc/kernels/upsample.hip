// The transposed-conv upsamplings (kernel = stride = u) of a map's stages
// into its slot, all of them in one launch (bf16, 64 / 128 / 256 input
// channels, 128 k output channels; other shapes take the implicit GEMM).
//
// GEMM view: M = input pixels, K = C_in, and one group of 128 output channels
// per phase (py, px) of the u x u kernel.  A block owns 64 input pixels and
// st.per consecutive groups.  It stages its pixels, all channels, in LDS with
// one burst and one barrier; each wavefront computes 64 pixels x 32 P channels
// of every group, weights loaded straight into registers part of a group ahead
// from a fragment-ordered copy (upsample_frag).  In that copy a fragment
// pair's channels are interleaved so that a lane ends with 8 consecutive
// channels of a pixel: it stores 16 bytes, and no output goes through LDS.
//
// P = 1: four wavefronts per block, for the shortest chain; each stores 64
// consecutive bytes per pixel.  P = 2: two wavefronts, and lanes trade halves
// so that each stores whole lines of 128 bytes: non-temporal stores of half a
// line reach 2.9 TB/s, of a line 4.9 (403 MB).  Stores through the L2 reach
// 4.8 either way but push out what the other streams of a frame keep there.
//
// What bounds it: at 8 maps of 256 x 256 pixels (128 / 256 / 256 channels) the
// bytes, 403 MB written and 218 MB read, 124 us at the rate of a large copy;
// on small maps, latency and launches.  The implicit GEMM it replaces
// (launches of their own, an LDS ring with a barrier per 32 channels, the
// tile stored through LDS) is limited by LDS traffic at u > 1.  us, before ->
// now, all three stages:
//   one map   50 x 176 20.1 -> 6.2   22 x 30 18.5 -> 4.6   256 x 256 35 -> 24
//   batches   6 x (50 x 176) 30 -> 20   3 x (128 x 128) 29.5 -> 17.6
//             8 x (256 x 256) 190 -> 153 (P = 1: 160; stores through the L2 200);
//             in a frame, maps cold and other streams busy, 229 -> 181 (210; 188)
// The steps are fenced for the scheduler: left alone it hoists every LDS read
// and weight load (P = 1: 248 instead of 146 registers, two instead of three
// blocks per CU; 8 x (256 x 256) 177 against 162 us with per = 4).
// The K order is that of the implicit GEMM: the same bits.
#include "kernels.hpp"

#include "mfma.hpp"

namespace rtcc {
namespace kern {

namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kPx = 64, kFM = kPx / 16;

__device__ inline unsigned swap_halves(unsigned v) {  // lanes l and l ^ 8 trade
    return unsigned(__builtin_amdgcn_update_dpp(0, int(v), 0x128 /* row_ror:8 */, 0xf, 0xf, false));
}

// Groups [g0, g1) of the block's pixels; KT = C_in / 32, a wavefront computes
// P fragment pairs of 32 channels.
template <int KT, int P>
__device__ inline void up_tile(const UpsampleArgs &a, const UpsampleStage &st, const uint16_t *in, uint16_t *out,
                               int m0, int g0, int g1, unsigned char *smem) {
    constexpr int KH = KT < 4 / P ? KT : 4 / P, NH = KT / KH;  // weights in flight: KH steps
    constexpr int NW = 4 / P, PAIR = KT * 2 * 64;
    constexpr int GROUP = 4 * KT * 2 * 64;             // vectors of a group's weights
    const uint32_t lds_base = lds_address(smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int M = st.Hi * st.Wi;
    // vector v of pixel row r of a 32-channel chunk sits at v ^ ((r >> 1) & 3)
    for (int q = wave; q < KT * kFM; q += NW) {
        const int c = q / kFM, blk = q - c * kFM;
        const int row = blk * 16 + (lane >> 2);
        const int vec = (lane & 3) ^ ((row >> 1) & 3);
        const int m = m0 + row < M ? m0 + row : M - 1;  // not stored
        load_lds16(in + size_t(m) * (KT * 32) + c * 32 + vec * 8, lds_base + (c * kPx + blk * 16) * 64);
    }
    const int fr = lane & 15, fk = lane >> 4;
    const uint4 *wf = static_cast<const uint4 *>(st.wfrag) + size_t(g0) * GROUP + wave * (P * PAIR) + lane;
    uint4 w[2][KH][P][2];
    auto load_w = [&](uint4 (&v)[KH][P][2], const uint4 *p) {
#pragma unroll
        for (int k = 0; k < KH; ++k)
#pragma unroll
            for (int j = 0; j < 2 * P; ++j) v[k][j >> 1][j & 1] = p[(j >> 1) * PAIR + (k * 2 + (j & 1)) * 64];
    };
    load_w(w[0], wf);
    // LDS offset of the lane's pixels, output position at phase (0, 0) of the
    // pixels that it stores: with two pairs 16 i + fr % 8 and 8 more
    int at[kFM], oy[kFM * P], ox[kFM * P];
#pragma unroll
    for (int i = 0; i < kFM; ++i) {
        const int r = i * 16 + fr;
        at[i] = r * 64 + ((fk ^ ((r >> 1) & 3)) << 4);
    }
#pragma unroll
    for (int i = 0; i < kFM * P; ++i) {
        const int m = m0 + i * (16 / P) + fr % (16 / P), iy = m / st.Wi;
        oy[i] = m < M ? iy * st.u : a.Ho;
        ox[i] = (m - iy * st.Wi) * st.u;
    }
    const bool upper = fr >= 8;
    const int blocks128 = a.Co >> 7;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's part of the pixels is in LDS
    __syncthreads();
    for (int g = g0; g < g1; ++g) {
        const int phase = g / blocks128, n = (g - phase * blocks128) * 128 + wave * (32 * P) + fk * 8;
        float4 b[P][2];
#pragma unroll
        for (int j = 0; j < 2 * P; ++j)
            b[j >> 1][j & 1] = *reinterpret_cast<const float4 *>(st.bias + n + (j >> 1) * 32 + (j & 1) * 4);
        f32x4_t acc[kFM][P][2];
#pragma unroll
        for (int i = 0; i < kFM; ++i)
#pragma unroll
            for (int j = 0; j < 2 * P; ++j) acc[i][j >> 1][j & 1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        uint4 x[2][kFM];
        auto read = [&](int k, uint4 (&v)[kFM]) {
#pragma unroll
            for (int i = 0; i < kFM; ++i) v[i] = *reinterpret_cast<const uint4 *>(smem + k * (kPx * 64) + at[i]);
        };
        read(0, x[0]);
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            // this group's next part, or the next group's first
            if (h + 1 < NH) load_w(w[(h + 1) & 1], wf + (h + 1) * (KH * 2 * 64));
            else if (g + 1 < g1) load_w(w[NH & 1], wf + GROUP);
#pragma unroll
            for (int k = 0; k < KH; ++k) {
                const int s = h * KH + k;
                if (s + 1 < KT) read(s + 1, x[(s + 1) & 1]);
#pragma unroll
                for (int i = 0; i < kFM; ++i)
#pragma unroll
                    for (int j = 0; j < 2 * P; ++j)
                        acc[i][j >> 1][j & 1] =
                            Step<uint16_t>::mma(w[h & 1][k][j >> 1][j & 1], x[s & 1][i], acc[i][j >> 1][j & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (NH == 1) {
#pragma unroll
            for (int k = 0; k < KH; ++k)
#pragma unroll
                for (int j = 0; j < 2 * P; ++j) w[0][k][j >> 1][j & 1] = w[1][k][j >> 1][j & 1];
        }
        wf += GROUP;
        const int py = phase / st.u, px = phase - py * st.u;
        auto store = [&](int i, int c, u32x4_t o) {
            const int y = oy[i] + py, xx = ox[i] + px;
            // read by the next kernel, past the L2
            if (y < a.Ho && xx < a.Wo)
                __builtin_nontemporal_store(
                    o, reinterpret_cast<u32x4_t *>(out + (size_t(y) * a.Wo + xx) * a.ldo + st.c_off + c));
        };
#pragma unroll
        for (int i = 0; i < kFM; ++i) {
            u32x4_t o[P];
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const f32x4_t p = acc[i][j][0], q = acc[i][j][1];
                const float4 b0 = b[j][0], b1 = b[j][1];
                o[j] = u32x4_t{pack_bf16(fmaxf(p[0] + b0.x, 0.f), fmaxf(p[1] + b0.y, 0.f)),
                               pack_bf16(fmaxf(p[2] + b0.z, 0.f), fmaxf(p[3] + b0.w, 0.f)),
                               pack_bf16(fmaxf(q[0] + b1.x, 0.f), fmaxf(q[1] + b1.y, 0.f)),
                               pack_bf16(fmaxf(q[2] + b1.z, 0.f), fmaxf(q[3] + b1.w, 0.f))};
            }
            if constexpr (P == 1) {
                store(i, n, o[0]);
            } else {
                // pixels 0 .. 7 keep their first pair and take it for pixels 8 .. 15,
                // which do so with the second: 8 pixels of 128 bytes in either store
                u32x4_t lo, hi;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned other = swap_halves(upper ? o[0][e] : o[1][e]);
                    lo[e] = upper ? other : o[0][e];
                    hi[e] = upper ? o[1][e] : other;
                }
                store(2 * i, n + (upper ? 32 : 0), lo);
                store(2 * i + 1, n + (upper ? 32 : 0), hi);
            }
        }
    }
}

template <int P>
__global__ __launch_bounds__(256 / P, 2) void k_upsample(UpsampleArgs a) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kPx * 256 * 2];
    // each XCD takes a contiguous run of every stage's blocks (a stage's blocks
    // are one run per map): a stage with many channels costs several times as
    // much per block, and as one run over all stages its blocks had a few XCDs to
    // themselves (64 / 128 / 256 channels at 256 x 256: one map 49 -> 39 us, three
    // 103 -> 82, eight, a map per XCD either way, 154)
    const int xcd = blockIdx.x & 7;
    int b = blockIdx.x >> 3, s = 0;
    while (b >= a.stage[s].run) b -= a.stage[s++].run;
    const UpsampleStage &st = a.stage[s];
    b += xcd * st.run;
    const int bt = b / st.blocks;
    if (bt >= a.batch) return;
    const int bid = b - bt * st.blocks;
    const int groups = st.u * st.u * (a.Co >> 7);
    const int runs = (groups + st.per - 1) / st.per;  // blocks per 64 pixels
    const int m0 = bid / runs * kPx, g0 = bid % runs * st.per;
    const int g1 = g0 + st.per < groups ? g0 + st.per : groups;
    const uint16_t *in = static_cast<const uint16_t *>(a.in[s][bt]);
    uint16_t *out = static_cast<uint16_t *>(a.out[bt]);
    if (st.Ci == 64) up_tile<2, P>(a, st, in, out, m0, g0, g1, smem);
    else if (st.Ci == 128) up_tile<4, P>(a, st, in, out, m0, g0, g1, smem);
    else up_tile<8, P>(a, st, in, out, m0, g0, g1, smem);
}

// Bt [u * u phases][Co][Ci] to [phase][128 channels][wavefront][step][j][lane]:
// lane (fr, fk) of fragment j holds vector fk of channel 32 wavefront + 8 (fr /
// 4) + 4 j + fr % 4, so that rows 4 fk .. 4 fk + 3 of the pair's products are
// channels 8 fk .. 8 fk + 7.
__global__ __launch_bounds__(256) void k_upsample_frag(const uint16_t *wt, uint4 *out, int groups, int KT) {
    const int total = groups * 4 * KT * 2 * 64;
    for (int v = blockIdx.x * 256 + threadIdx.x; v < total; v += gridDim.x * 256) {
        const int lane = v & 63, j = (v >> 6) & 1, k = (v >> 7) % KT, gw = (v >> 7) / KT;
        const int fr = lane & 15, fk = lane >> 4;
        const int n = gw * 32 + 8 * (fr >> 2) + 4 * j + (fr & 3);
        out[v] = *reinterpret_cast<const uint4 *>(wt + size_t(n) * KT * 32 + k * 32 + fk * 8);
    }
}

}  // namespace

hipError_t upsample_frag(const void *wt, void *out, int32_t u, int32_t Co, int32_t Ci, hipStream_t s) {
    if (!upsample_fits(true, Ci, Co)) return hipErrorInvalidValue;
    k_upsample_frag<<<256, 256, 0, s>>>(static_cast<const uint16_t *>(wt), static_cast<uint4 *>(out), u * u * (Co >> 7),
                                        Ci / 32);
    return hipGetLastError();
}

hipError_t upsample(UpsampleArgs a, hipStream_t s) {
    // One group per block and P = 1, for the shortest chain, until the blocks are
    // many times what runs at once; then four groups, so that the pixels are
    // staged for four phases, and P = 2.  One stage by itself (u = 1) takes all
    // groups of its pixels, and P = 2, from 2,560 blocks on; several stages, whose
    // blocks share a CU, gain less in a network than alone (eight maps of 128 x 128
    // with two groups per block 52.5 -> 50.4 alone, a frame 384 -> 386).  And P = 2
    // where its blocks, four per CU, run all at once and those of P = 1, three per
    // CU, do not.  us, over the blocks of one group, P = 1 -> P = 2 (groups per
    // block):
    //   one stage, 256 -> 128    825  17.3 -> 15.3 (1)    1,024 20.1 -> 17.3 (1)    2,048 32.4 -> 34.8 (1)
    //   one stage, 256 -> 256  4,096  50.1 -> 45.5 (2)    6,144 65.5 -> 62.2 (2)
    //   one stage, 256 -> 384    768  12.9 -> 16.2 (2)    3,072 39.6 -> 28.4 (3)    6,144 69.9 -> 60.5 (3)
    //   64 / 128 / 256 -> 128 24,576 189.5 -> 153.0 (4)
    int64_t single = 0;
    for (int q = 0; q < a.n_stages; ++q) {
        const UpsampleStage &st = a.stage[q];
        if (!upsample_fits(true, st.Ci, a.Co)) return hipErrorInvalidValue;
        single += int64_t((st.Hi * st.Wi + kPx - 1) / kPx) * st.u * st.u * (a.Co >> 7);
    }
    single *= a.batch;
    const bool many = single > 14336 || (a.n_stages == 1 && a.Co > 128 && single > 2560);
    const bool two = many || (single > 768 && single <= 1024);
    const int per = many ? 4 : 1;
    int64_t blocks = 0;
    for (int q = 0; q < a.n_stages; ++q) {
        UpsampleStage &st = a.stage[q];
        const int groups = st.u * st.u * (a.Co >> 7);
        st.per = per < groups ? per : groups;
        st.blocks = (st.Hi * st.Wi + kPx - 1) / kPx * ((groups + st.per - 1) / st.per);
        st.run = int32_t((int64_t(st.blocks) * a.batch + 7) / 8);
        blocks += int64_t(st.run) * 8;
    }
    if (two) k_upsample<2><<<unsigned(blocks), 128, 0, s>>>(a);
    else k_upsample<1><<<unsigned(blocks), 256, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace kern
}  // namespace rtcc
