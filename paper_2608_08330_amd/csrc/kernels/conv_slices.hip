// 3x3 convolution with its K loop cut into slices that the wavefronts of one
// block sum side by side, for the layers whose output tiles do not fill the
// chip (ConvPlan::slices).
//
// What bounds these layers is not arithmetic (a 25 x 88 x 128 -> 128 layer is
// 0.3 us of MFMA) but the serial chain of one block: a halo tile that walks
// its K loop step by step spends 20 to 70 steps of barrier, LDS read and
// weight-load latency, and a split over blocks pays a second launch and a
// round trip of the partial sums.  Here a block
//   * stages the whole input patch of its tile, every channel, in LDS with one
//     burst of direct loads and one barrier;
//   * gives every wavefront one K slice (KS chunks of 64 bytes of channels, 9
//     taps each) of its 16 FN output channels, whose weights it loads straight
//     into registers, all at once.  They are stored in fragment order
//     (conv_frag), so a load instruction reads 1 KB in a row; gathering them
//     from the [N][K] matrix takes four times as long, the quads of lanes
//     reading different rows;
//   * adds the slices' partial sums in LDS in slice order and stores the tile.
// The summation order is that of the halo tilings of the layer, cut into the
// same slices: at 128- and 256-byte pixels a slice is one chunk, its taps
// ascending; at 512 bytes it is two, with stride 1 tap by tap (one 128-byte
// chunk of those tilings), with stride 2 one after the other; the slices are
// added in order.  It does not depend on the tile shape: every tile below, and
// the halo tilings with GemmArgs::slices, give the same bits, so the launch picks
// one by the number of maps.
//
// Measured (us per launch; before: split-K tiles + k_splitk_reduce):
//   one map    50 x 176 x 64 -> 64     12.4 -> 4.4   25 x 88 x 128 -> 128  9.8 -> 4.8
//              13 x 44 x 256 -> 256     9.8 -> 5.4   64 x 64 x 32 -> 32 float32 13.5 -> 4.1
//   three maps 128 x 128 x 64 -> 64    26.3 -> 8.0   64 x 64 x 128 -> 128 19.2 -> 7.9
//              32 x 32 x 256 -> 256    17.7 -> 8.9   256 x 256 x 64 -> 64 stride 2  23.9 -> 10.5
//   eight maps 128 x 180 x 64 -> 64    65.4 -> 24.6  64 x 90 x 128 -> 128 36.3 -> 24.6
#include "kernels.hpp"

#include <hip/hip_ext.h>

#include "mfma.hpp"

namespace rtcc {
namespace kern {

namespace {

constexpr int cmax(int a, int b) { return a > b ? a : b; }

// A block owns TH x 16 output pixels and BN = 16 FN WC channels; wavefront
// (slice, wc) sums K slice `slice` of channels [16 FN wc, 16 FN (wc + 1)).
template <typename T, int TH, int FN, int S, int KS, int WC, int STRIDE>
__global__ __launch_bounds__(64 * S * WC) void k_conv_slices(GemmArgs a) {
    constexpr int EPV = Step<T>::EPV;
    constexpr int BK = 4 * EPV;  // channels of a 64-byte chunk
    constexpr int NW = S * WC, NT = 64 * NW;
    // input patch of the tile; with stride 2 the even patch columns are
    // stored first and the odd ones after them, so the 16 pixels a fragment
    // reads (columns 2 x + dx) are consecutive rows in LDS
    constexpr int TW = 16;
    constexpr int HW = STRIDE * (TW - 1) + 3, HH = STRIDE * (TH - 1) + 3;
    constexpr int EVEN = (HW + 1) / 2;
    constexpr int HALO = HH * HW;
    constexpr int IA = (HALO + 15) / 16;  // 1-KB loads (16 pixels x 64 bytes) per chunk
    constexpr int CHT = S * KS;           // chunks of the layer
    constexpr int BN = WC * FN * 16, PX = TH * TW;
    constexpr int RS = BN + 4;            // floats per pixel of a slice's partial tile
    __shared__ __attribute__((aligned(1024))) unsigned char smem[cmax(CHT * IA * 1024, S * PX * RS * 4)];
    const uint32_t lds_base = lds_address(smem);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int slice = wave / WC, wc = wave - slice * WC;

    // each XCD takes a contiguous run of tiles; map bt's blocks are one run
    int bid = blockIdx.x;
    const int nbx = gridDim.x;
    if ((nbx & 7) == 0) bid = (bid & 7) * (nbx >> 3) + (bid >> 3);
    const int nb = a.batch > 1 ? a.batch : 1;
    const int per_map = nbx / nb;
    const int bt = bid / per_map;
    bid -= bt * per_map;
    const T *in = static_cast<const T *>(nb > 1 ? a.in_b[bt] : a.in);
    T *out = static_cast<T *>(nb > 1 ? a.out_b[bt] : a.out);

    const int Ho = a.Ho, Wo = a.Wo;
    const int tx = (Wo + TW - 1) / TW, nt = a.N / BN;
    const int n0 = (bid % nt) * BN;
    const int sp = bid / nt;
    const int oy0 = (sp / tx) * TH, ox0 = (sp % tx) * TW;

    // the patch: 16-byte vector v of pixel row r sits at v ^ ((r >> 1) & 3),
    // so that 8 consecutive rows cover the 32 banks once per LDS read cycle
    for (int q = wave; q < CHT * IA; q += NW) {
        const int c = q / IA, row = (q - c * IA) * 16 + (lane >> 2);
        const int vec = (lane & 3) ^ ((row >> 1) & 3);
        const int hy = row / HW, lc = row - (row / HW) * HW;
        const int hx = STRIDE == 1 ? lc : (lc < EVEN ? 2 * lc : 2 * (lc - EVEN) + 1);
        const int iy = STRIDE * oy0 - 1 + hy, ix = STRIDE * ox0 - 1 + hx;
        const void *g = a.zero;
        if (row < HALO && unsigned(iy) < unsigned(a.Hi) && unsigned(ix) < unsigned(a.Wi))
            g = in + (size_t(iy) * a.Wi + ix) * a.Ci + c * BK + vec * EPV;
        load_lds16(g, lds_base + q * 1024);
    }
    // the wavefront's weights and the bias of the channels this thread stores
    uint4 w[9 * KS][FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const uint4 *p = static_cast<const uint4 *>(a.wfrag) +
                         (size_t((n0 >> 4) + wc * FN + j) * CHT + slice * KS) * (9 * 64) + lane;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) w[t * KS + ks][j] = p[(ks * 9 + t) * 64];
    }
    constexpr int VPP = BN / EPV;  // 16-byte vectors per output pixel
    static_assert(NT % VPP == 0, "a thread stores the same channels of every pixel it takes");
    const int ch = (tid % VPP) * EPV;
    float bias[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) bias[e] = a.bias[n0 + ch + e];

    f32x4_t acc[TH][FN];
#pragma unroll
    for (int i = 0; i < TH; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's part of the patch is in LDS
    __syncthreads();

    const int fr = lane & 15, fk = lane >> 4;
#pragma unroll
    for (int q = 0; q < 9 * KS; ++q) {
        // the halo tilings' order: at 512-byte rows with stride 1 both chunks of
        // a slice tap by tap (a 128-byte chunk there), with stride 2 one after
        // the other
        const int t = STRIDE == 1 ? q / KS : q % 9, ks = STRIDE == 1 ? q % KS : q / 9;
        const int dy = t / 3, dx = t % 3;
        const unsigned char *pa = smem + (slice * KS + ks) * (IA * 1024);
#pragma unroll
        for (int i = 0; i < TH; ++i) {
            const int col = STRIDE == 1 ? dx + fr : ((dx & 1) ? EVEN : dx >> 1) + fr;
            const int r = (STRIDE * i + dy) * HW + col;
            const uint4 x = *reinterpret_cast<const uint4 *>(pa + r * 64 + ((fk ^ ((r >> 1) & 3)) << 4));
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = Step<T>::mma(w[t * KS + ks][j], x, acc[i][j]);
        }
    }
    __syncthreads();  // the patch is read; its LDS holds the partial tiles now
    float *part = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int i = 0; i < TH; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
            *reinterpret_cast<f32x4_t *>(part + (slice * PX + i * 16 + fr) * RS + (wc * FN + j) * 16 + fk * 4) =
                acc[i][j];
    __syncthreads();
    for (int p = tid / VPP; p < PX; p += NT / VPP) {
        const int oy = oy0 + p / TW, ox = ox0 + p % TW;
        if (oy >= Ho || ox >= Wo) continue;
        const float *r = part + p * RS + ch;
        float v[EPV];
#pragma unroll
        for (int e = 0; e < EPV; e += 4) {
            f32x4_t x = *reinterpret_cast<const f32x4_t *>(r + e);
#pragma unroll
            for (int s = 1; s < S; ++s) x += *reinterpret_cast<const f32x4_t *>(r + s * PX * RS + e);
#pragma unroll
            for (int q = 0; q < 4; ++q) v[e + q] = fmaxf(x[q] + bias[e + q], 0.f);
        }
        uint4 o;
        if constexpr (sizeof(T) == 2)
            o = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
        else
            o = make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
        *reinterpret_cast<uint4 *>(out + (size_t(oy) * Wo + ox) * a.ldo + a.c_off + n0 + ch) = o;
    }
}

// Bt [N][9 Ci] to fragment order: fragment (16 channels, chunk, tap) is 64
// lanes x 16 bytes, lane (fr, fk) holding vector fk of channel fr's chunk.
template <typename T>
__global__ __launch_bounds__(256) void k_conv_frag(const T *wt, uint4 *out, int N, int Ci) {
    constexpr int EPV = Step<T>::EPV;
    const int chunks = Ci / (4 * EPV);
    const int total = N / 16 * chunks * 9 * 64;
    for (int v = blockIdx.x * 256 + threadIdx.x; v < total; v += gridDim.x * 256) {
        const int lane = v & 63, f = v >> 6;
        const int t = f % 9, c = f / 9 % chunks, n16 = f / 9 / chunks;
        out[v] = *reinterpret_cast<const uint4 *>(wt + size_t(n16 * 16 + (lane & 15)) * 9 * Ci + t * Ci +
                                                  c * 4 * EPV + (lane >> 4) * EPV);
    }
}

template <typename T, int TH, int FN, int S, int KS, int WC, int STRIDE>
hipError_t launch_tile(const GemmArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    constexpr int BN = WC * FN * 16;
    const unsigned g = unsigned((a.Wo + 15) / 16) * unsigned((a.Ho + TH - 1) / TH) * unsigned(a.N / BN) *
                       unsigned(a.batch > 1 ? a.batch : 1);
    const dim3 block(64 * S * WC);
    if (e0 || e1) hipExtLaunchKernelGGL((k_conv_slices<T, TH, FN, S, KS, WC, STRIDE>), dim3(g), block, 0, s, e0, e1, 0, a);
    else k_conv_slices<T, TH, FN, S, KS, WC, STRIDE><<<g, block, 0, s>>>(a);
    return hipGetLastError();
}

// The tile of a launch.  Where 32-channel tiles of two rows come to at most
// two blocks per CU, they are the fastest (one map of 25 x 88 x 128: 4.8
// against 5.0 us with four rows, 50 x 176 x 64: 4.4 against 4.7, 13 x 44 x
// 256: 5.4 against 6.9): the chain of one block is what counts.  Beyond that
// (several maps per launch) the patch is read for more pixels and channels at
// a time: four rows of 64 channels with two slices (three maps of 128 x 128 x
// 64: 8.0 against 10.4 us), four rows of 32 channels with four (three maps of
// 64 x 64 x 128: 7.9 against 10.0), and, with stride 2, whose patch is twice
// as large, two rows of 64 channels with four (three maps of 64 x 64 x 128 ->
// 256: 7.4 against 7.7 us; four rows: 8.3).
template <typename T, int S, int KS, int STRIDE>
hipError_t launch(const GemmArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const int64_t small = int64_t((a.Wo + 15) / 16) * ((a.Ho + 1) / 2) * (a.N / 32) * (a.batch > 1 ? a.batch : 1);
    if (small <= 2 * int64_t(a.n_cu)) return launch_tile<T, 2, 1, S, KS, 2, STRIDE>(a, s, e0, e1);
    if constexpr (S == 2) {
        if (a.N % 64 == 0) return launch_tile<T, 4, 2, S, KS, 2, STRIDE>(a, s, e0, e1);
    } else if constexpr (STRIDE == 2) {
        if (a.N % 64 == 0) return launch_tile<T, 2, 2, S, KS, 2, STRIDE>(a, s, e0, e1);
    }
    return launch_tile<T, 4, 2, S, KS, 1, STRIDE>(a, s, e0, e1);
}

}  // namespace

hipError_t conv_frag(bool bf16, const void *wt, void *out, int32_t N, int32_t Ci, hipStream_t s) {
    if (bf16) k_conv_frag<uint16_t><<<256, 256, 0, s>>>(static_cast<const uint16_t *>(wt), static_cast<uint4 *>(out), N, Ci);
    else k_conv_frag<float><<<256, 256, 0, s>>>(static_cast<const float *>(wt), static_cast<uint4 *>(out), N, Ci);
    return hipGetLastError();
}

hipError_t conv_slices(bool bf16, const GemmArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const int row = a.Ci * (bf16 ? 2 : 4);
#define RTCC_SLICES(ROW, S, KS)                                                                        \
    if (row == ROW && a.splits == S) {                                                                 \
        if (bf16)                                                                                      \
            return a.stride == 1 ? launch<uint16_t, S, KS, 1>(a, s, e0, e1) : launch<uint16_t, S, KS, 2>(a, s, e0, e1); \
        return a.stride == 1 ? launch<float, S, KS, 1>(a, s, e0, e1) : launch<float, S, KS, 2>(a, s, e0, e1);           \
    }
    RTCC_SLICES(128, 2, 1)
    RTCC_SLICES(256, 4, 1)
    RTCC_SLICES(512, 4, 2)
#undef RTCC_SLICES
    return hipErrorInvalidValue;
}

}  // namespace kern
}  // namespace rtcc
