// The learned-initialization network on the matrix cores: 3x3 convolutions as
// implicit GEMMs with BF16 operands and FP32 accumulation
// (v_mfma_f32_16x16x32_bf16, or 16x16x16 when a layer has 16 input
// channels), plus the input packing, training loss, weight packing, the
// per-crop fallback decision and a masked PSNR.
//
// Activations are NHWC BF16 with the channel count padded to a multiple of
// 16.  A convolution workgroup (4 waves) computes one 16 x 16 pixel tile after
// another, every output channel: the 18 x 18 input halo and the layer's
// weights [cout][9][cin] are staged in LDS (16-byte padded rows), and wave w
// computes tile rows 4w..4w+3 (four M-blocks of 16 pixels) against all
// output-channel N-blocks, the K loop running over the 9 taps x cin.
// Weight gradients are GEMMs over pixels: one workgroup per (pixel split, block
// of channels) accumulates the nine taps' dW_tap[cout][cin] over its tiles from
// LDS copies of the activation window and the output gradient, transposed by
// the LDS reads; a second kernel sums the splits in a fixed order.
#include <algorithm>
#include <type_traits>

#include "dqo_device.hpp"
#include "dqo_learned.h"
#include "net.hpp"

namespace dqo {
namespace net {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float x) {  // round to nearest even
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bool valid_px(const float* rgbdm, int64_t plane, int64_t base) {
    return rgbdm[base + 4 * plane] > 0.5f && rgbdm[base + 3 * plane] > 0.0f;
}

// Two floats to BF16 (round to nearest even), the first in the low half.
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f2bf_pair(float lo, float hi) {
    const bf16x2_t h = __builtin_convertvector(floatx2{lo, hi}, bf16x2_t);
    uint32_t u;
    __builtin_memcpy(&u, &h, 4);
    return u;
}

constexpr int kT = 16;       // output tile edge (pixels)
constexpr int kHalo = kT + 2;

enum { kEpiRelu = 0, kEpiGate = 1, kEpiOut = 2 };

// A workgroup stages the layer's weights once and walks a run of consecutive
// tiles (neighbours along an image row share their halo in L2): the next
// tile's input is in flight in registers while the matrix cores work on the
// current one from LDS.  The weights are the left operand, so a lane ends with
// consecutive channels of a pixel and stores (and gates) 16 bytes at a time.
// At 64 to 64 channels the weights and the input take 121 KB of LDS, so one
// workgroup of four waves has a CU to itself and nothing else hides its loads.
// For 32 crops of 128x128, one tile per workgroup with the weights staged
// every time and 2-byte stores took 101 us (gated: 111 us), 0.38 PFLOP/s; now
// 56 (59) us, 0.69 PFLOP/s, where the traffic of 134 MB (201 MB) takes 27
// (40) us at the copy rate.  Through LDS to 16-byte stores instead: 58 (85).
template <int CIN, int COUT, int EPI>
__global__ __launch_bounds__(256) void conv3x3_kernel(int H, int W, int n_tiles, int run,
                                                      const uint16_t* __restrict__ in,
                                                      const uint16_t* __restrict__ wk, const float* __restrict__ bias,
                                                      const uint16_t* __restrict__ gate, uint16_t* __restrict__ out_bf,
                                                      float* __restrict__ out_f, int nout) {
    constexpr int PIX = CIN + 8;       // LDS elements per halo pixel (16-byte pad)
    constexpr int WROW = 9 * CIN + 8;  // LDS elements per output channel of weights
    constexpr int KS = (CIN % 32 == 0) ? 32 : 16;
    constexpr int NT = COUT / 16;
    static_assert(CIN % 16 == 0 && COUT % 16 == 0, "channels must be multiples of 16");
    __shared__ __attribute__((aligned(16))) uint16_t s_in[kHalo * kHalo * PIX];
    __shared__ __attribute__((aligned(16))) uint16_t s_w[COUT * WROW];
    const int tiles_x = W / kT, tiles_img = tiles_x * (H / kT);
    const int tid = threadIdx.x;
    const int t0 = (int)blockIdx.x * run, t1 = min(n_tiles, t0 + run);
    // this thread's 16-byte pieces of a tile's input: channels c8 of halo pixels
    // tid / CCH, + 256 / CCH, ...
    constexpr int CCH = CIN / 8, kPieces = (kHalo * kHalo * CCH + 255) / 256;
    static_assert(256 % CCH == 0, "a thread keeps its channels");
    const int c8 = tid % CCH, pix0 = tid / CCH;
    uint4 pre[kPieces];
    auto load_tile = [&](int tile) {
        const int img = tile / tiles_img, t = tile - img * tiles_img;
        const int ty0 = (t / tiles_x) * kT, tx0 = (t % tiles_x) * kT;
        const uint16_t* base = in + (size_t)img * H * W * CIN + c8 * 8;
#pragma unroll
        for (int k = 0; k < kPieces; ++k) {
            const int pix = pix0 + k * (256 / CCH);
            const int hy = pix / kHalo, hx = pix - hy * kHalo;
            const int y = ty0 + hy - 1, x = tx0 + hx - 1;
            pre[k] = make_uint4(0u, 0u, 0u, 0u);
            if (pix < kHalo * kHalo && (uint32_t)y < (uint32_t)H && (uint32_t)x < (uint32_t)W)
                pre[k] = *reinterpret_cast<const uint4*>(base + ((size_t)y * W + x) * CIN);
        }
    };
    if (t0 < t1) load_tile(t0);
    constexpr int WCH = 9 * CIN / 8;
    for (int c = tid; c < COUT * WCH; c += 256) {
        const int co = c / WCH, k8 = c - co * WCH;
        // channel 4 NT g + 4 n + r is row 4 g + r of the n-th product, so a lane
        // ends with 4 NT consecutive channels (kEpiOut keeps the order)
        const int row = EPI == kEpiOut ? co : (co / 4 % NT) * 16 + (co / (4 * NT)) * 4 + co % 4;
        *reinterpret_cast<uint4*>(s_w + row * WROW + k8 * 8) =
            *reinterpret_cast<const uint4*>(wk + (size_t)co * 9 * CIN + k8 * 8);
    }
    const int lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    for (int tile = t0; tile < t1; ++tile) {
        const int img = tile / tiles_img, t = tile - img * tiles_img;
        const int ty0 = (t / tiles_x) * kT, tx0 = (t % tiles_x) * kT;
#pragma unroll
        for (int k = 0; k < kPieces; ++k) {
            const int pix = pix0 + k * (256 / CCH);
            if (pix < kHalo * kHalo) *reinterpret_cast<uint4*>(s_in + pix * PIX + c8 * 8) = pre[k];
        }
        __syncthreads();
        // outputs of a lane: pixel (row 4 wave + m, column lr), channels 4 NT lg + 0 ..
        const size_t o0 = (((size_t)img * H + ty0 + wave * 4) * W + tx0 + lr) * COUT + 4 * NT * lg;
        uint4 gt[EPI == kEpiGate ? 4 : 1][EPI == kEpiGate ? NT / 2 : 1];
        if constexpr (EPI == kEpiGate) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int q = 0; q < NT / 2; ++q)
                    gt[m][q] = *reinterpret_cast<const uint4*>(gate + o0 + (size_t)m * W * COUT + q * 8);
        }
        if (tile + 1 < t1) load_tile(tile + 1);
        floatx4 acc[4][NT];
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[m][n] = floatx4{0.f, 0.f, 0.f, 0.f};
        // Steps of KS input channels of one tap, in tap order; the operands of
        // the next step are read from LDS while the matrix cores take this
        // one's (one wave per SIMD: nothing else would hide the reads).
        typedef typename std::conditional<KS == 32, bf16x8_t, short4_t>::type frag_t;
        constexpr int kSteps = 9 * (CIN / KS), kLane = KS / 4;
        frag_t fa[2][4], fb[2][NT];
        auto read_step = [&](int st, frag_t(&a)[4], frag_t(&b)[NT]) {
            const int tap = st / (CIN / KS), kc = (st - tap * (CIN / KS)) * KS, dy = tap / 3, dx = tap - 3 * dy;
#pragma unroll
            for (int m = 0; m < 4; ++m)
                a[m] = *reinterpret_cast<const frag_t*>(s_in + ((wave * 4 + m + dy) * kHalo + lr + dx) * PIX + kc +
                                                        kLane * lg);
#pragma unroll
            for (int n = 0; n < NT; ++n)
                b[n] = *reinterpret_cast<const frag_t*>(s_w + (n * 16 + lr) * WROW + tap * CIN + kc + kLane * lg);
        };
        read_step(0, fa[0], fb[0]);
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
            if (st + 1 < kSteps) read_step(st + 1, fa[(st + 1) & 1], fb[(st + 1) & 1]);
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    // (kEpiOut, planar FP32, wants pixels in a lane's registers: the input on the left)
                    const frag_t l = EPI == kEpiOut ? fa[st & 1][m] : fb[st & 1][n];
                    const frag_t r = EPI == kEpiOut ? fb[st & 1][n] : fa[st & 1][m];
                    if constexpr (KS == 32)
                        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l, r, acc[m][n], 0, 0, 0);
                    else
                        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(l, r, acc[m][n], 0, 0, 0);
                }
        }
        __syncthreads();  // the input is read; its LDS takes the next one
        if constexpr (EPI == kEpiOut) {
            // acc[m][n][r] = output at pixel (row 4 wave + m, column 4 lg + r), channel 16 n + lr
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int y = ty0 + wave * 4 + m;
                const int x0 = tx0 + 4 * lg;
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    const int co = n * 16 + lr;
                    if (co < nout) {
                        const float b0 = bias[co];
                        float4 v = make_float4(acc[m][n][0] + b0, acc[m][n][1] + b0, acc[m][n][2] + b0,
                                               acc[m][n][3] + b0);
                        *reinterpret_cast<float4*>(out_f + (((size_t)img * nout + co) * H + y) * W + x0) = v;
                    }
                }
            }
        } else {
            static_assert(NT % 2 == 0, "16-byte stores");
#pragma unroll
            for (int q = 0; q < NT / 2; ++q) {
                float bv[8];
                if constexpr (EPI == kEpiRelu)
#pragma unroll
                    for (int e = 0; e < 8; ++e) bv[e] = bias[4 * NT * lg + q * 8 + e];
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    uint32_t o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float lo = acc[m][2 * q + e / 2][e % 2 * 2], hi = acc[m][2 * q + e / 2][e % 2 * 2 + 1];
                        if constexpr (EPI == kEpiRelu) {
                            o[e] = f2bf_pair(fmaxf(lo + bv[2 * e], 0.0f), fmaxf(hi + bv[2 * e + 1], 0.0f));
                        } else {  // zero where the gate (a ReLU output) is not positive
                            const uint32_t gw =
                                e == 0 ? gt[m][q].x : e == 1 ? gt[m][q].y : e == 2 ? gt[m][q].z : gt[m][q].w;
                            o[e] = f2bf_pair(bf2f((uint16_t)gw) > 0.0f ? lo : 0.0f,
                                             bf2f((uint16_t)(gw >> 16)) > 0.0f ? hi : 0.0f);
                        }
                    }
                    *reinterpret_cast<uint4*>(out_bf + o0 + (size_t)m * W * COUT + q * 8) =
                        make_uint4(o[0], o[1], o[2], o[3]);
                }
            }
        }
    }
}

// Partial weight gradients over one pixel split, of output channels
// co0 .. co0 + CO_B and input channels ci0 .. ci0 + CI_B (blockIdx.y), all taps:
// part[split][co][tap][ci] = sum over the split's pixels p of g[p][co] * act[p + (dy, dx)][ci],
// part_b[split][co] = sum_p g[p][co].
// Both operands are wanted with pixels along a lane's registers, but lie with
// channels first.  A tile's output gradient and activations (18 x 18, with the
// halo) are staged as they lie, in planes of 16 channels, and ds_read_tr16_b64
// transposes them on the way to the matrix cores, so that one staged copy
// serves the nine taps (a column shift is a pixel's address, where a
// transposed copy would need one copy for each).  Within a row, pixels 8 and
// on lie 4 places further: the 8 pixels that half a wavefront reads, x .. x + 3
// and x + 8 .. x + 11, then cover the 64 banks once.  A wave takes one block
// of 16 input channels, MW blocks of 16 output channels and DXW columns of
// taps; activation rows stay in registers for the next step, two rows on.  The
// last wave sums the output gradient, pixel by pixel in order.  The next
// tile is in flight in registers meanwhile.
// Bound by the loads of one workgroup per CU (43 of the 62 us at 64 to 64
// channels are left without the products and sums, 237 MB at 5.5 TB/s; the
// activations are read for each half of the output channels), then by the
// serial sum (7 to 12 us).  For 32 crops of 128x128, three workgroups per
// split (one for each column of taps) that staged transposed copies took 109
// us at 64 to 64 channels (32 to 64: 85, 64 to 16: 89, 16 to 32: 71); now 62
// (46, 39, 32).
template <int CIN, int COUT>
struct WgradCfg;
template <>
struct WgradCfg<64, 64> { static constexpr int CI_B = 64, CO_B = 32, MW = 2, DXW = 3; };
template <>
struct WgradCfg<32, 64> { static constexpr int CI_B = 32, CO_B = 32, MW = 1, DXW = 3; };
template <>
struct WgradCfg<64, 16> { static constexpr int CI_B = 32, CO_B = 16, MW = 1, DXW = 1; };
template <>
struct WgradCfg<16, 32> { static constexpr int CI_B = 16, CO_B = 16, MW = 1, DXW = 1; };

template <int CIN, int COUT>
constexpr int wgrad_waves() {
    using C = WgradCfg<CIN, COUT>;
    return (C::CI_B / 16) * (C::CO_B / 16 / C::MW) * (3 / C::DXW);
}

typedef __attribute__((address_space(3))) short4_t lds_short4_t;

// 8 consecutive pixels of one channel per lane, from two transposing reads.
__device__ __forceinline__ bf16x8_t read_tr(const uint16_t* lo, const uint16_t* hi) {
    const short4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)lo);
    const short4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)hi);
    bf16x8_t v;
    __builtin_memcpy(&v, &a, 8);
    __builtin_memcpy(reinterpret_cast<char*>(&v) + 8, &b, 8);
    return v;
}

template <int CIN, int COUT>
__global__ __launch_bounds__((wgrad_waves<CIN, COUT>() + 1) * 64) void conv3x3_wgrad_kernel(
    int H, int W, int n_tiles, int tiles_per_split, const uint16_t* __restrict__ act, const uint16_t* __restrict__ g,
    float* __restrict__ part, float* __restrict__ part_b) {
    using C = WgradCfg<CIN, COUT>;
    constexpr int CI_B = C::CI_B, CO_B = C::CO_B, MW = C::MW, DXW = C::DXW;
    constexpr int WAVES = wgrad_waves<CIN, COUT>(), NTHR = (WAVES + 1) * 64;
    constexpr int NTB = CI_B / 16, MTB = CO_B / 16, MG = MTB / MW;
    constexpr int AROW = 26 * 16, APLANE = kHalo * AROW;  // activations: 18 rows of 18 pixels
    constexpr int GROW = 20 * 16, GPLANE = kT * GROW;     // output gradient: 16 rows of 16 pixels
    __shared__ __attribute__((aligned(16))) uint16_t s_a[NTB * APLANE];
    __shared__ __attribute__((aligned(16))) uint16_t s_g[MTB * GPLANE];
    const int split = blockIdx.x;
    const int co0 = ((int)blockIdx.y % (COUT / CO_B)) * CO_B, ci0 = ((int)blockIdx.y / (COUT / CO_B)) * CI_B;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    const int tiles_x = W / kT, tiles_img = tiles_x * (H / kT);
    // this thread's 16-byte pieces (8 channels of a pixel) of a tile
    constexpr int ACH = CI_B / 8, kA = (kHalo * kHalo * ACH + NTHR - 1) / NTHR;
    constexpr int GCH = CO_B / 8, kG = (kT * kT * GCH + NTHR - 1) / NTHR;
    static_assert(NTHR % ACH == 0 && NTHR % GCH == 0, "a thread keeps its channels");
    const int ac = tid % ACH, apix0 = tid / ACH, gc = tid % GCH, gpix0 = tid / GCH;
    uint4 pa[kA], pg[kG];
    auto load_tile = [&](int tile) {
        const int img = tile / tiles_img, t = tile - img * tiles_img;
        const int ty0 = (t / tiles_x) * kT, tx0 = (t % tiles_x) * kT;
        const uint16_t* ba = act + (size_t)img * H * W * CIN + ci0 + ac * 8;
        const uint16_t* bg = g + (((size_t)img * H + ty0) * W + tx0) * COUT + co0 + gc * 8;
#pragma unroll
        for (int k = 0; k < kA; ++k) {
            const int pix = apix0 + k * (NTHR / ACH), hy = pix / kHalo, hx = pix - hy * kHalo;
            const int y = ty0 + hy - 1, x = tx0 + hx - 1;
            pa[k] = make_uint4(0u, 0u, 0u, 0u);
            if (pix < kHalo * kHalo && (uint32_t)y < (uint32_t)H && (uint32_t)x < (uint32_t)W)
                pa[k] = *reinterpret_cast<const uint4*>(ba + ((size_t)y * W + x) * CIN);
        }
#pragma unroll
        for (int k = 0; k < kG; ++k) {
            const int pix = gpix0 + k * (NTHR / GCH);
            pg[k] = make_uint4(0u, 0u, 0u, 0u);
            if (pix < kT * kT)
                pg[k] = *reinterpret_cast<const uint4*>(bg + ((size_t)(pix / kT) * W + pix % kT) * COUT);
        }
    };
    // the wave's part, and where its lanes read: a transposing read of 16 lanes
    // takes 4 pixels x 16 channels, lane i giving pixel i / 4, channels 4 (i % 4) ..
    const int nt = wave % NTB, mg = wave / NTB % MG, dx0 = wave / (NTB * MG) * DXW;
    const int cx = 8 * (lg & 1) + (lr >> 2), cc = 4 * (lr & 3);
    const uint16_t* ra[DXW][2];
#pragma unroll
    for (int x = 0; x < DXW; ++x)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int hx = cx + 4 * h + dx0 + x;
            ra[x][h] = s_a + nt * APLANE + (lg >> 1) * AROW + (hx + 4 * (hx >> 3)) * 16 + cc;
        }
    const uint16_t* rg = s_g + mg * MW * GPLANE + (lg >> 1) * GROW + (cx + 4 * (cx >> 3)) * 16 + cc;
    floatx4 acc[MW][DXW][3];
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int x = 0; x < DXW; ++x)
#pragma unroll
            for (int d = 0; d < 3; ++d) acc[m][x][d] = floatx4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.0f;
    const int t_begin = split * tiles_per_split;
    const int t_end = min(n_tiles, t_begin + tiles_per_split);
    if (t_begin < t_end) load_tile(t_begin);
    for (int t = t_begin; t < t_end; ++t) {
        if (t != t_begin) __syncthreads();  // the previous tile is read
#pragma unroll
        for (int k = 0; k < kA; ++k) {
            const int pix = apix0 + k * (NTHR / ACH), hy = pix / kHalo, hx = pix - hy * kHalo;
            if (pix < kHalo * kHalo)
                *reinterpret_cast<uint4*>(s_a + (ac >> 1) * APLANE + hy * AROW + (hx + 4 * (hx >> 3)) * 16 +
                                          (ac & 1) * 8) = pa[k];
        }
#pragma unroll
        for (int k = 0; k < kG; ++k) {
            const int pix = gpix0 + k * (NTHR / GCH), x = pix % kT;
            if (pix < kT * kT)
                *reinterpret_cast<uint4*>(s_g + (gc >> 1) * GPLANE + (pix / kT) * GROW + (x + 4 * (x >> 3)) * 16 +
                                          (gc & 1) * 8) = pg[k];
        }
        __syncthreads();
        if (t + 1 < t_end) load_tile(t + 1);
        if (wave < WAVES) {
            // step s: pixel rows 2 s and 2 s + 1; tap row d reads activation rows 2 s + d and + 1
            constexpr int kSteps = kT / 2;
            bf16x8_t fg[2][MW], fa[2 * kSteps + 1][DXW];
#pragma unroll
            for (int m = 0; m < MW; ++m) fg[0][m] = read_tr(rg + m * GPLANE, rg + m * GPLANE + 4 * 16);
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int x = 0; x < DXW; ++x) fa[r][x] = read_tr(ra[x][0] + r * AROW, ra[x][1] + r * AROW);
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                if (s + 1 < kSteps) {
#pragma unroll
                    for (int m = 0; m < MW; ++m) {
                        const uint16_t* p = rg + m * GPLANE + 2 * (s + 1) * GROW;
                        fg[(s + 1) & 1][m] = read_tr(p, p + 4 * 16);
                    }
#pragma unroll
                    for (int r = 2 * s + 3; r < 2 * s + 5; ++r)
#pragma unroll
                        for (int x = 0; x < DXW; ++x) fa[r][x] = read_tr(ra[x][0] + r * AROW, ra[x][1] + r * AROW);
                }
#pragma unroll
                for (int m = 0; m < MW; ++m)
#pragma unroll
                    for (int x = 0; x < DXW; ++x)
#pragma unroll
                        for (int d = 0; d < 3; ++d)
                            acc[m][x][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fg[s & 1][m], fa[2 * s + d][x],
                                                                                   acc[m][x][d], 0, 0, 0);
            }
        } else if (ci0 == 0) {
            // lane: channel lr of plane lg % MTB, 4 pixels at a time
            const uint16_t* p = s_g + (lg % MTB) * GPLANE + (lr >> 2) * 16 + cc;
#pragma unroll 2
            for (int row = 0; row < kT; ++row) {
                short4_t v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (lds_short4_t*)(p + row * GROW + (4 * q + 4 * (q >> 1)) * 16));
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int j = 0; j < 4; ++j) bsum += bf2f((uint16_t)v[q][j]);
            }
        }
    }
    if (wave < WAVES) {
        // acc[m][x][d][r] = dW[co = 16 mt + 4 lg + r][tap = 3 d + dx][ci = 16 nt + lr]
#pragma unroll
        for (int m = 0; m < MW; ++m)
#pragma unroll
            for (int x = 0; x < DXW; ++x)
#pragma unroll
                for (int d = 0; d < 3; ++d)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int co = co0 + (mg * MW + m) * 16 + 4 * lg + r, ci = ci0 + nt * 16 + lr;
                        part[((size_t)split * COUT + co) * 9 * CIN + (3 * d + dx0 + x) * CIN + ci] = acc[m][x][d][r];
                    }
    } else if (ci0 == 0 && lg < MTB) {
        part_b[split * COUT + co0 + lane] = bsum;
    }
}

// Sums the splits' partial weight gradients: a workgroup takes 64 entries,
// its four waves a quarter of the splits each (split q, q + 4, ... in order),
// and the four partial sums are added in wave order (a fixed order: the
// result does not depend on timing).
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(int S, int64_t E, int cout, const float* __restrict__ part,
                                                           const float* __restrict__ part_b, float* __restrict__ gw,
                                                           float* __restrict__ gb) {
    __shared__ float s_sum[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int64_t e = (int64_t)blockIdx.x * 64 + lane;  // entries E.. are the biases
    const bool is_w = e < E, is_b = !is_w && e < E + cout;
    const float* src = is_w ? part + e : part_b + (e - E);
    const int64_t stride = is_w ? E : (int64_t)cout;
    float s = 0.0f;
    if (is_w || is_b)
        for (int k0 = q; k0 < S; k0 += 32) {
            // eight loads in flight, then added in split order
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = (k0 + 4 * j < S) ? src[(int64_t)(k0 + 4 * j) * stride] : 0.0f;
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[j];
        }
    s_sum[q][lane] = s;
    __syncthreads();
    if (q == 0 && (is_w || is_b)) {
        const float t = ((s_sum[0][lane] + s_sum[1][lane]) + s_sum[2][lane]) + s_sum[3][lane];
        if (is_w) gw[e] = t;
        else gb[e - E] = t;
    }
}

// Per-crop reductions (smallest depth, mean log-error, PSNR): one workgroup of
// kCropThreads per crop, kCropUnroll pixels per thread in flight, wavefront
// shuffles and one LDS step.  They are bound by the latency of one CU's reads
// (128 KB per 128x128 crop): 256 threads with one pixel in flight and a
// barrier tree took 10 to 30 us.
constexpr int kCropThreads = 1024;
constexpr int kCropUnroll = 4;

// The workgroup's combination of one value per thread, in thread 0 (a fixed order).
template <typename A, typename F>
__device__ __forceinline__ A crop_reduce(A v, A (&s)[kCropThreads / kWave], F f) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = f(v, (A)__shfl_xor(v, d));
    if ((threadIdx.x & (kWave - 1)) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    A r = s[0];
    for (int w = 1; w < kCropThreads / kWave; ++w) r = f(r, s[w]);
    return r;
}

// Smallest valid depth of each crop.
__global__ __launch_bounds__(kCropThreads) void dmin_kernel(int HW, const float* __restrict__ rgbdm,
                                                            float* __restrict__ dmin) {
    __shared__ float s[kCropThreads / kWave];
    const int b = blockIdx.x;
    const float* base = rgbdm + (size_t)b * 5 * HW;
    float m = INFINITY;
    for (int i0 = threadIdx.x; i0 < HW; i0 += kCropUnroll * kCropThreads) {
        float d[kCropUnroll], k[kCropUnroll];
#pragma unroll
        for (int u = 0; u < kCropUnroll; ++u) {
            const int i = min(i0 + u * kCropThreads, HW - 1);  // a pixel twice does not change the least
            d[u] = base[3 * HW + i];
            k[u] = base[4 * HW + i];
        }
#pragma unroll
        for (int u = 0; u < kCropUnroll; ++u)
            if (k[u] > 0.5f && d[u] > 0.0f) m = fminf(m, d[u]);
    }
    m = crop_reduce(m, s, [](float a, float c) { return fminf(a, c); });
    if (threadIdx.x == 0) dmin[b] = m;
}

// NHWC16 BF16 input: r, g, b, 4 (d - d_min) / d_min (valid pixels), valid, zeros.
__global__ __launch_bounds__(256) void input_kernel(int64_t P, int HW, const float* __restrict__ rgbdm,
                                                    const float* __restrict__ dmin, uint16_t* __restrict__ x0) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= P) return;
    const int64_t b = p / HW, i = p - b * HW;
    const int64_t base = b * 5 * HW + i;
    const bool ok = valid_px(rgbdm, HW, base);
    float rel = 0.0f;
    if (ok) {
        const float dm = dmin[b];
        rel = 4.0f * __fdiv_rn(rgbdm[base + 3 * HW] - dm, dm);
    }
    uint32_t w[8];
    w[0] = (uint32_t)f2bf(rgbdm[base]) | ((uint32_t)f2bf(rgbdm[base + HW]) << 16);
    w[1] = (uint32_t)f2bf(rgbdm[base + 2 * HW]) | ((uint32_t)f2bf(rel) << 16);
    w[2] = (uint32_t)f2bf(ok ? 1.0f : 0.0f);
#pragma unroll
    for (int k = 3; k < 8; ++k) w[k] = 0u;
    uint4* dst = reinterpret_cast<uint4*>(x0 + p * 16);
    dst[0] = make_uint4(w[0], w[1], w[2], w[3]);
    dst[1] = make_uint4(w[4], w[5], w[6], w[7]);
}

// theta -> BF16 forward copy (same order) and transposed copy [cin][9 - 1 - tap][cout].
__global__ __launch_bounds__(256) void pack_kernel(int cin, int cout, const float* __restrict__ w,
                                                   uint16_t* __restrict__ wf, uint16_t* __restrict__ wt) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= cout * 9 * cin) return;
    const int co = e / (9 * cin), r = e - co * 9 * cin, tap = r / cin, ci = r - tap * cin;
    const uint16_t h = f2bf(w[e]);
    wf[e] = h;
    wt[(ci * 9 + (8 - tap)) * cout + co] = h;
}

__global__ __launch_bounds__(256) void count_kernel(int64_t P, int HW, const float* __restrict__ rgbdm,
                                                    int32_t* __restrict__ cnt) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int c = 0;
    if (p < P) {
        const int64_t b = p / HW, i = p - b * HW;
        c = valid_px(rgbdm, HW, b * 5 * HW + i) ? 1 : 0;
    }
    __shared__ int s[256];
    s[threadIdx.x] = c;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) s[threadIdx.x] += s[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) cnt[blockIdx.x] = s[0];
}

__global__ __launch_bounds__(256) void count_total_kernel(int nblk, const int32_t* __restrict__ cnt,
                                                          int64_t* __restrict__ total) {
    __shared__ int64_t s[256];
    int64_t c = 0;
    for (int i = threadIdx.x; i < nblk; i += 256) c += cnt[i];
    s[threadIdx.x] = c;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) s[threadIdx.x] += s[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = s[0];
}

struct ChanW {
    float w[5];
};

// Per valid pixel: the loss terms and dL/dout (BF16, NHWC16, zero elsewhere).
__global__ __launch_bounds__(256) void loss_kernel(int64_t P, int HW, const float* __restrict__ rgbdm,
                                                   const float* __restrict__ out, const float* __restrict__ lab,
                                                   ChanW cw, const int64_t* __restrict__ total,
                                                   uint16_t* __restrict__ g4, double* __restrict__ part) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double l_all = 0.0, l_fit = 0.0;
    if (p < P) {
        const int64_t b = p / HW, i = p - b * HW;
        const bool ok = valid_px(rgbdm, HW, b * 5 * HW + i);
        uint32_t w[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
        if (ok) {
            const float inv_m = 1.0f / (float)max(*total, (int64_t)1);
            float e[5], s = 0.0f;
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                e[c] = out[(b * 6 + c) * HW + i] - lab[(b * 5 + c) * HW + i];
                s += cw.w[c] * e[c] * e[c];
            }
            const float r = logf(s + 1e-4f);
            const float d5 = out[(b * 6 + 5) * HW + i] - r;
            l_all = (double)s + (double)d5 * d5;
            l_fit = (double)s;
            uint16_t h[6];
#pragma unroll
            for (int c = 0; c < 5; ++c) h[c] = f2bf(2.0f * cw.w[c] * e[c] * inv_m);
            h[5] = f2bf(2.0f * d5 * inv_m);
            w[0] = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
            w[1] = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
            w[2] = (uint32_t)h[4] | ((uint32_t)h[5] << 16);
        }
        uint4* dst = reinterpret_cast<uint4*>(g4 + p * 16);
        dst[0] = make_uint4(w[0], w[1], w[2], w[3]);
        dst[1] = make_uint4(w[4], w[5], w[6], w[7]);
    }
    __shared__ double s0[256], s1[256];
    s0[threadIdx.x] = l_all;
    s1[threadIdx.x] = l_fit;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) {
            s0[threadIdx.x] += s0[threadIdx.x + k];
            s1[threadIdx.x] += s1[threadIdx.x + k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = s0[0];
        part[2 * blockIdx.x + 1] = s1[0];
    }
}

__global__ __launch_bounds__(256) void loss_final_kernel(int nblk, const double* __restrict__ part,
                                                         const int64_t* __restrict__ total, double* __restrict__ loss) {
    __shared__ double s0[256], s1[256];
    double a = 0.0, f = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 256) {
        a += part[2 * i];
        f += part[2 * i + 1];
    }
    s0[threadIdx.x] = a;
    s1[threadIdx.x] = f;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) {
            s0[threadIdx.x] += s0[threadIdx.x + k];
            s1[threadIdx.x] += s1[threadIdx.x + k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double m = (double)max(*total, (int64_t)1);
        loss[0] = s0[0] / m;
        loss[1] = s1[0] / m;
    }
}

// Mean predicted log-error over each crop's valid pixels and the decision.
__global__ __launch_bounds__(kCropThreads) void fallback_kernel(int HW, const float* __restrict__ rgbdm,
                                                                const float* __restrict__ out, float thr,
                                                                int32_t* __restrict__ use_pred,
                                                                float* __restrict__ mean_out) {
    __shared__ float ss[kCropThreads / kWave];
    __shared__ int sc[kCropThreads / kWave];
    const int64_t b = blockIdx.x;
    const float* c5 = rgbdm + b * 5 * HW;
    const float* o = out + (b * 6 + 5) * HW;
    float s = 0.0f;
    int c = 0;
    for (int i0 = threadIdx.x; i0 < HW; i0 += kCropUnroll * kCropThreads) {
        float d[kCropUnroll], k[kCropUnroll], e[kCropUnroll];
#pragma unroll
        for (int u = 0; u < kCropUnroll; ++u) {
            const int i = min(i0 + u * kCropThreads, HW - 1);
            d[u] = c5[3 * (int64_t)HW + i];
            k[u] = c5[4 * (int64_t)HW + i];
            e[u] = o[i];
        }
#pragma unroll
        for (int u = 0; u < kCropUnroll; ++u)
            if (i0 + u * kCropThreads < HW && k[u] > 0.5f && d[u] > 0.0f) {
                s += e[u];
                ++c;
            }
    }
    s = crop_reduce(s, ss, [](float a, float x) { return a + x; });
    c = crop_reduce(c, sc, [](int a, int x) { return a + x; });
    if (threadIdx.x == 0) {
        const float mean = c > 0 ? s / (float)c : INFINITY;
        use_pred[b] = mean <= thr ? 1 : 0;
        if (mean_out) mean_out[b] = mean;
    }
}

__global__ __launch_bounds__(kCropThreads) void psnr_kernel(int HW, const float* __restrict__ color,
                                                            const float* __restrict__ rgbdm,
                                                            double* __restrict__ psnr) {
    __shared__ double ss[kCropThreads / kWave];
    __shared__ int sc[kCropThreads / kWave];
    const int64_t v = blockIdx.x, N = HW;
    const float* c5 = rgbdm + v * 5 * N;
    const float* col = color + v * 3 * N;
    double s = 0.0;
    int c = 0;
    for (int i0 = threadIdx.x; i0 < HW; i0 += kCropUnroll * kCropThreads) {
        float d[kCropUnroll], k[kCropUnroll], a[kCropUnroll][3], t[kCropUnroll][3];
#pragma unroll
        for (int u = 0; u < kCropUnroll; ++u) {
            const int64_t i = min(i0 + u * kCropThreads, HW - 1);
            d[u] = c5[3 * N + i];
            k[u] = c5[4 * N + i];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                a[u][q] = col[q * N + i];
                t[u][q] = c5[q * N + i];
            }
        }
#pragma unroll
        for (int u = 0; u < kCropUnroll; ++u)
            if (i0 + u * kCropThreads < HW && k[u] > 0.5f && d[u] > 0.0f) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const double e = (double)a[u][q] - (double)t[u][q];
                    s += e * e;
                }
                ++c;
            }
    }
    s = crop_reduce(s, ss, [](double x, double y) { return x + y; });
    c = crop_reduce(c, sc, [](int x, int y) { return x + y; });
    if (threadIdx.x == 0) psnr[v] = c > 0 ? 10.0 * log10(3.0 * c / s) : 0.0;
}

// ------------------------------------------------------------------ launchers
template <int CIN, int COUT, int EPI>
static void conv(int B, int H, int W, const uint16_t* in, const uint16_t* wk, const float* bias, const uint16_t* gate,
                 uint16_t* out_bf, float* out_f, int nout, hipStream_t st) {
    const int n_tiles = B * (H / kT) * (W / kT);
    // as many workgroups as the device holds at once, the tiles dealt to them
    // in equal runs (one tile each while there are fewer tiles)
    const int resident = std::max(256, resident_blocks<conv3x3_kernel<CIN, COUT, EPI>, 256>());
    const int run = (n_tiles + resident - 1) / resident;
    hipLaunchKernelGGL((conv3x3_kernel<CIN, COUT, EPI>), dim3((unsigned)((n_tiles + run - 1) / run)), dim3(256), 0, st,
                       H, W, n_tiles, run, in, wk, bias, gate, out_bf, out_f, nout);
}

template <int CIN, int COUT>
static void wgrad(const Work& w, int B, int H, int W, const uint16_t* act, const uint16_t* g, float* gw, float* gb,
                  hipStream_t st) {
    const int n_tiles = B * (H / kT) * (W / kT);
    const int S = w.splits;
    const int per = (n_tiles + S - 1) / S;
    using C = WgradCfg<CIN, COUT>;
    hipLaunchKernelGGL((conv3x3_wgrad_kernel<CIN, COUT>), dim3(S, (CIN / C::CI_B) * (COUT / C::CO_B)),
                       dim3((wgrad_waves<CIN, COUT>() + 1) * 64), 0, st, H, W, n_tiles, per, act, g, w.part, w.part_b);
    const int64_t E = (int64_t)COUT * 9 * CIN;
    hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((unsigned)((E + COUT + 63) / 64)), dim3(256), 0, st, S, E, COUT, w.part,
                       w.part_b, gw, gb);
}

hipError_t launch_pack(const dqo_net_layout& L, const float* theta, uint16_t* wf, uint16_t* wt, hipStream_t st) {
    for (int l = 0; l < DQO_NET_LAYERS; ++l) {
        const int ci = L.cin_pad[l], co = L.cout_pad[l];
        const int E = co * 9 * ci;
        hipLaunchKernelGGL(pack_kernel, dim3((E + 255) / 256), dim3(256), 0, st, ci, co, theta + L.w_offset[l],
                           wf + L.wk_offset[l], wt + L.wk_offset[l]);
    }
    return hipGetLastError();
}

hipError_t launch_forward(const dqo_net_layout& L, const Work& w, int B, int H, int W, const float* rgbdm,
                          const uint16_t* wf, const float* theta, float* out, hipStream_t st) {
    const int HW = H * W;
    const int64_t P = (int64_t)B * HW;
    const unsigned pb = (unsigned)((P + 255) / 256);
    hipLaunchKernelGGL(dmin_kernel, dim3(B), dim3(kCropThreads), 0, st, HW, rgbdm, w.dmin);
    hipLaunchKernelGGL(input_kernel, dim3(pb), dim3(256), 0, st, P, HW, rgbdm, w.dmin, w.x0);
    conv<16, 32, kEpiRelu>(B, H, W, w.x0, wf + L.wk_offset[0], theta + L.b_offset[0], nullptr, w.a1, nullptr, 0, st);
    conv<32, 64, kEpiRelu>(B, H, W, w.a1, wf + L.wk_offset[1], theta + L.b_offset[1], nullptr, w.a2, nullptr, 0, st);
    conv<64, 64, kEpiRelu>(B, H, W, w.a2, wf + L.wk_offset[2], theta + L.b_offset[2], nullptr, w.a3, nullptr, 0, st);
    conv<64, 16, kEpiOut>(B, H, W, w.a3, wf + L.wk_offset[3], theta + L.b_offset[3], nullptr, nullptr, out,
                          DQO_NET_OUT, st);
    return hipGetLastError();
}

hipError_t launch_loss(const Work& w, int B, int H, int W, const float* rgbdm, const float* out, const float* labels,
                       const double* chan_w, double* loss, hipStream_t st) {
    const int HW = H * W;
    const int64_t P = (int64_t)B * HW;
    const int nblk = (int)((P + 255) / 256);
    ChanW cw;
    for (int c = 0; c < 5; ++c) cw.w[c] = (float)chan_w[c];
    hipLaunchKernelGGL(count_kernel, dim3(nblk), dim3(256), 0, st, P, HW, rgbdm, w.cnt);
    hipLaunchKernelGGL(count_total_kernel, dim3(1), dim3(256), 0, st, nblk, w.cnt, w.total);
    hipLaunchKernelGGL(loss_kernel, dim3(nblk), dim3(256), 0, st, P, HW, rgbdm, out, labels, cw, w.total, w.g4,
                       w.lpart);
    hipLaunchKernelGGL(loss_final_kernel, dim3(1), dim3(256), 0, st, nblk, w.lpart, w.total, loss);
    return hipGetLastError();
}

hipError_t launch_backward(const dqo_net_layout& L, const Work& w, int B, int H, int W, const uint16_t* wt,
                           float* grad, hipStream_t st) {
    wgrad<64, 16>(w, B, H, W, w.a3, w.g4, grad + L.w_offset[3], grad + L.b_offset[3], st);
    conv<16, 64, kEpiGate>(B, H, W, w.g4, wt + L.wk_offset[3], nullptr, w.a3, w.gA, nullptr, 0, st);
    wgrad<64, 64>(w, B, H, W, w.a2, w.gA, grad + L.w_offset[2], grad + L.b_offset[2], st);
    conv<64, 64, kEpiGate>(B, H, W, w.gA, wt + L.wk_offset[2], nullptr, w.a2, w.gB, nullptr, 0, st);
    wgrad<32, 64>(w, B, H, W, w.a1, w.gB, grad + L.w_offset[1], grad + L.b_offset[1], st);
    conv<64, 32, kEpiGate>(B, H, W, w.gB, wt + L.wk_offset[1], nullptr, w.a1, w.gA, nullptr, 0, st);
    wgrad<16, 32>(w, B, H, W, w.x0, w.gA, grad + L.w_offset[0], grad + L.b_offset[0], st);
    return hipGetLastError();
}

hipError_t launch_fallback(int B, int H, int W, const float* rgbdm, const float* out, float thr, int32_t* use_pred,
                           float* mean_out, hipStream_t st) {
    hipLaunchKernelGGL(fallback_kernel, dim3(B), dim3(kCropThreads), 0, st, H * W, rgbdm, out, thr, use_pred, mean_out);
    return hipGetLastError();
}

hipError_t launch_psnr(int V, int H, int W, const float* color, const float* rgbdm, double* psnr, hipStream_t st) {
    hipLaunchKernelGGL(psnr_kernel, dim3(V), dim3(kCropThreads), 0, st, H * W, color, rgbdm, psnr);
    return hipGetLastError();
}

}  // namespace net
}  // namespace dqo
