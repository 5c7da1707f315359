// Gaussians spawned from RGB-D crops, one per valid pixel in raster order
// (plain back-projection, optionally corrected by the network's per-pixel
// prediction), and the training labels read back from converged Gaussians.
// A crop is split into at most kInitChunks runs of pixels, a workgroup each;
// every valid pixel's column is the crop's first plus the valid pixels in
// front of it, which the workgroup counts itself.
#include "dqo_device.hpp"
#include "net.hpp"

namespace dqo {
namespace net {

constexpr int kInitThreads = 512;
constexpr int kInitChunks = 64;

__device__ __forceinline__ bool valid_at(const float* c, int HW, int i) {
    return c[4 * HW + i] > 0.5f && c[3 * HW + i] > 0.0f;
}

// Pixels per workgroup: whole rounds of kInitThreads.
inline int init_chunk(int HW) {
    const int per = (HW + kInitChunks - 1) / kInitChunks;
    return (per + kInitThreads - 1) / kInitThreads * kInitThreads;
}

// The valid pixels of a crop before pixel n, and the ranks of later ones.
// The count reads 8 bytes per pixel in front of the run again (up to 128 KB
// for the last run of a 128x128 crop, eight loads in flight per thread),
// which needs no pass of its own and no scratch memory.
struct InitRank {
    static constexpr int kWaves = kInitThreads / kWave;
    int base;  // valid pixels in front of the next round

    __device__ void start(const float* c, int HW, int n, int (&s)[2][kWaves]) {
        int cnt = 0;
        constexpr int U = 4;
        for (int i0 = threadIdx.x; i0 < n; i0 += U * kInitThreads) {
            float mk[U], dp[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int i = min(i0 + k * kInitThreads, HW - 1);
                mk[k] = c[4 * HW + i];
                dp[k] = c[3 * HW + i];
            }
#pragma unroll
            for (int k = 0; k < U; ++k) cnt += (i0 + k * kInitThreads < n && mk[k] > 0.5f && dp[k] > 0.0f) ? 1 : 0;
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d);
        if ((threadIdx.x & (kWave - 1)) == 0) s[0][threadIdx.x >> 6] = cnt;
        __syncthreads();
        base = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) base += s[0][w];
    }
    // The rank of this thread's pixel (if valid) in round `round` = 0, 1, ...;
    // the two buffers take turns, so one barrier a round is enough.
    __device__ int next(bool ok, int round, int (&s)[2][kWaves]) {
        const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
        const uint64_t bal = __ballot(ok);
        int(&sb)[kWaves] = s[(round + 1) & 1];
        if (lane == 0) sb[wave] = (int)__popcll(bal);
        __syncthreads();
        int rank = base + (int)__popcll(bal & (lane ? (~0ull >> (kWave - lane)) : 0ull));
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            rank += w < wave ? sb[w] : 0;
            base += sb[w];
        }
        return rank;
    }
};

// One workgroup per crop with a thread on 16 consecutive pixels took 68 us on
// one 128x128 crop; now 6 us (latency of the count and of one round).
__global__ __launch_bounds__(kInitThreads) void init_kernel(int H, int W, int chunk, const float* __restrict__ rgbdm,
                                                            InitCams cams, const int64_t* __restrict__ offsets,
                                                            const float* __restrict__ pred,
                                                            const int32_t* __restrict__ use_pred, int64_t n,
                                                            float* __restrict__ params, int32_t* __restrict__ ids,
                                                            int32_t obj_id) {
    __shared__ int s_rank[2][InitRank::kWaves];
    const int b = blockIdx.y, HW = H * W;
    const float* c = rgbdm + (size_t)b * 5 * HW;
    const int i0 = (int)blockIdx.x * chunk, i1 = min(HW, i0 + chunk);
    const int64_t first = offsets[b], last = min(offsets[b + 1], n);
    const bool corr = pred != nullptr && (use_pred == nullptr || use_pred[b] != 0);
    const float fx = cams.fx[b], fy = cams.fy[b], cx = cams.cx[b], cy = cams.cy[b];
    const float* R = cams.R[b];
    const float* t = cams.t[b];
    InitRank rk;
    rk.start(c, HW, i0, s_rank);
    for (int r0 = i0, round = 0; r0 < i1; r0 += kInitThreads, ++round) {
        const int i = r0 + (int)threadIdx.x;
        const bool ok = i < i1 && valid_at(c, HW, i);
        const int64_t col = first + rk.next(ok, round, s_rank);
        if (!ok || col < 0 || col >= last) continue;
        const int v = i / W, u = i - v * W;
        const float d = c[3 * HW + i];
        const float xc[3] = {d * ((float)u + 0.5f - cx) / fx - t[0], d * ((float)v + 0.5f - cy) / fy - t[1],
                             d - t[2]};
        float ls = logf(d / fx), eta = logf(9.0f);
        float rgb[3] = {c[i], c[HW + i], c[2 * HW + i]};
        if (corr) {
            const float* pp = pred + (size_t)b * 6 * HW + i;
            ls += pp[0];
            eta = pp[HW];
            rgb[0] += pp[2 * HW];
            rgb[1] += pp[3 * HW];
            rgb[2] += pp[4 * HW];
        }
        float vals[kParams];
        // world mean = R^T (x_c - t)
        vals[0] = R[0] * xc[0] + R[3] * xc[1] + R[6] * xc[2];
        vals[1] = R[1] * xc[0] + R[4] * xc[1] + R[7] * xc[2];
        vals[2] = R[2] * xc[0] + R[5] * xc[1] + R[8] * xc[2];
        vals[3] = vals[4] = vals[5] = ls;
        vals[6] = 1.0f;
        vals[7] = vals[8] = vals[9] = 0.0f;
        vals[10] = eta;
        vals[11] = rgb[0];
        vals[12] = rgb[1];
        vals[13] = rgb[2];
#pragma unroll
        for (int r = 0; r < kParams; ++r) params[(int64_t)r * n + col] = vals[r];
        ids[col] = obj_id;
    }
}

__global__ __launch_bounds__(kInitThreads) void labels_kernel(int H, int W, int chunk, const float* __restrict__ rgbdm,
                                                              InitCams cams, const int64_t* __restrict__ offsets,
                                                              const float* __restrict__ params, int64_t n,
                                                              float* __restrict__ labels) {
    __shared__ int s_rank[2][InitRank::kWaves];
    const int b = blockIdx.y, HW = H * W;
    const float* c = rgbdm + (size_t)b * 5 * HW;
    float* lab = labels + (size_t)b * 5 * HW;
    const int i0 = (int)blockIdx.x * chunk, i1 = min(HW, i0 + chunk);
    const int64_t first = offsets[b], last = min(offsets[b + 1], n);
    const float fx = cams.fx[b];
    InitRank rk;
    rk.start(c, HW, i0, s_rank);
    for (int r0 = i0, round = 0; r0 < i1; r0 += kInitThreads, ++round) {
        const int i = r0 + (int)threadIdx.x;
        const bool ok = i < i1 && valid_at(c, HW, i);
        const int64_t col = first + rk.next(ok, round, s_rank);
        if (i >= i1) continue;
        float l[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if (ok && col >= 0 && col < last) {
            const float d = c[3 * HW + i];
            l[0] = (params[3 * n + col] + params[4 * n + col] + params[5 * n + col]) / 3.0f - logf(d / fx);
            l[1] = params[10 * n + col];
            l[2] = params[11 * n + col] - c[i];
            l[3] = params[12 * n + col] - c[HW + i];
            l[4] = params[13 * n + col] - c[2 * HW + i];
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) lab[k * HW + i] = l[k];
    }
}

hipError_t launch_init(int B, int H, int W, const float* rgbdm, const InitCams& cams, const int64_t* offsets,
                       const float* pred, const int32_t* use_pred, int64_t n, float* params, int32_t* ids,
                       int32_t obj_id, hipStream_t st) {
    const int chunk = init_chunk(H * W);
    hipLaunchKernelGGL(init_kernel, dim3((unsigned)((H * W + chunk - 1) / chunk), (unsigned)B), dim3(kInitThreads), 0,
                       st, H, W, chunk, rgbdm, cams, offsets, pred, use_pred,
                       n, params, ids, obj_id);
    return hipGetLastError();
}

hipError_t launch_labels(int B, int H, int W, const float* rgbdm, const InitCams& cams, const int64_t* offsets,
                         const float* params, int64_t n, float* labels, hipStream_t st) {
    const int chunk = init_chunk(H * W);
    hipLaunchKernelGGL(labels_kernel, dim3((unsigned)((H * W + chunk - 1) / chunk), (unsigned)B), dim3(kInitThreads), 0,
                       st, H, W, chunk, rgbdm, cams, offsets, params, n,
                       labels);
    return hipGetLastError();
}

}  // namespace net
}  // namespace dqo
