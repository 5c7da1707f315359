// Incremental update (Eq. (7)-(8)): unstable-pixel masks per object from a
// loss-mode render, and new Gaussians back-projected at those pixels.
#include <algorithm>

#include "dqo_device.hpp"

namespace dqo {

constexpr int kMaskThreads = 256;
constexpr int kDensThreads = 1024;

template <typename T>
struct IncCfg {
    T theta_alpha, theta_d, theta_c3;  // theta_c3 = 3 theta_c (the colour test compares the channel sum)
    T eta_og, eta_tg;                  // opacity logits of OG and TG Gaussians
};

// View blockIdx.y, kMaskRounds pixels per thread.  The counts of a
// wavefront's pixels are taken object by object with ballots (neighbouring
// pixels show few objects), added up in LDS, then in the global counters
// (integers: the totals are exact).  Bound by its reads (36 B per pixel, 88 MB
// at 8 views of 640x480) once three things are gone that held it at 107 us:
// per-pixel LDS atomics, a 64-bit division per pixel, and global atomics of
// 256-pixel workgroups on the same few counters (4096 pixels: 31 us).
constexpr int kMaskRounds = 16;
template <typename T>
__global__ __launch_bounds__(kMaskThreads) void masks_kernel(int64_t HW, int K, const T* __restrict__ C,
                                                             const T* __restrict__ D, const T* __restrict__ pt,
                                                             const T* __restrict__ tc, const T* __restrict__ td,
                                                             const int32_t* __restrict__ tid, IncCfg<T> cfg,
                                                             uint8_t* __restrict__ masks,
                                                             int32_t* __restrict__ counts) {
    __shared__ int32_t s_cnt[DQO_MAX_K * 2];
    for (int k = threadIdx.x; k < 2 * K; k += kMaskThreads) s_cnt[k] = 0;
    __syncthreads();
    const int64_t v = blockIdx.y, p0 = v * HW;
    const T *C0 = C + 3 * p0, *tc0 = tc + 3 * p0;
    const int64_t base = (int64_t)blockIdx.x * (kMaskThreads * kMaskRounds);
    for (int r = 0; r < kMaskRounds; ++r) {
        const int64_t i = base + r * kMaskThreads + threadIdx.x;
        if (base + r * kMaskThreads >= HW) break;  // uniform
        int t = -1;
        bool geo = false, rgb = false;
        if (i < HW) {
            t = tid[p0 + i];
            const T dobs = td[p0 + i], d = D[p0 + i], q = pt[p0 + i];
            T e = T(0);
#pragma unroll
            for (int c = 0; c < 3; ++c) e += fabs(C0[c * HW + i] - tc0[c * HW + i]);
            if (t >= 0 && t < K) {
                geo = q < cfg.theta_alpha || (dobs > T(0) && fabs(d - dobs) > cfg.theta_d);
                rgb = e > cfg.theta_c3;
            }
            masks[p0 + i] = (uint8_t)((geo ? 1 : 0) | (rgb ? 2 : 0));
        }
        uint64_t todo = __ballot(geo || rgb);
        while (todo) {
            const int k = __shfl(t, __ffsll((unsigned long long)todo) - 1);
            const bool mine = t == k;
            const uint64_t bg = __ballot(mine && geo), br = __ballot(mine && rgb);
            if ((threadIdx.x & (kWave - 1)) == 0) {
                if (bg) atomicAdd(&s_cnt[2 * k], (int)__popcll(bg));
                if (br) atomicAdd(&s_cnt[2 * k + 1], (int)__popcll(br));
            }
            todo &= ~(bg | br);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < 2 * K; k += kMaskThreads)
        if (s_cnt[k]) atomicAdd(&counts[k], s_cnt[k]);
}

__device__ __forceinline__ bool spawns(uint8_t m, float d) { return m != 0 && d > 0.0f; }
__device__ __forceinline__ bool spawns(uint8_t m, double d) { return m != 0 && d > 0.0; }

// Densification splits each view into at most kDensChunks runs of pixels, a
// workgroup each.  A workgroup finds its first column from the views' totals
// (counts, pass 1) and by counting the pixels of its view in front of its run
// again: that is one mask byte per pixel, read 16 at a time, and the depth of
// the few pixels with a mask, and no scratch memory is needed.  More runs make
// a run shorter and the counting longer.  The write at 640x480 with 16, 32, 64,
// 128 and 256 runs per view: 8 views, a keyframe batch, 50, 37, 48, 59 and 70
// us; 2 views 47, 34, 25, 22 and 26; one view, whose 32 workgroups leave most
// of the CUs idle, 44, 32, 24, 21 and 20.
constexpr int kDensChunks = 32;
constexpr int kDensMinChunk = 1024;

inline int64_t dens_chunk(int64_t HW) {
    const int64_t per = (HW + kDensChunks - 1) / kDensChunks;
    return std::max<int64_t>(kDensMinChunk, (per + kDensThreads - 1) / kDensThreads * kDensThreads);
}

// This thread's share of the spawning pixels among the first n of a view.
template <typename T>
__device__ __forceinline__ int dens_count(const uint8_t* __restrict__ m, const T* __restrict__ d, int64_t n) {
    int c = 0;
    // bytes up to the first 16-byte boundary and past the last one, words between
    const int64_t lead = min(n, (int64_t)((16u - (uint32_t)((uintptr_t)m & 15u)) & 15u));
    const int64_t groups = (n - lead) / 16;
    if ((int64_t)threadIdx.x < lead) c += spawns(m[threadIdx.x], d[threadIdx.x]) ? 1 : 0;
    const int64_t tail = lead + 16 * groups + threadIdx.x;
    if (tail < n) c += spawns(m[tail], d[tail]) ? 1 : 0;
    const uint4* w = reinterpret_cast<const uint4*>(m + lead);
    constexpr int U = 4;
    for (int64_t g0 = threadIdx.x; g0 < groups; g0 += U * kDensThreads) {
        uint4 q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t g = g0 + u * kDensThreads;
            q[u] = g < groups ? w[g] : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!(q[u].x | q[u].y | q[u].z | q[u].w)) continue;
            const uint32_t x[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
            const T* dg = d + lead + 16 * (g0 + u * kDensThreads);
            T dv[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) dv[j] = dg[j];
#pragma unroll
            for (int j = 0; j < 16; ++j) c += spawns((uint8_t)(x[j >> 2] >> (8 * (j & 3))), dv[j]) ? 1 : 0;
        }
    }
    return c;
}

__device__ __forceinline__ int dens_wave_sum(int v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s);
    return v;
}

// Pass 1: the number of Gaussians each view adds (counts cleared before).
template <typename T>
__global__ __launch_bounds__(kDensThreads) void densify_count_kernel(int64_t HW, int64_t chunk,
                                                                     const uint8_t* __restrict__ masks,
                                                                     const T* __restrict__ td,
                                                                     int64_t* __restrict__ counts) {
    __shared__ int s_c;
    if (threadIdx.x == 0) s_c = 0;
    __syncthreads();
    const int64_t v = blockIdx.y, i0 = (int64_t)blockIdx.x * chunk;
    const int c = dens_wave_sum(dens_count<T>(masks + v * HW + i0, td + v * HW + i0, min(chunk, HW - i0)));
    if ((threadIdx.x & (kWave - 1)) == 0 && c) atomicAdd(&s_c, c);
    __syncthreads();
    if (threadIdx.x == 0 && s_c) atomicAdd((unsigned long long*)&counts[1 + v], (unsigned long long)s_c);
}

// Pass 2: each round takes kDensThreads consecutive pixels; a spawning pixel's
// column is the run's first plus its rank (wave ballots, then the waves'
// counts), so columns follow raster order and stores of a round coalesce.
// One workgroup per view, each thread on a contiguous run of pixels, took
// 1378 us at 8 views of 640x480; now 37 us (and pass 1 97 -> 5 us).
template <typename T>
__global__ __launch_bounds__(kDensThreads) void densify_write_kernel(Views<T> V, int64_t HW, int W, int64_t chunk,
                                                                     const uint8_t* __restrict__ masks,
                                                                     const T* __restrict__ tc,
                                                                     const T* __restrict__ td,
                                                                     const int32_t* __restrict__ tid, IncCfg<T> cfg,
                                                                     int64_t n_old, int64_t n_cap, T* __restrict__ params,
                                                                     int32_t* __restrict__ ids,
                                                                     int64_t* __restrict__ counts) {
    constexpr int kWaves = kDensThreads / kWave;
    __shared__ int s_w[2][kWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int v = blockIdx.y;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = min(HW, i0 + chunk);
    int64_t base = n_old;
    for (int u = 0; u < v; ++u) base += counts[1 + u];
    if (v == 0 && blockIdx.x == 0 && threadIdx.x == 0) {
        int64_t total = 0;
        for (int u = 0; u < V.n_views; ++u) total += counts[1 + u];
        counts[0] = total;
    }
    const int before = dens_wave_sum(dens_count<T>(masks + v * HW, td + v * HW, i0));
    if (lane == 0) s_w[0][wave] = before;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) base += s_w[0][w];
    const DevCam<T>& cam = V.cam[v];
    int buf = 1;
    for (int64_t r0 = i0; r0 < i1; r0 += kDensThreads, buf ^= 1) {
        const int64_t i = r0 + threadIdx.x;
        uint8_t m = 0;
        T d = T(0);
        if (i < i1) {
            m = masks[v * HW + i];
            d = td[v * HW + i];
        }
        const bool go = spawns(m, d);
        const uint64_t bal = __ballot(go);
        if (lane == 0) s_w[buf][wave] = (int)__popcll(bal);
        __syncthreads();  // the other buffer's readers are a barrier behind
        int64_t col = base + (int)__popcll(bal & (lane ? (~0ull >> (kWave - lane)) : 0ull));
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int c = s_w[buf][w];
            col += w < wave ? c : 0;
            base += c;
        }
        if (!go || col < n_old || col >= n_cap) continue;
        const int py = (int)(i / W), px = (int)(i - (int64_t)py * W);
        const T xc0 = d * ((T(px) + T(0.5) - cam.cx) / cam.fx) - cam.t[0];
        const T xc1 = d * ((T(py) + T(0.5) - cam.cy) / cam.fy) - cam.t[1];
        const T xc2 = d - cam.t[2];
        const T* R = cam.R;
        T vals[kParams];
        vals[0] = R[0] * xc0 + R[3] * xc1 + R[6] * xc2;  // R^T (x_c - t)
        vals[1] = R[1] * xc0 + R[4] * xc1 + R[7] * xc2;
        vals[2] = R[2] * xc0 + R[5] * xc1 + R[8] * xc2;
        vals[3] = vals[4] = vals[5] = log(d / cam.fx);
        vals[6] = T(1);
        vals[7] = vals[8] = vals[9] = T(0);
        vals[10] = (m & 1) ? cfg.eta_og : cfg.eta_tg;
        vals[11] = tc[(v * 3 + 0) * HW + i];
        vals[12] = tc[(v * 3 + 1) * HW + i];
        vals[13] = tc[(v * 3 + 2) * HW + i];
#pragma unroll
        for (int r = 0; r < kParams; ++r) params[(int64_t)r * n_cap + col] = vals[r];
        ids[col] = tid[v * HW + i];
    }
}

template <typename T>
IncCfg<T> inc_cfg(const dqo_increment_cfg& c) {
    IncCfg<T> g;
    g.theta_alpha = (T)c.theta_alpha;
    g.theta_d = (T)c.theta_d;
    g.theta_c3 = (T)(3.0 * c.theta_c);
    g.eta_og = (T)log(c.og_opacity / (1.0 - c.og_opacity));
    g.eta_tg = (T)log(c.tg_opacity / (1.0 - c.tg_opacity));
    return g;
}

template <typename T>
hipError_t launch_incremental_masks(const Frame<T>& f, const dqo_images& img, const dqo_targets& tgt,
                                    const dqo_increment_cfg& cfg, uint8_t* masks, int32_t* counts, hipStream_t st) {
    const int64_t HW = (int64_t)f.views.W * f.views.H;
    hipError_t e = launch_zero_words((uint32_t*)counts, 2 * (int64_t)f.K, st);
    if (e != hipSuccess) return e;
    if (HW * f.views.n_views == 0) return hipSuccess;
    hipLaunchKernelGGL(masks_kernel<T>,
                       dim3((unsigned)((HW + kMaskThreads * kMaskRounds - 1) / (kMaskThreads * kMaskRounds)),
                            (unsigned)f.views.n_views),
                       dim3(kMaskThreads), 0, st, HW, f.K, (const T*)img.color, (const T*)img.depth,
                       (const T*)img.p_target, (const T*)tgt.color, (const T*)tgt.depth, tgt.id, inc_cfg<T>(cfg), masks, counts);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_densify(const Frame<T>& f, const dqo_targets& tgt, const uint8_t* masks,
                          const dqo_increment_cfg& cfg, int64_t n_old, int64_t n_cap, T* params, int32_t* ids,
                          int64_t* counts, hipStream_t st) {
    const int64_t HW = (int64_t)f.views.W * f.views.H;
    const int V = f.views.n_views;
    const int64_t chunk = dens_chunk(HW);
    const dim3 grid((unsigned)((HW + chunk - 1) / chunk), (unsigned)V);
    hipError_t e = launch_zero_words((uint32_t*)counts, 2 * ((int64_t)V + 1), st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(densify_count_kernel<T>, grid, dim3(kDensThreads), 0, st, HW, chunk, masks,
                       (const T*)tgt.depth, counts);
    hipLaunchKernelGGL(densify_write_kernel<T>, grid, dim3(kDensThreads), 0, st, f.views, HW, f.views.W, chunk, masks,
                       (const T*)tgt.color, (const T*)tgt.depth, tgt.id, inc_cfg<T>(cfg), n_old, n_cap, params,
                       ids, counts);
    return hipGetLastError();
}

template hipError_t launch_incremental_masks<float>(const Frame<float>&, const dqo_images&, const dqo_targets&,
                                                    const dqo_increment_cfg&, uint8_t*, int32_t*, hipStream_t);
template hipError_t launch_incremental_masks<double>(const Frame<double>&, const dqo_images&, const dqo_targets&,
                                                     const dqo_increment_cfg&, uint8_t*, int32_t*, hipStream_t);
template hipError_t launch_densify<float>(const Frame<float>&, const dqo_targets&, const uint8_t*,
                                          const dqo_increment_cfg&, int64_t, int64_t, float*, int32_t*, int64_t*,
                                          hipStream_t);
template hipError_t launch_densify<double>(const Frame<double>&, const dqo_targets&, const uint8_t*,
                                           const dqo_increment_cfg&, int64_t, int64_t, double*, int32_t*, int64_t*,
                                           hipStream_t);

}  // namespace dqo
