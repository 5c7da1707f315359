// Tile rasterization: forward alpha blending and its adjoint.
//
// The unit of work is a wavefront on 8 x 8 pixels, one lane per pixel.  A tile
// (8x8, 16x8, 16x16, 32x8 or 8x32: the granularity of the binning) has one to
// four such parts.  In the forward each part is a workgroup of its own that
// streams the tile's sorted pair range through LDS in batches of 64 records,
// keeps those that can contribute in its 8 x 8 pixels and walks them from LDS
// (broadcast reads); it never waits for the other parts.  Blending is a
// per-pixel recurrence, not a dense contraction, so this path is VALU and
// transcendental bound and uses no matrix cores.
//
// The inner loops are written without divergent branches: every lane computes
// the contribution test, non-contributing lanes carry a zero weight, and whole
// steps are skipped only when the entire wavefront agrees (ballots), so the
// per-pair cost is a straight line of VALU work instead of exec-mask juggling.
//
// The forward keeps only T_final and the position of the last blended
// Gaussian per pixel.  The backward walks each pixel from that position back to
// the front of its tile's range, recomputing alpha exactly as the forward did
// and the transmittance by division (T_i = T_{i+1} / (1 - alpha_i)).  One
// wavefront takes all parts of a tile (a lane holds a pixel of each), so a
// Gaussian's gradients are summed over the parts in the lane first and then
// once over the wavefront: six Gaussians x ten values are transposed-and-summed
// across the 64 lanes (each lane ends up owning one value) and written once
// per (tile, Gaussian) pair to its own slot, which is marked written (pairs
// left unwritten count as zero); the per-Gaussian totals are formed later in a
// fixed order, so no atomics and no barriers are needed and the result is
// deterministic.
#include "dqo_device.hpp"

namespace dqo {

template <typename T>
__device__ __forceinline__ T fmadd(T a, T b, T c) { return fma(a, b, c); }

__device__ __forceinline__ bool wave_any(bool p) { return __ballot(p) != 0ull; }

// Walk records: what the render kernels keep in LDS for each pair of a batch,
// the splat restated in the coordinates of the pair's tile.  With (du, dv) a
// pixel centre's offset from the splat's mean, the pixel's alpha before the
// clamp is 2^E with E = a du^2 + 2b du dv + c dv^2 + log2(o): the conic of
// Eq. (12)'s Gaussian scaled by -log2(e)/2 and the opacity folded in.  A
// pair contributes at a pixel exactly when E reaches the record's threshold,
// max(log2 o - q_max log2(e)/2, log2 alpha_min), which is Q <= q_max and
// alpha >= alpha_min at once.  Forward and backward evaluate E with the same
// code from the same record, so both take the same decisions.
//   [0, 1] mean relative to the tile's corner (mu, mv); [2, 3, 4] a, b, c;
//   [5] log2 o; [6] threshold; [7] the pair's position; [8] depth; [9] object
//   id; [10, 11, 12] colour; [13..15] unused.
constexpr int kWalkWords = 16;
enum WalkWord { kWMu = 0, kWMv = 1, kWA = 2, kWM = 3, kWC = 4, kWLop = 5, kWThr = 6, kWPos = 7, kWZ = 8,
                kWId = 9, kWR = 10, kWG = 11, kWB = 12 };
template <typename T>
__device__ __forceinline__ T neg_half_log2e() { return T(-0.72134752044448170368); }

template <typename T>
__device__ __forceinline__ T log2_of(T x);
template <>
__device__ __forceinline__ float log2_of<float>(float x) { return log2f(x); }
template <>
__device__ __forceinline__ double log2_of<double>(double x) { return log2(x); }
template <typename T>
__device__ __forceinline__ T exp2_of(T x);
template <>
__device__ __forceinline__ float exp2_of<float>(float x) { return __builtin_amdgcn_exp2f(x); }
template <>
__device__ __forceinline__ double exp2_of<double>(double x) { return exp2(x); }

// Walk record of splat record r (mx, my, A, B, C, o, z, id, r, g, b) for the
// tile whose first pixel's corner is (ox, oy), stored at dst (LDS).
template <typename T>
__device__ __forceinline__ void store_walk_record(T* dst, const T (&r)[kRecWords], T ox, T oy, int pos,
                                                  const Consts<T>& cs) {
    const T kq = neg_half_log2e<T>();
    const T lop = log2_of<T>(r[5]);
    T w[kWalkWords];
    w[kWMu] = r[0] - ox;
    w[kWMv] = r[1] - oy;
    w[kWA] = kq * r[2];
    w[kWM] = kq * r[3];
    w[kWC] = kq * r[4];
    w[kWLop] = lop;
    w[kWThr] = max(fmadd(kq, cs.q_max, lop), log2_of<T>(cs.alpha_min));
    w[kWPos] = id_to_word<T>(pos);
    w[kWZ] = r[6];
    w[kWId] = r[7];
    w[kWR] = r[8];
    w[kWG] = r[9];
    w[kWB] = r[10];
    w[13] = w[14] = w[15] = T(0);
    if constexpr (sizeof(T) == 4) {
        float4* d4 = reinterpret_cast<float4*>(dst);
#pragma unroll
        for (int q = 0; q < 4; ++q) d4[q] = make_float4(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < kWalkWords; ++k) dst[k] = w[k];
    }
}

// The exponent E at the pixel centre (u, v) of the tile (offsets from its
// corner), as du p + dv r + log2 o with (du, dv) its offset from the mean and
// (p, r) = (a du + b dv, b du + c dv), the scaled conic times (du, dv): half
// the gradient of E with respect to (du, dv), which the backward reuses.
template <typename T>
__device__ __forceinline__ T walk_exponent(const T* w, T u, T v, T& du, T& dv, T& p, T& r) {
    du = u - w[kWMu];
    dv = v - w[kWMv];
    p = fmadd(w[kWA], du, w[kWM] * dv);
    r = fmadd(w[kWC], dv, w[kWM] * du);
    return fmadd(du, p, fmadd(dv, r, w[kWLop]));
}

// The first kRecWords values of a splat record from global memory into
// registers; the pad value (word 11) is not loaded (set to zero).  Loading it
// into a register the compiler counts as free would make the next write of
// that register wait for the load, and with it for every load before.
template <typename T>
__device__ __forceinline__ void load_splat_global(T (&r)[kRecWords], const T* src) {
#pragma unroll
    for (int k = 0; k < kRecWords - 1; ++k) r[k] = src[k];
    r[kRecWords - 1] = T(0);
}
template <>
__device__ __forceinline__ void load_splat_global<float>(float (&r)[kRecWords], const float* src) {
    const float4* s4 = reinterpret_cast<const float4*>(src);
    const float4 a = s4[0], b = s4[1];
    const float3 c = *reinterpret_cast<const float3*>(src + 8);
    r[0] = a.x; r[1] = a.y; r[2] = a.z; r[3] = a.w;
    r[4] = b.x; r[5] = b.y; r[6] = b.z; r[7] = b.w;
    r[8] = c.x; r[9] = c.y; r[10] = c.z;
    r[11] = 0.0f;
}
// The walked values of a splat record and the slot of its (tile tx, ty) pair:
// the item's first slot plus the tile's place in its rectangle, row-major
// (the record's last four values, the same 64-byte line in FP32).
template <typename T>
__device__ __forceinline__ uint32_t load_splat_slot(T (&r)[kRecWords], const T* src, int tx, int ty) {
    load_splat_global<T>(r, src);
    const uint32_t base = (uint32_t)word_to_id<T>(src[kSpSlot]);
    const uint32_t xy = (uint32_t)word_to_id<T>(src[kSpRect]);
    const uint32_t w = (uint32_t)word_to_id<T>(src[kSpRectW]);
    return base + (uint32_t)(ty - (int)(xy >> 16)) * w + (uint32_t)(tx - (int)(xy & 0xFFFFu));
}
template <>
__device__ __forceinline__ uint32_t load_splat_slot<float>(float (&r)[kRecWords], const float* src, int tx, int ty) {
    load_splat_global<float>(r, src);
    const float3 t = *reinterpret_cast<const float3*>(src + kSpSlot);  // the pad after them is not loaded either
    const uint32_t base = __float_as_uint(t.x), xy = __float_as_uint(t.y), w = __float_as_uint(t.z);
    return base + (uint32_t)(ty - (int)(xy >> 16)) * w + (uint32_t)(tx - (int)(xy & 0xFFFFu));
}

// Whether a splat can contribute at any rendered pixel centre of a tile,
// whose centres lie in the box [bx0, bx1] x [by0, by1]: the smallest
// Mahalanobis form Q over the box (Q is convex: 0 where the mean lies in the
// box, else the least of the four edge minima, each edge's at its clamped
// stationary point) against q_max, and the largest alpha, o exp(-Q_min / 2),
// against alpha_min.  About a quarter of the (tile, Gaussian) pairs that the
// 3-sigma box puts in a tile fail it.  Both bounds keep a margin, so the
// per-pixel tests, evaluated in other arithmetic, can never accept a splat
// this rejects: skipping the rejected ones leaves every result bitwise the
// same (a rejected splat would carry zero weight at every pixel).
template <typename T>
__device__ __forceinline__ bool tile_may_contribute(const T (&sp)[kRecWords], int px0, int px1, int py0, int py1,
                                                    const Consts<T>& cs) {
    if (px0 > px1 || py0 > py1) return false;
    const T bx0 = T(px0) + T(0.5), bx1 = T(px1) + T(0.5), by0 = T(py0) + T(0.5), by1 = T(py1) + T(0.5);
    const T mx = sp[0], my = sp[1], A = sp[2], B = sp[3], C = sp[4];
    auto qf = [&](T dx, T dy) { return fmadd(A * dx, dx, fmadd(T(2) * B * dx, dy, C * dy * dy)); };
    // approximate reciprocals: they only move the clamped stationary points,
    // where Q is flat to first order, far inside the bounds' margins
    const T iA = fast_rcp<T>(A), iC = fast_rcp<T>(C);
    T q = T(0);
    if (!(mx >= bx0 && mx <= bx1 && my >= by0 && my <= by1)) {
        const T ex0 = bx0 - mx, ex1 = bx1 - mx, ey0 = by0 - my, ey1 = by1 - my;
        q = min(min(qf(ex0, min(max(-B * ex0 * iC, ey0), ey1)), qf(ex1, min(max(-B * ex1 * iC, ey0), ey1))),
                min(qf(min(max(-B * ey0 * iA, ex0), ex1), ey0), qf(min(max(-B * ey1 * iA, ex0), ex1), ey1)));
    }
    return q <= cs.q_max * T(1.001) + T(1e-3) && sp[5] * fast_exp<T>(T(-0.5) * q) >= cs.alpha_min * T(0.999);
}

// The pixels of a tile that are rendered (inside the image and the view's
// window): columns [px0, px1], rows [py0, py1] (empty when px0 > px1 or
// py0 > py1).  Wave-uniform integers.
template <typename T>
__device__ __forceinline__ void tile_pixel_box(const Views<T>& V, int view, int tx, int ty, int TW, int TH, int& px0,
                                               int& px1, int& py0, int& py1) {
    const DevCam<T>& c = V.cam[view];
    px0 = max(tx * TW, c.win_x0);
    px1 = min(tx * TW + TW, c.win_x1) - 1;
    py0 = max(ty * TH, c.win_y0);
    py1 = min(ty * TH + TH, c.win_y1) - 1;
}

// Number of set bits of a wave-wide ballot below this lane.
__device__ __forceinline__ int rank_below(uint64_t bal) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
}

// Records whose contribution tests are evaluated together (FP32; FP64 keeps 4
// to bound register use).
#ifndef DQO_FWD_GROUP
#define DQO_FWD_GROUP 8
#endif
template <typename T>
constexpr int fwd_group() { return (sizeof(T) == 8 && DQO_FWD_GROUP > 4) ? 4 : DQO_FWD_GROUP; }

// The 64-pixel parts of a tile: part q covers columns 8 (q mod kAcross) .. + 7
// and rows 8 (q / kAcross) .. + 7 of the tile.
template <int TW, int TH>
struct Parts {
    static constexpr int kCount = TW * TH / kWave, kAcross = TW / 8;
    static_assert(TW % 8 == 0 && TH % 8 == 0 && kCount >= 1 && kCount <= 4, "8 x 8 pixel parts");
    __device__ static int x0(int q) { return 8 * (q % kAcross); }
    __device__ static int y0(int q) { return 8 * (q / kAcross); }
};

// PROBS: with the instance channels (an LDS column per lane); NB: with the
// per-pixel blend count.  Workgroup b runs on XCD b mod 8: the parts of a tile, which gather the same
// records, are consecutive workgroups of one XCD.
// One workgroup per tile with its waves in step (a barrier per batch, every
// wave walking every record that touches the tile) took 202 us on 30k
// Gaussians at 333x251 in 16x16 tiles with instance channels, 593 us on eight
// keyframes of 1.2M in 16x8 tiles; with a workgroup per part 110 and 414 us.
template <typename T, int TW, int TH, bool PROBS, bool NB = true>
__global__ __launch_bounds__(kWave) void render_forward_kernel(
    Views<T> V, Consts<T> cs, int K, const T* __restrict__ splats, uint32_t* __restrict__ pvals,
    const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ schedule, T* __restrict__ color, T* __restrict__ depth, T* __restrict__ tfinal,
    int32_t* __restrict__ last, T* __restrict__ probs, int32_t* __restrict__ idmap,
    const int32_t* __restrict__ target, T* __restrict__ ptarget, int32_t* __restrict__ nblend, uint32_t cap,
    uint32_t M, T* __restrict__ ckpt, uint32_t ckpt_cap,
    int32_t* __restrict__ tile_last, const uint32_t* __restrict__ seg_base, uint4* __restrict__ seg_list,
    uint32_t seg_cap, uint32_t seg_len, Ctrl* __restrict__ ctrl) {
    using P = Parts<TW, TH>;
    constexpr int BLOCK = kWave;
    if constexpr (P::kCount == 1) seg_len = kSegLen;
    __shared__ __align__(16) T s_sp[BLOCK * kWalkWords];
    extern __shared__ unsigned char s_dyn[];
    T* s_P = reinterpret_cast<T*>(s_dyn);  // [K][BLOCK] when PROBS

    const int tid = threadIdx.x;
    const uint32_t n_tiles = (uint32_t)(V.n_views * V.tiles_per_view);
    uint32_t rank = blockIdx.x;
    int part = 0;
    if constexpr (P::kCount > 1) {
        const uint32_t x = blockIdx.x % 8u, r = blockIdx.x / 8u;
        part = (int)(r % P::kCount);
        rank = (r / P::kCount) * 8u + x;
        if (rank >= n_tiles) return;
    }
    const int tile = (int)min(schedule[rank], n_tiles - 1u);
    const int view = tile / V.tiles_per_view;
    const int t = tile - view * V.tiles_per_view;
    const int ty = t / V.tiles_x, tx = t - ty * V.tiles_x;
    const int lx = P::x0(part) + (tid & 7), ly = P::y0(part) + (tid >> 3);  // in the tile
    const int px = tx * TW + lx, py = ty * TH + ly;
    // pixels of the image outside the view's window are written as empty
    const bool in_img = px < V.W && py < V.H;
    const bool inside = in_img && in_window(V.cam[view], px, py);
    const int64_t HW = (int64_t)V.W * V.H;
    const int64_t pix = (int64_t)py * V.W + px;
    // the pixel centre relative to the tile's corner
    const T u = T(lx) + T(0.5), v = T(ly) + T(0.5);
    const T ox = T(tx * TW), oy = T(ty * TH);
    const uint32_t re = min(ranges[2 * tile + 1], cap), rs = min(ranges[2 * tile], re);
    const uint32_t sbase = ckpt ? seg_base[tile] : 0u;  // used at the end
    int tgt = -2;
    if (target && in_img) tgt = job_target(V.cam[view].job, target[view * HW + pix]);
    if constexpr (PROBS)
        for (int k = 0; k < K; ++k) s_P[k * BLOCK + tid] = T(0);

    T Tt = T(1), c0 = T(0), c1 = T(0), c2 = T(0), dd = T(0), pt = T(0);
    int lastpos = -1, nb_count = 0;
    bool done = !inside;
    int bx0, bx1, by0, by1;
    tile_pixel_box<T>(V, view, tx, ty, TW, TH, bx0, bx1, by0, by1);
    const int tx0 = bx0, tx1 = bx1, ty0 = by0, ty1 = by1;  // the tile's pixels; from here on the part's
    if constexpr (P::kCount > 1) {
        bx0 = max(bx0, tx * TW + P::x0(part));
        bx1 = min(bx1, tx * TW + P::x0(part) + 7);
        by0 = max(by0, ty * TH + P::y0(part));
        by1 = min(by1, ty * TH + P::y0(part) + 7);
    }
    // Software prefetch: this lane's record of the next batch is loaded into
    // registers while the current batch is walked; the pair index one batch
    // further ahead is loaded one step earlier still.
    T pf[kRecWords];
    uint32_t pv = (rs + tid < re) ? pvals[rs + tid] : 0u, rec2 = 0u;
    if (rs + tid < re) load_splat_global<T>(pf, splats + (size_t)min(pv & kPairItem, M - 1) * kSplatWords);
    // (the index is masked and clamped where it is used: doing it here would
    // wait for the load, and with it for every load issued before)
    if (rs + BLOCK + tid < re) rec2 = pvals[rs + BLOCK + tid];
    for (uint32_t b0 = rs; b0 < re; b0 += BLOCK) {
        if (!wave_any(!done)) break;
        {
            // State before each segment boundary of the pair range, for the
            // segmented backward (which restarts there).
            const uint32_t rel = b0 - rs;
            if (ckpt && rel > 0 && (rel & (seg_len - 1u)) == 0 && rel / seg_len < (uint32_t)kSegMax) {
                const uint32_t e = boundary_record(rs, rel / seg_len, seg_len);
                if (e < ckpt_cap) {
                    T* c = ckpt + ((size_t)e * P::kCount + part) * 6 * kWave + tid;
                    c[0 * kWave] = Tt;
                    c[1 * kWave] = c0;
                    c[2 * kWave] = c1;
                    c[3 * kWave] = c2;
                    c[4 * kWave] = dd;
                    c[5 * kWave] = pt;
                }
            }
        }
        // The batch's records that may contribute somewhere in the part, in
        // order, compacted into LDS with their positions in the pad word.
        const bool live = b0 + tid < re;
        const bool cand = live && tile_may_contribute<T>(pf, bx0, bx1, by0, by1, cs);
        // those that cannot contribute in the whole tile are marked for the
        // backward, which then skips them (part 0 looks at the whole tile)
        if (part == 0 && live && !cand && !(pv & kPairSkip)) {
            bool none = true;
            if constexpr (P::kCount > 1) none = !tile_may_contribute<T>(pf, tx0, tx1, ty0, ty1, cs);
            if (none) pvals[b0 + tid] = pv | kPairSkip;
        }
        const uint64_t bal = __ballot(cand);
        const int nb = __popcll(bal);
        __syncthreads();
        if (cand) store_walk_record<T>(s_sp + rank_below(bal) * kWalkWords, pf, ox, oy, (int)(b0 + tid), cs);
        __syncthreads();
        pv = rec2;
        if (b0 + BLOCK + tid < re) load_splat_global<T>(pf, splats + (size_t)min(pv & kPairItem, M - 1) * kSplatWords);
        if (b0 + 2 * BLOCK + tid < re) rec2 = pvals[b0 + 2 * BLOCK + tid];
        // Groups of fwd_group<T>() records: their contribution tests (exponent,
        // exponential, threshold) are independent and evaluated side
        // by side, which hides the VALU and LDS latency that one wavefront
        // per SIMD would otherwise expose; only the transmittance recurrence
        // then runs serially, in depth order, with the same arithmetic as a
        // one-by-one walk.
        constexpr int kFwdGroup = fwd_group<T>();
        for (int j0 = 0; j0 < nb; j0 += kFwdGroup) {
            // the test words (and positions) of the group first; the blending
            // words are read only where the group has a contribution
            T rec[kFwdGroup][kWPos + 1];
            T a0[kFwdGroup];
            bool c0k[kFwdGroup];
            bool any = false;
#pragma unroll
            for (int k = 0; k < kFwdGroup; ++k) {
                const T* w = s_sp + min(j0 + k, nb - 1) * kWalkWords;
#pragma unroll
                for (int q = 0; q <= kWPos; ++q) rec[k][q] = w[q];
            }
#pragma unroll
            for (int k = 0; k < kFwdGroup; ++k) {
                T dx, dy, pp, rr;
                const T E = walk_exponent(rec[k], u, v, dx, dy, pp, rr);
                a0[k] = min(exp2_of<T>(E), cs.alpha_max);
                c0k[k] = (j0 + k < nb) && (E >= rec[k][kWThr]);
                any = any || c0k[k];
            }
            if (!wave_any(any && !done)) continue;
            T bl[kFwdGroup][kWB - kWZ + 1];  // depth, id, colour of each record
#pragma unroll
            for (int k = 0; k < kFwdGroup; ++k) {
                const T* w = s_sp + min(j0 + k, nb - 1) * kWalkWords;
#pragma unroll
                for (int q = kWZ; q <= kWB; ++q) bl[k][q - kWZ] = w[q];
            }
            // (taken as written here: the reads are issued together and
            // waited for once, not one record at a time inside the recurrence)
#pragma unroll
            for (int k = 0; k < kFwdGroup; ++k)
#pragma unroll
                for (int q = 0; q <= kWB - kWZ; ++q) asm volatile("" : "+v"(bl[k][q]));
#pragma unroll
            for (int k = 0; k < kFwdGroup; ++k) {
                const T* bw = bl[k] - kWZ;
                const bool contrib = c0k[k] && !done;
                const T a = contrib ? a0[k] : T(0);
                const T Tn = Tt * (T(1) - a);
                const bool stop = contrib && (Tn < cs.t_min);
                const T w = stop ? T(0) : a * Tt;
                c0 = fmadd(w, bw[kWR], c0);
                c1 = fmadd(w, bw[kWG], c1);
                c2 = fmadd(w, bw[kWB], c2);
                dd = fmadd(w, bw[kWZ], dd);
                const int id = word_to_id<T>(bw[kWId]);
                pt += (id == tgt) ? w : T(0);
                const bool blended = w != T(0);
                lastpos = blended ? word_to_id<T>(rec[k][kWPos]) : lastpos;
                if constexpr (NB) nb_count += blended ? 1 : 0;
                // (only the lanes that blend: as an LDS atomic add of every
                // lane, which nothing would wait for, it made the forward three
                // times slower, and as registers indexed by the object 1.4 times)
                if (PROBS && blended && id >= 0 && id < K) s_P[id * BLOCK + tid] += w;
                Tt = stop ? Tt : Tn;
                done = done || stop;
            }
            if (!wave_any(!done)) break;
        }
    }
    if (ckpt) {
        // The part's last blended position: how far its backward has work.
        int m = lastpos;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = max(m, __shfl_xor(m, d));
        if (tid == 0) tile_last[tile * P::kCount + part] = m;
        // The tile's entries of the backward's segment list, at the place the
        // sort reserved for its segments: the segment, the end of its walk
        // and the boundary record at its end (none for the range's last).
        // With one part the walk ends one past the last blended position where
        // that lies in the segment (then nothing restarts at its end), and
        // the segments behind are marked empty (no walk); with several, the
        // backward takes the end from the parts' last positions.
        const uint32_t nseg = tile_segments(re - rs, seg_len);
        constexpr bool kTrim = P::kCount == 1;
        const uint32_t k = !kTrim ? nseg
                           : (m >= (int)rs && m < (int)re) ? min(((uint32_t)m - rs) / seg_len + 1u, nseg)
                                                           : 0u;
        const uint32_t last_end = kTrim ? (uint32_t)m + 1u : 0xFFFFFFFFu;
        for (uint32_t j = (uint32_t)tid; part == 0 && j < nseg; j += kWave) {
            const uint32_t pos = sbase + j;
            if (pos >= seg_cap) break;
            const uint32_t s0 = rs + j * seg_len;
            const bool tail = j + 1u >= nseg;  // the last segment takes the rest of the range
            const uint32_t s1 = tail ? re : s0 + seg_len;
            const bool past = !tail && last_end > s1;
            seg_list[pos] = j < k ? make_uint4((uint32_t)tile, s0, min(last_end, s1),
                                               past ? boundary_record(rs, j + 1u, seg_len) : kNoBoundary)
                                  : make_uint4((uint32_t)tile, 0u, 0u, kNoBoundary);
        }
        if (blockIdx.x == 0 && tid == 0) {
            // the forward these states belong to (checked by the backward)
            ctrl->seg_stamp[0] = ctrl->epoch;
            ctrl->seg_stamp[1] = (uint64_t)(uintptr_t)last;
            ctrl->seg_stamp[2] = (uint64_t)(uintptr_t)target;
        }
    }
    if (!in_img) return;
    const int64_t o = view * HW + pix;
    color[(view * 3 + 0) * HW + pix] = c0 + Tt * cs.bg[0];
    color[(view * 3 + 1) * HW + pix] = c1 + Tt * cs.bg[1];
    color[(view * 3 + 2) * HW + pix] = c2 + Tt * cs.bg[2];
    depth[o] = dd;
    tfinal[o] = Tt;
    last[o] = lastpos;
    if (NB && nblend) nblend[o] = nb_count;
    if (ptarget && target) ptarget[o] = (tgt == -1) ? Tt : pt;
    if constexpr (PROBS) {
        int best = K;
        T bv = Tt;
        for (int k = K - 1; k >= 0; --k) {
            const T pk = s_P[k * BLOCK + tid];
            probs[((int64_t)view * K + k) * HW + pix] = pk;
            if (pk >= bv) {
                bv = pk;
                best = k;
            }
        }
        if (idmap) idmap[o] = (best == K) ? -1 : best;
    }
}

// ---------------------------------------------------------------- backward
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;  // pair slot of a record that is not loaded
constexpr int kChunk = 6;  // Gaussians per transposed reduction (6 x 10 = 60 of 64 lanes)

template <typename T, int D, int M>
__device__ __forceinline__ void butterfly_step(T (&v)[64], int lane) {
    const bool up = (lane & D) != 0;
#pragma unroll
    for (int i = 0; i < M / 2; ++i) {
        const T send = up ? v[i] : v[i + M / 2];
        const T keep = up ? v[i + M / 2] : v[i];
        v[i] = keep + __shfl_xor(send, D);
    }
}

// After the call, v[0] of lane L holds the sum over the wave of value L.
template <typename T>
__device__ __forceinline__ void wave_transpose_sum(T (&v)[64], int lane) {
    butterfly_step<T, 32, 64>(v, lane);
    butterfly_step<T, 16, 32>(v, lane);
    butterfly_step<T, 8, 16>(v, lane);
    butterfly_step<T, 4, 8>(v, lane);
    butterfly_step<T, 2, 4>(v, lane);
    butterfly_step<T, 1, 2>(v, lane);
}

// FP32 on gfx950.  The two cross-row levels use v_permlane32_swap /
// v_permlane16_swap: swapping the upper half of x = v[i] with the lower half of
// y = v[i + M/2] and adding the two results leaves, in every lane, the pair sum
// of exactly the value that lane keeps (one swap and one add per value pair).
// The in-row levels pair lanes with DPP row_mirror (lane ^ 15), row_half_mirror
// (lane ^ 7) and quad_perm (lane ^ 2, lane ^ 1); with 32 and 16 these masks are
// linearly independent, so each lane still sums all 64 lanes once, and the lane
// bit that selects the kept half is the same as in the XOR butterfly.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

template <int CTRL, int D, int M>
__device__ __forceinline__ void dpp_step(float (&v)[64], int lane) {
    const bool up = (lane & D) != 0;
#pragma unroll
    for (int i = 0; i < M / 2; ++i) {
        const float send = up ? v[i] : v[i + M / 2];
        const float keep = up ? v[i + M / 2] : v[i];
        v[i] = keep + dpp_mov<CTRL>(send);
    }
}

template <>
__device__ __forceinline__ void wave_transpose_sum<float>(float (&v)[64], int lane) {
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 32]), false,
                                                        false);
        v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 16]), false,
                                                        false);
        v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    dpp_step<0x140, 8, 16>(v, lane);  // row_mirror: lane ^ 15
    dpp_step<0x141, 4, 8>(v, lane);   // row_half_mirror: lane ^ 7
    dpp_step<0x4E, 2, 4>(v, lane);    // quad_perm [2,3,0,1]: lane ^ 2
    dpp_step<0xB1, 1, 2>(v, lane);    // quad_perm [1,0,3,2]: lane ^ 1
}


// Backward for 64-pixel tiles: the workgroup is one wavefront, so the
// transposed wave sums are already the tile sums and no barrier is needed
// between chunks.  The conic words are summed without their constant factors
// (-1/2 on the two diagonal words, -1 on the mixed one), which the lane that
// stores a word's sum applies once.  Only Gaussians that contribute somewhere in the tile take a
// reduction slot: the walk finds the next contributing Gaussian, fills slot c
// (c = 0..5, a separate statically indexed code section each, so the slot
// values stay in fixed registers), and after six slots the wave transposes and
// sums them.  Pairs that take no slot are not written (unmarked: zero
// partials).  Every take writes all
// ten values of its slot, so nothing is cleared between chunks: the values
// past the NS filled slots are set to zero here, as constants.
template <int NS, typename T>
__device__ __forceinline__ void flush_slots(T (&v)[64], uint32_t chunk, T* __restrict__ partials,
                                            uint8_t* __restrict__ written, uint32_t cap) {
    // The lane's place in the transposed sums, derived here at each flush (an
    // opaque copy of the lane index keeps the compiler from hoisting it out
    // of the walk, where these values would only occupy registers).
    int lane = (int)__lane_id();
    asm volatile("" : "+v"(lane));
    const int lane_slot = (lane * 205) >> 11;  // lane / kGradWords for lane < 64
    const int word = lane - lane_slot * kGradWords;
#pragma unroll
    for (int k = NS * kGradWords; k < 64; ++k) v[k] = T(0);
    wave_transpose_sum<T>(v, lane);
    const uint32_t slot = (uint32_t)__shfl((int)chunk, lane_slot);
    if (lane < NS * kGradWords) {
        if (slot < cap) {
            const T factor = (word <= 1) ? T(1) / neg_half_log2e<T>()
                             : (word == 2 || word == 4) ? T(-0.5) : (word == 3) ? T(-1) : T(1);
            partials[(size_t)slot * kGradWords + word] = v[0] * factor;
            if (word == 0) written[slot] = 1;
        }
    }
}

// Sum of w dL/dw over a tile's segments behind boundary record bnd, which ends
// the segment [s0, s1) of a range starting at rs: records bnd, bnd + 1, ...
// up to the segment of the tile's last blended position (the range's segment
// kSegMax - 1 is its last).
template <typename T>
__device__ __forceinline__ T sum_of_later_segments(const T* __restrict__ sums, int stride, uint32_t bnd, uint32_t s0,
                                                   uint32_t s1, uint32_t rs, uint32_t seg_len, int tlast,
                                                   uint32_t ckpt_cap) {
    const uint32_t next = (s0 - rs) / seg_len + 1u;
    const uint32_t n = min(((uint32_t)tlast - s1) / seg_len, (uint32_t)kSegMax - 1u - next) + 1u;
    T a = T(0);
    for (uint32_t k = 0; k < n; ++k) a += sums[(size_t)min(bnd + k, ckpt_cap - 1u) * stride];
    return a;
}

#ifndef DQO_BWD_PARTS_OCC
#define DQO_BWD_PARTS_OCC 3
#endif
template <int C>
struct SlotIdx {
    static constexpr int value = C;
};

template <typename T, int TW, int TH, bool PROBS, bool PREFETCH>
__device__ __forceinline__ void backward_unit(
    const Views<T>& V, const Consts<T>& cs, int K, const T* __restrict__ splats,
    const uint32_t* __restrict__ pvals, const uint32_t* __restrict__ ranges,
    const uint32_t* __restrict__ schedule, const T* __restrict__ tfinal, const int32_t* __restrict__ last,
    const int32_t* __restrict__ target, const T* __restrict__ dC, const T* __restrict__ dD, const T* __restrict__ dT,
    const T* __restrict__ dP, const T* __restrict__ dPt, T* __restrict__ partials, uint8_t* __restrict__ written,
    uint32_t cap, uint32_t M, const uint4* __restrict__ seg_list, const T* __restrict__ ckpt, uint32_t ckpt_cap,
    const T* __restrict__ color, const T* __restrict__ depth, const T* __restrict__ ptarget,
    const T* __restrict__ seg_sums, const int32_t* __restrict__ tile_last, T* s_sp, uint32_t* s_slot, uint32_t unit) {
    const int lane = threadIdx.x;
    const uint32_t n_tiles = (uint32_t)(V.n_views * V.tiles_per_view);
    // A listed segment comes with its walk [s0, hi) and the boundary record
    // at its end (pixels blending past s1 restart from it); a whole tile
    // walks its range up to its pixels' last blended position.
    int tile;
    uint32_t s0, s1, hi_seg = 0u, bnd = kNoBoundary;
    if (seg_list) {
        const uint4 en = seg_list[unit];
        if (en.z <= en.y) return;  // a segment behind its tile's last blended position (uniform)
        tile = (int)min(en.x, n_tiles - 1u);
        s0 = min(en.y, cap);
        hi_seg = min(max(en.z, s0), cap);
        bnd = en.w;
        s1 = (bnd == kNoBoundary) ? 0xFFFFFFFFu : s0 + (uint32_t)kSegLen;
    } else {
        tile = (int)min(schedule[unit], n_tiles - 1u);
        s0 = min(ranges[2 * tile], cap);
        s1 = min(ranges[2 * tile + 1], cap);
    }
    const int view = tile / V.tiles_per_view;
    const int t = tile - view * V.tiles_per_view;
    const int ty = t / V.tiles_x, tx = t - ty * V.tiles_x;
    const int px = tx * TW + (lane % TW), py = ty * TH + (lane / TW);
    const bool inside = px < V.W && py < V.H && in_window(V.cam[view], px, py);
    const int64_t HW = (int64_t)V.W * V.H;
    const int64_t pix = (int64_t)py * V.W + px;
    const int64_t o = view * HW + pix;
    // the pixel centre relative to the tile's corner
    const T u = T(lane % TW) + T(0.5), v_px = T(lane / TW) + T(0.5);
    const T ox = T(tx * TW), oy = T(ty * TH);

    // Batches of up to 64 pairs, from the walk's end down.  A listed
    // segment knows where its walk ends, so the first batch's pair indices
    // are loaded before the pixels' values, and its records (which need the
    // indices) right after them; the pixel values are used only then.
    auto batch_lo = [&](uint32_t e) { return (e - s0 > (uint32_t)kWave) ? e - kWave : s0; };
    uint32_t rec_first = 0u;
    if (seg_list && lane < (int)(hi_seg - batch_lo(hi_seg))) rec_first = pvals[batch_lo(hi_seg) + lane];

    int lastp = -1;
    T Tcur = T(1), gc0 = T(0), gc1 = T(0), gc2 = T(0), gd = T(0), gt = T(0), gpt = T(0);
    int tgt = -2, tgt_raw = -1;
    T ck[6] = {}, later = T(0), col0 = T(0), col1 = T(0), col2 = T(0), dep = T(0), ptg = T(0);
    if (inside) {
        lastp = last[o];
        Tcur = tfinal[o];
        gc0 = dC[(view * 3 + 0) * HW + pix];
        gc1 = dC[(view * 3 + 1) * HW + pix];
        gc2 = dC[(view * 3 + 2) * HW + pix];
        gd = dD ? dD[o] : T(0);
        gt = dT ? dT[o] : T(0);
        if (dPt && target) {
            tgt_raw = target[o];
            gpt = dPt[o];
        }
        if (bnd != kNoBoundary) {
            // Some pixels blend past this segment: they restart at its end
            // from the state the forward stored there (loaded for every
            // pixel, beside the values above).
            const T* c = ckpt + (size_t)min(bnd, ckpt_cap - 1u) * 6 * kWave + lane;
            ck[0] = c[0];
            if constexpr (PROBS) {
                later = sum_of_later_segments<T>(seg_sums + lane, kWave, bnd, s0, s1, ranges[2 * tile], kSegLen,
                                                 tile_last[tile], ckpt_cap);
            } else {
#pragma unroll
            for (int q = 1; q < 6; ++q) ck[q] = c[q * kWave];
            col0 = color[(view * 3 + 0) * HW + pix];
            col1 = color[(view * 3 + 1) * HW + pix];
            col2 = color[(view * 3 + 2) * HW + pix];
            dep = depth[o];
            ptg = ptarget ? ptarget[o] : T(0);
            }
        }
    }
    // A lane's record of a batch and its pair slot (kNoSlot: a pair the
    // forward marked as contributing nowhere in the tile, not loaded).
    T pf[kRecWords];
    uint32_t pf_slot = kNoSlot;
    auto load_pair = [&](uint32_t pv) {
        if (pv & kPairSkip) pf_slot = kNoSlot;
        else pf_slot = load_splat_slot<T>(pf, splats + (size_t)min(pv, M - 1) * kSplatWords, tx, ty);
    };
    if (seg_list && lane < (int)(hi_seg - batch_lo(hi_seg))) load_pair(rec_first);

    bool restart = false;
    T S_restart = T(0);
    if (inside) {
        // nothing in this segment (whole tiles: nothing of this frame's)
        if (lastp < (int)s0 || (!seg_list && lastp >= (int)s1)) lastp = -1;
        if (dPt && target) {
            tgt = job_target(V.cam[view].job, tgt_raw);
            if (tgt == -1) gt += gpt;
        }
        if (bnd != kNoBoundary) {
            // The sum behind the boundary is the total minus the part in front
            // of it (colour without the background term, depth, target
            // probability), or with instance channels the later segments' sums.
            if (lastp >= (int)s1) {
                const T Tf = Tcur;
                const T behind = PROBS ? later : gc0 * ((col0 - Tf * cs.bg[0]) - ck[1]) + gc1 * ((col1 - Tf * cs.bg[1]) - ck[2]) +
                                 gc2 * ((col2 - Tf * cs.bg[2]) - ck[3]) + gd * (dep - ck[4]) +
                                 (tgt >= 0 ? gpt * (ptg - ck[5]) : T(0));
                S_restart = behind + Tf * (gc0 * cs.bg[0] + gc1 * cs.bg[1] + gc2 * cs.bg[2] + gt);
                Tcur = ck[0];
                lastp = (int)s1 - 1;
                restart = true;
            }
        }
    }
    // Pairs behind every pixel's last blended Gaussian, and pairs that
    // contribute nowhere in the tile, are not written and stay unmarked
    // (their partials count as zero).
    uint32_t hi = hi_seg;
    if (!seg_list) {
        int maxlast = lastp;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) maxlast = max(maxlast, __shfl_xor(maxlast, d));
        // Equal in every lane; said so, the walk state derived from it lives
        // in scalar registers and the loop control is scalar branches
        // (measured 10% faster than the same walk with its state in vector
        // registers).
        maxlast = __builtin_amdgcn_readfirstlane(maxlast);
        hi = (maxlast >= (int)s0) ? (uint32_t)(maxlast + 1) : s0;
    }
    T S = restart ? S_restart : Tcur * (gc0 * cs.bg[0] + gc1 * cs.bg[1] + gc2 * cs.bg[2] + gt);
    T v[64];
#pragma unroll
    for (int k = 0; k < 64; ++k) v[k] = T(0);
    uint32_t chunk = 0u;  // lane c < kChunk: the pair slot of the Gaussian in reduction slot c
    // the target-probability gradient joins a Gaussian's colour sum where its
    // object is the pixel's target (tgt -1: T_final's gradient carries it)
    const T gpt_obj = tgt >= 0 ? gpt : T(0);
    // walk state (wave-uniform): the LDS batch holds positions [bstart, bend)
    uint32_t bend = hi, bstart = hi;
    int jl = -1;
    // contribution state of the Gaussian found by `next`, zero in the lanes
    // it does not blend: alpha, and alpha where it is not clamped (the factor
    // of alpha's derivatives)
    const T* sp = s_sp;
    T dx = T(0), dy = T(0), a = T(0), a_free = T(0), pp = T(0), rr = T(0);

    // The first batch is A = [a_s, a_e) (already loaded for a listed
    // segment).  With PREFETCH (whole tiles: many batches) the next batch's
    // records are held in registers while the current one is walked, and the
    // pair indices of the batch after it (B) are loaded one step earlier
    // still; without it (segments: mostly one batch) later batches are
    // loaded when reached, and the record registers are free during the walk.
    uint32_t a_e = hi, a_s = batch_lo(hi);
    if (!seg_list && lane < (int)(a_e - a_s)) load_pair(pvals[a_s + lane]);
    uint32_t b_e = a_s, b_s = batch_lo(a_s), rec_b = 0u;
    // (clamped where used, so that nothing waits for this load early)
    if constexpr (PREFETCH) rec_b = (lane < (int)(b_e - b_s)) ? pvals[b_s + lane] : 0u;
    bool first_batch = true;

    // The walk record of the Gaussian being tested, read from LDS (16-byte
    // broadcast reads at a 24-bit multiply of its index; the compiler issues
    // each where its values are first used).
    T cur[kWPos + 1];
    auto lds_rec = [&](int j) {
        if constexpr (sizeof(T) == 4) {
            const float4* s4 = reinterpret_cast<const float4*>(reinterpret_cast<const char*>(s_sp) +
                                                               __mul24(j, (int)(kWalkWords * sizeof(T))));
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float4 a = s4[q];
                cur[4 * q] = a.x;
                cur[4 * q + 1] = a.y;
                cur[4 * q + 2] = a.z;
                cur[4 * q + 3] = a.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k <= kWPos; ++k) cur[k] = s_sp[j * kWalkWords + k];
        }
    };
    // Advances to the next Gaussian (descending) that contributes at some pixel
    // of the tile; false at the end of the range.  The two wave-wide tests are
    // ballots of single comparisons combined as masks, which keeps them in
    // scalar instructions.
    auto next = [&]() -> bool {
        for (;;) {
            if (jl < 0) {
                if (a_e <= a_s) return false;
                bend = a_e;
                bstart = a_s;
                const int nbr = (int)(bend - bstart);
                if constexpr (!PREFETCH) {
                    if (!first_batch && lane < nbr) load_pair(pvals[bstart + lane]);
                    first_batch = false;
                }
                __syncthreads();
                // the records that may contribute in the tile (those the
                // forward did not mark), compacted in order
                const bool cand = lane < nbr && pf_slot != kNoSlot;
                const uint64_t bal = __builtin_amdgcn_ballot_w64(cand);
                if (cand) {
                    const int q = rank_below(bal);
                    store_walk_record<T>(s_sp + q * kWalkWords, pf, ox, oy, (int)(bstart + lane), cs);
                    s_slot[q] = pf_slot;
                }
                __syncthreads();
                jl = __popcll(bal) - 1;
                a_e = b_e;
                a_s = b_s;
                b_e = a_s;
                b_s = batch_lo(a_s);
                if constexpr (PREFETCH) {
                    if (lane < (int)(a_e - a_s)) load_pair(rec_b);
                    rec_b = (lane < (int)(b_e - b_s)) ? pvals[b_s + lane] : 0u;
                }
                if (jl < 0) continue;  // nothing in this batch can contribute
            }
            lds_rec(jl);
            sp = cur;
            const T E = walk_exponent(sp, u, v_px, dx, dy, pp, rr);
            const T araw = exp2_of<T>(E);
            const bool clamped = !(araw < cs.alpha_max);
            const T a0 = clamped ? cs.alpha_max : araw;  // min(araw, alpha_max), one select
            const bool contrib = (E >= sp[kWThr]) & (word_to_id<T>(sp[kWPos]) <= lastp);
            a = contrib ? a0 : T(0);
            if (__builtin_amdgcn_ballot_w64(a != T(0)) == 0ull) {
                --jl;
                continue;
            }
            a_free = clamped ? T(0) : a;
            return true;
        }
    };
    // Gradient of the found Gaussian into slot C; advances the walk.
    // In the lanes the Gaussian does not blend, a = 0 leaves T and S as they
    // are and zeroes every word (w = 0, a_free = 0).
    auto take = [&](auto cidx) {
        constexpr int C = decltype(cidx)::value;
        const T roma = fast_rcp<T>(T(1) - a);
        const T Ti = Tcur * roma;
        const T w = a * Ti;
        const T* bw = s_sp + jl * kWalkWords;  // the blending words
        const int id = word_to_id<T>(bw[kWId]);
        T vv = fmadd(gc0, bw[kWR], fmadd(gc1, bw[kWG], fmadd(gc2, bw[kWB], gd * bw[kWZ])));
        vv += (id == tgt) ? gpt_obj : T(0);
        if constexpr (PROBS) {
            if (a != T(0) && id >= 0 && id < K) vv += dP[((int64_t)view * K + id) * HW + pix];
        }
        const T dalpha = fmadd(Ti, vv, -(S * roma));
        S = fmadd(w, vv, S);
        Tcur = Ti;
        // dq = -2 dL/dQ: the mean words are dq (p, r) (the scaled conic
        // times the offset), the conic words dq dx^2, dq dx dy, dq dy^2, each
        // before its constant factor; the opacity word is dq = o dL/do
        const T dq = dalpha * a_free;
        const T t1 = dq * dx, t2 = dq * dy;
        v[C * kGradWords + 0] = dq * pp;
        v[C * kGradWords + 1] = dq * rr;
        v[C * kGradWords + 2] = t1 * dx;
        v[C * kGradWords + 3] = t1 * dy;
        v[C * kGradWords + 4] = t2 * dy;
        v[C * kGradWords + 5] = dq;
        v[C * kGradWords + 6] = gc0 * w;
        v[C * kGradWords + 7] = gc1 * w;
        v[C * kGradWords + 8] = gc2 * w;
        v[C * kGradWords + 9] = gd * w;
        const uint32_t pslot = s_slot[jl];
        chunk = (lane == C) ? pslot : chunk;
        --jl;
    };
    // Six slots: four and five (fewer registers, five waves per SIMD with
    // four) measured slower, the transposed sums then costing more per slot.
    constexpr int NS = kChunk;
    static_assert(NS >= 2 && NS <= 6, "reduction slots");
    for (;;) {
        if (!next()) break;
        take(SlotIdx<0>{});
        if (!next()) { flush_slots<1>(v, chunk, partials, written, cap); break; }
        take(SlotIdx<1>{});
        if constexpr (NS > 2) {
            if (!next()) { flush_slots<2>(v, chunk, partials, written, cap); break; }
            take(SlotIdx<2>{});
        }
        if constexpr (NS > 3) {
            if (!next()) { flush_slots<3>(v, chunk, partials, written, cap); break; }
            take(SlotIdx<3>{});
        }
        if constexpr (NS > 4) {
            if (!next()) { flush_slots<4>(v, chunk, partials, written, cap); break; }
            take(SlotIdx<4>{});
        }
        if constexpr (NS > 5) {
            if (!next()) { flush_slots<5>(v, chunk, partials, written, cap); break; }
            take(SlotIdx<5>{});
        }
        flush_slots<NS>(v, chunk, partials, written, cap);
    }
}

// The backward of a tile of several 64-pixel parts, by one wavefront: lane l
// holds pixel l of every part.  A record is read from LDS and controlled once
// for all parts, tested only on the parts that its bounds reach (a mask per
// record, found when the batch is staged), and the parts' gradients meet in the
// lane before the transposed sums, so those cost one part's work per Gaussian.
// With a workgroup of one wavefront per 64 pixels of the tile in step (every
// wave testing every record, sums over the waves through LDS with a barrier
// per six Gaussians) the backward of 30k Gaussians at 333x251 in 16x16 tiles
// took 445 us, of eight keyframes of 1.2M in 16x8 tiles 1375 us; now 66 (and 20 for
// the segments' sums of the instance channels) and 927 us.
template <typename T, int TW, int TH, bool PROBS, bool PREFETCH>
__device__ __forceinline__ void backward_parts(
    const Views<T>& V, const Consts<T>& cs, int K, const T* __restrict__ splats,
    const uint32_t* __restrict__ pvals, const uint32_t* __restrict__ ranges,
    const uint32_t* __restrict__ schedule, const T* __restrict__ tfinal, const int32_t* __restrict__ last,
    const int32_t* __restrict__ target, const T* __restrict__ dC, const T* __restrict__ dD, const T* __restrict__ dT,
    const T* __restrict__ dP, const T* __restrict__ dPt, T* __restrict__ partials, uint8_t* __restrict__ written,
    uint32_t cap, uint32_t M, const uint4* __restrict__ seg_list, const T* __restrict__ ckpt, uint32_t ckpt_cap,
    const T* __restrict__ color, const T* __restrict__ depth, const T* __restrict__ ptarget,
    const T* __restrict__ seg_sums, const int32_t* __restrict__ tile_last, uint32_t seg_len, T* s_sp, uint32_t* s_slot,
    uint32_t* s_mask, uint32_t unit) {
    using P = Parts<TW, TH>;
    constexpr int N = P::kCount;
    const int lane = threadIdx.x;
    const uint32_t n_tiles = (uint32_t)(V.n_views * V.tiles_per_view);
    int tile;
    uint32_t s0, s1, hi = 0u, bnd = kNoBoundary;
    int tlast = -1;
    if (seg_list) {
        const uint4 en = seg_list[unit];
        tile = (int)min(en.x, n_tiles - 1u);
        s0 = min(en.y, cap);
        s1 = min(max(en.z, s0), cap);
#pragma unroll
        for (int q = 0; q < N; ++q) tlast = max(tlast, tile_last[tile * N + q]);
        if (tlast < (int)s0) return;  // behind every pixel's last blended position (uniform)
        hi = min((uint32_t)tlast + 1u, s1);
        bnd = tlast >= (int)s1 ? en.w : kNoBoundary;
    } else {
        tile = (int)min(schedule[unit], n_tiles - 1u);
        s0 = min(ranges[2 * tile], cap);
        s1 = min(ranges[2 * tile + 1], cap);
    }
    const int view = tile / V.tiles_per_view;
    const int t = tile - view * V.tiles_per_view;
    const int ty = t / V.tiles_x, tx = t - ty * V.tiles_x;
    const int64_t HW = (int64_t)V.W * V.H;
    const T ox = T(tx * TW), oy = T(ty * TH);
    auto batch_lo = [&](uint32_t e) { return (e - s0 > (uint32_t)kWave) ? e - kWave : s0; };
    uint32_t rec_first = 0u;
    if (seg_list && lane < (int)(hi - batch_lo(hi))) rec_first = pvals[batch_lo(hi) + lane];

    int lastp[N], tgt[N];
    T Tcur[N], S[N], gc0[N], gc1[N], gc2[N], gd[N], gpt[N];
    int64_t at[N];
    int maxlast = -1;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int px = tx * TW + P::x0(q) + (lane & 7), py = ty * TH + P::y0(q) + (lane >> 3);
        const int64_t pix = (int64_t)py * V.W + px, o = view * HW + pix;
        at[q] = pix;
        lastp[q] = -1;
        tgt[q] = -2;
        Tcur[q] = T(1);
        S[q] = gc0[q] = gc1[q] = gc2[q] = gd[q] = gpt[q] = T(0);
        if (!(px < V.W && py < V.H && in_window(V.cam[view], px, py))) continue;
        lastp[q] = last[o];
        Tcur[q] = tfinal[o];
        gc0[q] = dC[(view * 3 + 0) * HW + pix];
        gc1[q] = dC[(view * 3 + 1) * HW + pix];
        gc2[q] = dC[(view * 3 + 2) * HW + pix];
        gd[q] = dD ? dD[o] : T(0);
        T gt = dT ? dT[o] : T(0);
        if (dPt && target) {
            tgt[q] = job_target(V.cam[view].job, target[o]);
            gpt[q] = dPt[o];
            if (tgt[q] == -1) gt += gpt[q];
        }
        if (lastp[q] < (int)s0 || (!seg_list && lastp[q] >= (int)s1)) lastp[q] = -1;
        const T Tf = Tcur[q];
        T behind = T(0);
        if (bnd != kNoBoundary && lastp[q] >= (int)s1) {
            // the pixel blends past this segment: it restarts at its end
            const uint32_t e = min(bnd, ckpt_cap - 1u);
            const T* c = ckpt + ((size_t)e * N + q) * 6 * kWave + lane;
            if constexpr (PROBS) {
                behind = sum_of_later_segments<T>(seg_sums + q * kWave + lane, N * kWave, bnd, s0, s1, ranges[2 * tile],
                                                  seg_len, tlast, ckpt_cap);
            } else {
                behind = gc0[q] * ((color[(view * 3 + 0) * HW + pix] - Tf * cs.bg[0]) - c[1 * kWave]) +
                         gc1[q] * ((color[(view * 3 + 1) * HW + pix] - Tf * cs.bg[1]) - c[2 * kWave]) +
                         gc2[q] * ((color[(view * 3 + 2) * HW + pix] - Tf * cs.bg[2]) - c[3 * kWave]) +
                         gd[q] * (depth[o] - c[4 * kWave]) +
                         (tgt[q] >= 0 ? gpt[q] * ((ptarget ? ptarget[o] : T(0)) - c[5 * kWave]) : T(0));
            }
            Tcur[q] = c[0];
            lastp[q] = (int)s1 - 1;
        }
        S[q] = behind + Tf * (gc0[q] * cs.bg[0] + gc1[q] * cs.bg[1] + gc2[q] * cs.bg[2] + gt);
        // the target-probability gradient joins a Gaussian's colour sum where
        // its object is the pixel's target (tgt -1: T_final's gradient carries it)
        if (tgt[q] < 0) gpt[q] = T(0);
        maxlast = max(maxlast, lastp[q]);
    }
    if (!seg_list) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) maxlast = max(maxlast, __shfl_xor(maxlast, d));
        maxlast = __builtin_amdgcn_readfirstlane(maxlast);  // uniform: scalar walk bounds
        hi = (maxlast >= (int)s0) ? (uint32_t)(maxlast + 1) : s0;
    }
    T pf[kRecWords];
    uint32_t pf_slot = kNoSlot;
    auto load_pair = [&](uint32_t pv) {
        if (pv & kPairSkip) pf_slot = kNoSlot;
        else pf_slot = load_splat_slot<T>(pf, splats + (size_t)min(pv, M - 1) * kSplatWords, tx, ty);
    };
    int bx0, bx1, by0, by1;
    tile_pixel_box<T>(V, view, tx, ty, TW, TH, bx0, bx1, by0, by1);

    T v[64];
#pragma unroll
    for (int k = 0; k < 64; ++k) v[k] = T(0);
    uint32_t chunk = 0u;
    int filled = 0;  // reduction slots in use
    uint32_t a_e = hi, a_s = batch_lo(hi);
    if (lane < (int)(a_e - a_s)) load_pair(seg_list ? rec_first : pvals[a_s + lane]);
    while (a_e > a_s) {
        const uint32_t bstart = a_s;
        const int nbr = (int)(a_e - a_s);
        uint32_t mask = 0u;
        if (lane < nbr && pf_slot != kNoSlot) {
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const int x0 = tx * TW + P::x0(q), y0 = ty * TH + P::y0(q);
                if (tile_may_contribute<T>(pf, max(bx0, x0), min(bx1, x0 + 7), max(by0, y0), min(by1, y0 + 7), cs))
                    mask |= 1u << q;
            }
        }
        __syncthreads();
        const uint64_t bal = __builtin_amdgcn_ballot_w64(mask != 0u);
        if (mask) {
            const int k = rank_below(bal);
            store_walk_record<T>(s_sp + k * kWalkWords, pf, ox, oy, (int)(bstart + lane), cs);
            s_slot[k] = pf_slot;
            s_mask[k] = mask;
        }
        __syncthreads();
        const int nb = __popcll(bal);
        const uint32_t mine = lane < nb ? s_mask[lane] : 0u;
        uint64_t reach[N];  // bit j: record j reaches part q
#pragma unroll
        for (int q = 0; q < N; ++q) reach[q] = __builtin_amdgcn_ballot_w64((mine >> q) & 1u);
        // the next batch (its records in flight during the walk with PREFETCH)
        a_e = a_s;
        a_s = batch_lo(a_s);
        uint32_t next_pv = 0u;
        if (lane < (int)(a_e - a_s)) next_pv = pvals[a_s + lane];
        if constexpr (PREFETCH) {
            if (lane < (int)(a_e - a_s)) load_pair(next_pv);
        }
        for (int jl = nb - 1; jl >= 0; --jl) {
            const T* rec = s_sp + jl * kWalkWords;
            T w[kWB + 1];
#pragma unroll
            for (int k = 0; k <= kWB; ++k) w[k] = rec[k];
            T g[kGradWords];
#pragma unroll
            for (int k = 0; k < kGradWords; ++k) g[k] = T(0);
            bool any = false;
            const int id = word_to_id<T>(w[kWId]), pos = word_to_id<T>(w[kWPos]);
#pragma unroll
            for (int q = 0; q < N; ++q) {
                if (!((reach[q] >> jl) & 1ull)) continue;  // uniform
                const T u = T(P::x0(q) + (lane & 7)) + T(0.5), vp = T(P::y0(q) + (lane >> 3)) + T(0.5);
                T dx, dy, pp, rr;
                const T E = walk_exponent(w, u, vp, dx, dy, pp, rr);
                const T araw = exp2_of<T>(E);
                const bool clamped = !(araw < cs.alpha_max);
                const bool contrib = (E >= w[kWThr]) & (pos <= lastp[q]);
                const T a = contrib ? (clamped ? cs.alpha_max : araw) : T(0);
                if (__builtin_amdgcn_ballot_w64(a != T(0)) == 0ull) continue;
                any = true;
                const T a_free = clamped ? T(0) : a;
                const T roma = fast_rcp<T>(T(1) - a);
                const T Ti = Tcur[q] * roma;
                const T wt = a * Ti;
                T vv = fmadd(gc0[q], w[kWR], fmadd(gc1[q], w[kWG], fmadd(gc2[q], w[kWB], gd[q] * w[kWZ])));
                vv += (id == tgt[q]) ? gpt[q] : T(0);
                if constexpr (PROBS) {
                    if (a != T(0) && id >= 0 && id < K) vv += dP[((int64_t)view * K + id) * HW + at[q]];
                }
                const T dalpha = fmadd(Ti, vv, -(S[q] * roma));
                S[q] = fmadd(wt, vv, S[q]);
                Tcur[q] = Ti;
                const T dq = dalpha * a_free;
                const T t1 = dq * dx, t2 = dq * dy;
                g[0] = fmadd(dq, pp, g[0]);
                g[1] = fmadd(dq, rr, g[1]);
                g[2] = fmadd(t1, dx, g[2]);
                g[3] = fmadd(t1, dy, g[3]);
                g[4] = fmadd(t2, dy, g[4]);
                g[5] += dq;
                g[6] = fmadd(gc0[q], wt, g[6]);
                g[7] = fmadd(gc1[q], wt, g[7]);
                g[8] = fmadd(gc2[q], wt, g[8]);
                g[9] = fmadd(gd[q], wt, g[9]);
            }
            if (!any) continue;
            const uint32_t pslot = s_slot[jl];
            chunk = (lane == filled) ? pslot : chunk;
#pragma unroll
            for (int c = 0; c < kChunk; ++c)
                if (filled == c) {  // uniform
#pragma unroll
                    for (int k = 0; k < kGradWords; ++k) v[c * kGradWords + k] = g[k];
                }
            if (++filled == kChunk) {
                flush_slots<kChunk>(v, chunk, partials, written, cap);
                filled = 0;
            }
        }
        if constexpr (!PREFETCH) {
            if (lane < (int)(a_e - a_s)) load_pair(next_pv);
        }
    }
    if (filled == 1) flush_slots<1>(v, chunk, partials, written, cap);
    else if (filled == 2) flush_slots<2>(v, chunk, partials, written, cap);
    else if (filled == 3) flush_slots<3>(v, chunk, partials, written, cap);
    else if (filled == 4) flush_slots<4>(v, chunk, partials, written, cap);
    else if (filled == 5) flush_slots<5>(v, chunk, partials, written, cap);
}

// The segmented backward's states belong to one particular forward; if the
// frame was binned again since, or the images are another forward's, they are
// not this backward's and every tile is walked whole instead.
__device__ __forceinline__ bool seg_states_valid(const Ctrl* ctrl, const void* last, const void* target) {
    return ctrl->seg_stamp[0] == (uint64_t)ctrl->epoch && ctrl->seg_stamp[1] == (uint64_t)(uintptr_t)last &&
           ctrl->seg_stamp[2] == (uint64_t)(uintptr_t)target;
}

// Segment units in chunks of 16 consecutive list entries (a tile's segments,
// which read the same pixel inputs) on one XCD: workgroup b runs on XCD b % 8,
// and the chunks are dealt to the XCDs round-robin, so the heavy tiles at the
// head of the list still spread over the device.  Each XCD has its own L2; at
// the 200k view this cut the backward's HBM reads from 148 to 103 MB (chunks
// of 4: 116 MB, of 64: 99 MB but slower).
#ifndef DQO_BWD_XCD_CHUNK
#define DQO_BWD_XCD_CHUNK 16
#endif
__device__ __forceinline__ uint32_t seg_unit(uint32_t b) {
    constexpr uint32_t c = DQO_BWD_XCD_CHUNK;
    if constexpr (c == 0) return b;
    const uint32_t x = b % 8u, r = b / 8u;
    return ((r / c) * 8u + x) * c + r % c;
}

// Instance-channel gradients, segmented: the part of a pixel's suffix sum that
// a segment holds, sum of w dL/dw over the pairs it blends there, from the
// state the forward stored at the segment's start (the forward cannot know
// these: they need the upstream gradients).  The segments of a tile run side
// by side, and a backward segment then starts from the sum of the later ones
// (a tile's first segment is nobody's later one and is left out).
// A wavefront takes one 64-pixel part of one segment.
template <typename T, int TW, int TH>
__global__ __launch_bounds__(kWave) void segment_sums_kernel(
    Views<T> V, Consts<T> cs, int K, const T* __restrict__ splats, const uint32_t* __restrict__ pvals,
    const uint32_t* __restrict__ ranges, const int32_t* __restrict__ last, const int32_t* __restrict__ target,
    const T* __restrict__ dC, const T* __restrict__ dD, const T* __restrict__ dP, const T* __restrict__ dPt,
    uint32_t cap, uint32_t M, const uint4* __restrict__ seg_list, const T* __restrict__ ckpt, uint32_t ckpt_cap,
    const int32_t* __restrict__ tile_last, uint32_t seg_len, T* __restrict__ seg_sums, const Ctrl* __restrict__ ctrl) {
    using P = Parts<TW, TH>;
    constexpr uint32_t N = P::kCount;
    __shared__ __align__(16) T s_sp[kWave * kWalkWords];
    if (!seg_states_valid(ctrl, last, target)) return;
    const uint32_t b = seg_unit(blockIdx.x), unit = b / N;
    const int part = (int)(b % N);
    if (unit >= ctrl->counters[kCounterSegTotal]) return;
    const int lane = threadIdx.x;
    const uint4 en = seg_list[unit];
    if (en.z <= en.y) return;
    const int tile = (int)min(en.x, (uint32_t)(V.n_views * V.tiles_per_view) - 1u);
    const uint32_t rs = min(ranges[2 * tile], cap), s0 = min(en.y, cap), s1 = min(max(en.z, s0), cap);
    int tlast = -1;
#pragma unroll
    for (int q = 0; q < (int)N; ++q) tlast = max(tlast, tile_last[tile * (int)N + q]);
    if (s0 <= rs || tlast < (int)s0) return;  // nobody's later segment
    const int plast = tile_last[tile * (int)N + part];
    const uint32_t hi = plast < (int)s0 ? s0 : min((uint32_t)plast + 1u, s1);  // (a part that ends before: zeros)
    const uint32_t e = min(boundary_record(rs, (s0 - rs) / seg_len, seg_len), ckpt_cap - 1u);
    const int view = tile / V.tiles_per_view;
    const int t = tile - view * V.tiles_per_view;
    const int ty = t / V.tiles_x, tx = t - ty * V.tiles_x;
    const int64_t HW = (int64_t)V.W * V.H;
    const T ox = T(tx * TW), oy = T(ty * TH);
    const int lx = P::x0(part) + (lane & 7), ly = P::y0(part) + (lane >> 3);
    const int px = tx * TW + lx, py = ty * TH + ly;
    const T u = T(lx) + T(0.5), vp = T(ly) + T(0.5);
    const int64_t pix = (int64_t)py * V.W + px, o = view * HW + pix;
    int lastp = -1, tgt = -2;
    T Tt = T(0), A = T(0), gc0 = T(0), gc1 = T(0), gc2 = T(0), gd = T(0), gpt = T(0);
    if (hi > s0 && px < V.W && py < V.H && in_window(V.cam[view], px, py)) {
        lastp = last[o];
        Tt = ckpt[((size_t)e * N + part) * 6 * kWave + lane];
        gc0 = dC[(view * 3 + 0) * HW + pix];
        gc1 = dC[(view * 3 + 1) * HW + pix];
        gc2 = dC[(view * 3 + 2) * HW + pix];
        gd = dD ? dD[o] : T(0);
        if (dPt && target) {
            tgt = job_target(V.cam[view].job, target[o]);
            gpt = tgt >= 0 ? dPt[o] : T(0);
        }
    }
    int bx0, bx1, by0, by1;
    tile_pixel_box<T>(V, view, tx, ty, TW, TH, bx0, bx1, by0, by1);
    bx0 = max(bx0, tx * TW + P::x0(part));
    bx1 = min(bx1, tx * TW + P::x0(part) + 7);
    by0 = max(by0, ty * TH + P::y0(part));
    by1 = min(by1, ty * TH + P::y0(part) + 7);
    for (uint32_t b0 = s0; b0 < hi; b0 += kWave) {
        T pf[kRecWords];
        bool cand = false;
        const uint32_t pv = b0 + lane < hi ? pvals[b0 + lane] : kPairSkip;
        if (!(pv & kPairSkip)) {
            load_splat_global<T>(pf, splats + (size_t)min(pv, M - 1) * kSplatWords);
            cand = N == 1 || tile_may_contribute<T>(pf, bx0, bx1, by0, by1, cs);
        }
        __syncthreads();
        const uint64_t bal = __builtin_amdgcn_ballot_w64(cand);
        if (cand) store_walk_record<T>(s_sp + rank_below(bal) * kWalkWords, pf, ox, oy, (int)(b0 + lane), cs);
        __syncthreads();
        const int nb = __popcll(bal);
        for (int jl = 0; jl < nb; ++jl) {
            const T* rec = s_sp + jl * kWalkWords;
            T w[kWB + 1];
#pragma unroll
            for (int k = 0; k <= kWB; ++k) w[k] = rec[k];
            const int id = word_to_id<T>(w[kWId]), pos = word_to_id<T>(w[kWPos]);
            T dx, dy, pp, rr;
            const T E = walk_exponent(w, u, vp, dx, dy, pp, rr);
            const bool contrib = (E >= w[kWThr]) & (pos <= lastp);
            const T a = contrib ? min(exp2_of<T>(E), cs.alpha_max) : T(0);
            if (__builtin_amdgcn_ballot_w64(a != T(0)) == 0ull) continue;
            T vv = fmadd(gc0, w[kWR], fmadd(gc1, w[kWG], fmadd(gc2, w[kWB], gd * w[kWZ])));
            vv += (id == tgt) ? gpt : T(0);
            if (a != T(0) && id >= 0 && id < K) vv += dP[((int64_t)view * K + id) * HW + pix];
            A = fmadd(a * Tt, vv, A);
            Tt = Tt * (T(1) - a);
        }
    }
    seg_sums[((size_t)e * N + part) * kWave + lane] = A;
}

// PROBS: with gradients of the instance channels; SEG: a launch over the
// segment list (instantiations of their own)
template <typename T, int TW, int TH, bool PROBS, bool SEG>
__global__ __launch_bounds__(kWave, TW* TH == kWave ? 4 : DQO_BWD_PARTS_OCC) void render_backward_wave_kernel(
    Views<T> V, Consts<T> cs, int K, const T* __restrict__ splats,
    const uint32_t* __restrict__ pvals, const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ schedule,
    const T* __restrict__ tfinal, const int32_t* __restrict__ last, const int32_t* __restrict__ target,
    const T* __restrict__ dC, const T* __restrict__ dD, const T* __restrict__ dT, const T* __restrict__ dP,
    const T* __restrict__ dPt, T* __restrict__ partials, uint8_t* __restrict__ written, uint32_t cap, uint32_t M,
    const uint4* __restrict__ seg_list, const T* __restrict__ ckpt, uint32_t ckpt_cap, const T* __restrict__ color,
    const T* __restrict__ depth, const T* __restrict__ ptarget, const T* __restrict__ seg_sums,
    const int32_t* __restrict__ tile_last, uint32_t seg_len, const Ctrl* __restrict__ ctrl) {
    __shared__ __align__(16) T s_sp[kWave * kWalkWords];
    __shared__ uint32_t s_slot[kWave];

    // One wavefront per tile, or (with a segment list) per listed segment of
    // a tile's pair range; the list is built after the forward, so its length
    // is read here and the rest of the grid, sized for the longest possible
    // list, exits at once (it holds at least one workgroup per tile).  (A
    // resident grid drawing entries from a work counter was measured slower:
    // the loop around the walk raised its register demand past the budget and
    // spilled.)
    const uint32_t n_tiles = (uint32_t)(V.n_views * V.tiles_per_view);
    if (seg_list && !seg_states_valid(ctrl, last, target)) seg_list = nullptr;
    const uint32_t n_units = seg_list ? ctrl->counters[kCounterSegTotal] : n_tiles;
    uint32_t unit = blockIdx.x;
    if (SEG && seg_list) unit = seg_unit(blockIdx.x);
    if (unit >= n_units) return;
    // (a segmented launch walks a stale frame's whole tiles without prefetch)
    if constexpr (TW * TH == kWave) {
        backward_unit<T, TW, TH, PROBS, !SEG>(V, cs, K, splats, pvals, ranges, schedule, tfinal, last, target, dC, dD,
                                              dT, dP, dPt, partials, written, cap, M, seg_list, ckpt, ckpt_cap, color,
                                              depth, ptarget, seg_sums, tile_last, s_sp, s_slot, unit);
    } else {
        __shared__ uint32_t s_mask[kWave];
        backward_parts<T, TW, TH, PROBS, !SEG>(V, cs, K, splats, pvals, ranges, schedule, tfinal, last, target, dC, dD,
                                               dT, dP, dPt, partials, written, cap, M, seg_list, ckpt, ckpt_cap, color,
                                               depth, ptarget, seg_sums, tile_last, seg_len, s_sp, s_slot, s_mask, unit);
    }
}

// ---------------------------------------------------------------- launchers
template <typename T, int TW, int TH>
static hipError_t fwd_tile(const Frame<T>& f, const dqo_images& img, hipStream_t st) {
    const int blocks = f.views.n_views * f.views.tiles_per_view;
    if (blocks == 0) return hipSuccess;
    const StatePtrs& s = f.s;
    constexpr int N = Parts<TW, TH>::kCount;
    const unsigned grid = N == 1 ? (unsigned)blocks : (unsigned)((blocks + 7) / 8 * 8 * N);
    // Boundary states, last positions and the backward's segment list, for a
    // backward that can run segmented.
    const bool seg = segmented_backward(s, blocks), probs = img.probs && f.K > 0;
    const size_t dyn = probs ? (size_t)f.K * kWave * sizeof(T) : 0;
    auto kern = probs         ? render_forward_kernel<T, TW, TH, true, true>
                : img.n_blend ? render_forward_kernel<T, TW, TH, false, true>
                              : render_forward_kernel<T, TW, TH, false, false>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kWave), dyn, st, f.views, f.consts, f.K, (const T*)s.splats,
                       s.pair_vals[0], s.ranges, s.schedule, (T*)img.color, (T*)img.depth, (T*)img.t_final, img.last,
                       (T*)(probs ? img.probs : nullptr), probs ? img.id_map : nullptr, img.target, (T*)img.p_target,
                       img.n_blend, (uint32_t)s.capacity, (uint32_t)s.items, (T*)(seg ? s.ckpt : nullptr),
                       (uint32_t)s.ckpt_cap, s.tile_last, s.seg_base, s.seg_list, (uint32_t)s.seg_cap, (uint32_t)s.seg_len,
                       s.ctrl);
    return hipGetLastError();
}

template <typename T, int TW, int TH>
static hipError_t bwd_tile(const Frame<T>& f, const dqo_images& img, const dqo_image_grads& g, hipStream_t st) {
    const int blocks = f.views.n_views * f.views.tiles_per_view;
    if (blocks == 0) return hipSuccess;
    const StatePtrs& s = f.s;
    // Segments of the pair ranges, each restarted from the forward's boundary
    // states; with instance-channel gradients after a pass that sums every
    // segment's share of the pixels' suffix sums.
    const bool seg = segmented_backward(s, blocks) &&
                     (g.d_probs || (img.color && img.depth && (img.p_target || !g.d_p_target)));
    // units: the segments, at most tiles + pairs / segment length = seg_cap
    const int64_t gq = 8 * std::max(1, DQO_BWD_XCD_CHUNK);  // whole XCD chunks
    const unsigned grid = seg ? (unsigned)((std::max<int64_t>(s.seg_cap, blocks) + gq - 1) / gq * gq)
                              : (unsigned)blocks;
    if (seg && g.d_probs)
        hipLaunchKernelGGL((segment_sums_kernel<T, TW, TH>), dim3(grid * Parts<TW, TH>::kCount), dim3(kWave), 0, st, f.views, f.consts, f.K,
                           (const T*)s.splats, s.pair_vals[0], s.ranges, img.last, img.target, (const T*)g.d_color,
                           (const T*)g.d_depth, (const T*)g.d_probs, (const T*)g.d_p_target, (uint32_t)s.capacity,
                           (uint32_t)s.items, s.seg_list, (const T*)s.ckpt, (uint32_t)s.ckpt_cap, s.tile_last,
                           (uint32_t)s.seg_len, (T*)s.seg_sums, s.ctrl);
    auto kern = g.d_probs ? (seg ? render_backward_wave_kernel<T, TW, TH, true, true>
                                 : render_backward_wave_kernel<T, TW, TH, true, false>)
                          : (seg ? render_backward_wave_kernel<T, TW, TH, false, true>
                                 : render_backward_wave_kernel<T, TW, TH, false, false>);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kWave), 0, st, f.views, f.consts, f.K, (const T*)s.splats,
                       s.pair_vals[0], s.ranges, s.schedule, (const T*)img.t_final, img.last, img.target,
                       (const T*)g.d_color, (const T*)g.d_depth, (const T*)g.d_t_final, (const T*)g.d_probs,
                       (const T*)g.d_p_target, (T*)s.partials, s.written, (uint32_t)s.capacity,
                       (uint32_t)s.items, seg ? s.seg_list : nullptr, (const T*)s.ckpt, (uint32_t)s.ckpt_cap,
                       (const T*)img.color, (const T*)img.depth, (const T*)img.p_target, (const T*)s.seg_sums,
                       s.tile_last, (uint32_t)s.seg_len, s.ctrl);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_render_forward(const Frame<T>& f, const dqo_images& img, hipStream_t st) {
    const int tw = f.views.tile_w, th = f.views.tile_h;
    if (tw == 16 && th == 16) return fwd_tile<T, 16, 16>(f, img, st);
    if (tw == 8 && th == 8) return fwd_tile<T, 8, 8>(f, img, st);
    if (tw == 16 && th == 8) return fwd_tile<T, 16, 8>(f, img, st);
    if (tw == 32 && th == 8) return fwd_tile<T, 32, 8>(f, img, st);
    if (tw == 8 && th == 32) return fwd_tile<T, 8, 32>(f, img, st);
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_render_backward(const Frame<T>& f, const dqo_images& img, const dqo_image_grads& g,
                                  hipStream_t st) {
    const int tw = f.views.tile_w, th = f.views.tile_h;
    if (tw == 16 && th == 16) return bwd_tile<T, 16, 16>(f, img, g, st);
    if (tw == 8 && th == 8) return bwd_tile<T, 8, 8>(f, img, g, st);
    if (tw == 16 && th == 8) return bwd_tile<T, 16, 8>(f, img, g, st);
    if (tw == 32 && th == 8) return bwd_tile<T, 32, 8>(f, img, g, st);
    if (tw == 8 && th == 32) return bwd_tile<T, 8, 32>(f, img, g, st);
    return hipErrorInvalidValue;
}

template hipError_t launch_render_forward<float>(const Frame<float>&, const dqo_images&, hipStream_t);
template hipError_t launch_render_forward<double>(const Frame<double>&, const dqo_images&, hipStream_t);
template hipError_t launch_render_backward<float>(const Frame<float>&, const dqo_images&, const dqo_image_grads&,
                                                  hipStream_t);
template hipError_t launch_render_backward<double>(const Frame<double>&, const dqo_images&,
                                                   const dqo_image_grads&, hipStream_t);

}  // namespace dqo
