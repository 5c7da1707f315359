// Stable LSD radix sort passes (8-bit digits) and tile ranges.
//
// A pass whose grid fits on the device at once is one kernel: a block reads
// threads x IPT (key, value) items, ranks them stably inside the block with
// wave-wide match ballots, obtains its global offset per digit by decoupled
// look-back over the preceding blocks, then writes the items out digit-sorted
// through LDS so stores are coalesced.  Block order is the workgroup index
// (every block it waits on is running); after a wait has timed out it is
// taken from an atomic ticket, so that every block waited on has started (a
// contended global atomic per block, 2.5 us at 383 blocks).  Digit histograms
// of every pass are accumulated before the first pass by the kernel that
// produced the keys.  A larger grid runs as a split pass, three kernels and a
// small one, without a look-back.
#include <algorithm>

#include "dqo_device.hpp"
#include "sort_common.hpp"

namespace dqo {

// The depth passes' digits (see DepthRel), from the key range the projection
// left in copies; wave 0 calls it, the result is in s_krange after a barrier.
__device__ __forceinline__ void depth_key_range(const Ctrl* ctrl, int tid, uint32_t (&s_krange)[2]) {
    uint32_t v = tid < 2 * kHistCopies ? (&ctrl->dkey_range[0][0])[tid] : 0u;
    // lanes of even index hold max(~key) copies, odd ones max(key)
#pragma unroll
    for (int d = 2; d < 2 * kHistCopies; d <<= 1) v = max(v, (uint32_t)__shfl_xor(v, d));
    if (tid < 2) s_krange[tid] = v;
}

struct DepthDigits {
    uint32_t kbase, clamp;
    bool three;  // three passes suffice
};
__device__ __forceinline__ DepthDigits depth_digits(const uint32_t (&s_krange)[2]) {
    const uint32_t kmin = ~s_krange[0], kmax = s_krange[1];
    const bool any = kmax >= kmin;
    DepthDigits d;
    d.kbase = any ? (kmin & ~(uint32_t)(kRadixBins - 1)) : 0u;
    d.three = any && kmax - d.kbase < 0xFFFFFFu;
    d.clamp = d.three ? 0xFFFFFFu : 0xFFFFFFFFu;
    return d;
}

template <int NT, int IPT, bool REL>
__global__ __launch_bounds__(NT) void radix_pass_kernel(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
    uint32_t* __restrict__ vout, const uint32_t* __restrict__ n_dev, uint32_t n_host, int shift,
    const uint32_t* __restrict__ ghist, int hist_stride, int hist_copies, uint64_t* lb, uint32_t* counter,
    Ctrl* ctrl, DepthRel rel) {
    static_assert(NT >= kRadixBins && NT % kWave == 0, "one thread per digit at least");
    constexpr int kTile = NT * IPT;
    constexpr int kWaves = NT / kWave;
    __shared__ uint32_t s_keys[kTile];
    __shared__ uint32_t s_vals[kTile];
    __shared__ uint32_t s_wcnt[kWaves][kRadixBins];
    __shared__ uint32_t s_dstart[kRadixBins];
    __shared__ uint32_t s_gbase[kRadixBins];
    __shared__ uint32_t s_tmp[kWaves];
    __shared__ uint32_t s_bid, s_epoch, s_grouped;
    __shared__ uint32_t s_next[REL ? kRadixBins : 1];  // REL: counts of the next pass's digit

    const int tid = threadIdx.x;
    // REL: the digits of key - base (clamped to 2^24 - 1 when three passes
    // suffice), from the key range the projection left in copies
    __shared__ uint32_t s_krange[2];
    if (REL && tid < kWave) depth_key_range(ctrl, tid, s_krange);
    const int lane = tid & (kWave - 1);
    const int wave = tid >> 6;
    // Every load that does not depend on another is issued before the first
    // wait: the item count, the block's keys at its workgroup index (the order
    // in force unless a ticket is drawn; bounded by the buffer's size n_host,
    // the tail past the count is masked below), the digit totals and the
    // control words.
    const uint32_t n_read = n_dev ? *n_dev : n_host;
    uint32_t key[IPT], val[IPT], rank[IPT];
    auto load_block = [&](uint32_t b) {
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            const uint32_t pos = b * (uint32_t)kTile + wave * (kWave * IPT) + i * kWave + lane;
            key[i] = pos < n_host ? kin[pos] : 0u;
            val[i] = pos < n_host ? vin[pos] : 0u;
        }
    };
    load_block(blockIdx.x);
    const int t = tid;
    const bool owner = t < kRadixBins;
    uint32_t gcount = 0;
    if (owner) {
        // the digit's count over all keys: the sum of the histogram copies
        for (int c = 0; c < hist_copies; ++c) gcount += ghist[c * hist_stride + t];
    }
    if (tid == 0) {
        // Once a bounded wait has given up (status bit, kept until the caller
        // clears it) the order comes from the ticket, every frame.  The
        // resident grid, whose blocks all start together, sums its
        // predecessors in groups; ticket order (blocks staggered in time)
        // walks the chain.
        const bool ticket = (ctrl->status & (uint32_t)DQO_STATUS_TIMEOUT) != 0u;
        s_bid = ticket ? atomicAdd(counter, 1u) : blockIdx.x;
        s_grouped = (ticket || !DQO_LB_GROUPED) ? 0u : 1u;
        s_epoch = ctrl->epoch;
    }
    for (int i = tid; i < kWaves * kRadixBins; i += NT) (&s_wcnt[0][0])[i] = 0;
    if (REL && tid < kRadixBins) s_next[tid] = 0u;
    __syncthreads();
    uint32_t kbase = 0u, clamp = 0xFFFFFFFFu;
    if constexpr (REL) {
        const DepthDigits dd = depth_digits(s_krange);
        kbase = dd.kbase;
        clamp = dd.clamp;
        const bool three = dd.three;
        if (rel.pass == 3 && three) return;  // uniform: nothing left to sort
        if (rel.pass == 2 && three) {
            kout = rel.kout_final;
            vout = rel.vout_final;
            rel.next_hist = nullptr;  // no fourth pass to count for
        }
    }
    auto digit = [&](uint32_t k, int sh) -> uint32_t {
        if constexpr (REL) k = min(k - kbase, clamp);
        return (k >> sh) & (kRadixBins - 1);
    };
    const uint32_t bid = s_bid;
    const uint32_t n = min(n_read, n_host);
    const uint32_t base = bid * (uint32_t)kTile;
    if (base >= n) return;  // uniform over the block; no later block waits on this one
    const uint32_t epoch = s_epoch;
    if (bid != blockIdx.x) load_block(bid);  // ticket order: the block's keys now

    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const uint32_t pos = base + wave * (kWave * IPT) + i * kWave + lane;
        const bool valid = pos < n;
        const uint32_t d = digit(key[i], shift);
        if (REL && rel.next_hist && valid) atomicAdd(&s_next[digit(key[i], shift + kRadixBits)], 1u);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRadixBits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
        uint32_t old = 0;
        if (valid) old = s_wcnt[wave][d];
        const bool leader = valid && ((peers >> lane) == 1ull);
        if (leader) s_wcnt[wave][d] = old + (uint32_t)__popcll(peers);
        rank[i] = old + below;
    }
    __syncthreads();

    // Thread t < 256 owns digit t: per-wave exclusive offsets and the block total.
    uint32_t total = 0;
    if (owner) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = s_wcnt[w][t];
            s_wcnt[w][t] = total;
            total += c;
        }
    }
    const uint32_t dstart = block_exclusive_scan<NT>(total, s_tmp);
    const uint32_t gdig = block_exclusive_scan<NT>(gcount, s_tmp);
    if (owner) {
        s_dstart[t] = dstart;
        // A digit that no key has anywhere needs no chain: every block skips it.
        uint32_t excl = 0u;
        if (gcount) {
            excl = s_grouped ? lookback_grouped(lb + t, lb + (size_t)gridDim.x * kRadixBins + t, kRadixBins, (int)bid,
                                                total, epoch, &ctrl->status)
                             : lookback_exclusive(lb + t, kRadixBins, (int)bid, total, epoch, &ctrl->status);
        }
        s_gbase[t] = gdig + excl;
    }
    __syncthreads();

#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const uint32_t pos = base + wave * (kWave * IPT) + i * kWave + lane;
        if (pos < n) {
            const uint32_t d = digit(key[i], shift);
            const uint32_t p = s_dstart[d] + s_wcnt[wave][d] + rank[i];
            if (p < (uint32_t)kTile) {
                s_keys[p] = key[i];
                s_vals[p] = val[i];
            }
        }
    }
    __syncthreads();
    const uint32_t cnt = min((uint32_t)kTile, n - base);
    for (uint32_t q = tid; q < cnt; q += NT) {
        const uint32_t k = s_keys[q];
        const uint32_t d = digit(k, shift);
        const uint32_t o = s_gbase[d] + (q - s_dstart[d]);
        if (o < n) {  // always true unless a bounded wait gave up (status bit set)
            kout[o] = k;
            vout[o] = s_vals[q];
        }
    }
    if constexpr (REL) {
        if (rel.next_hist && owner) {
            const uint32_t c = s_next[t];
            if (c) atomicAdd(&rel.next_hist[(size_t)(blockIdx.x % hist_copies) * hist_stride + t], c);
        }
    }
}

// ---------------------------------------------------------------- split passes
// A pass whose grid does not fit on the device at once runs as kernels of its
// own: counts per block and digit, their prefix over the blocks (groups of
// blocks, then the groups), ranking and writing.  No block waits on another,
// so blocks need no order and any may run on any XCD: neighbouring blocks,
// whose runs of a digit touch, go to the same one, whose L2 then joins the
// runs' ends into whole lines.  The keys are read twice, which the look-back
// chain outweighs by far (blocks that start in ticket order see it advance a
// window of 8 per round trip over the fabric).  27.8M pairs, one pass: 289 us
// by look-back in ticket order, now 22 + 5 + 4 + 113, where 445 MB take 88 us
// at the copy rate; 49M pairs: 580, now 87 + 6 + 5 + 192; 9.6M depth items:
// 130, now 19 + 5 + 5 + 51.
// The block is 1024 threads x 8 items (512 x 16: 117 us at 27.8M); keys and
// values go through the same 32 KB of LDS in turn, so that two blocks share a
// CU.
constexpr uint32_t kXcds = 8;
constexpr int kSplitNt = 1024, kSplitIpt = 8;
static_assert(kSplitNt * kSplitIpt == kSplitTile, "one count row per block");

// cnt[block][digit]
template <bool REL>
__global__ __launch_bounds__(256) void radix_count_kernel(const uint32_t* __restrict__ kin,
                                                          const uint32_t* __restrict__ n_dev, uint32_t n_host,
                                                          int shift, uint32_t* __restrict__ cnt,
                                                          const Ctrl* __restrict__ ctrl, int pass) {
    __shared__ uint32_t s_h[256 / kWave][kRadixBins];
    __shared__ uint32_t s_krange[2];
    const int tid = threadIdx.x, wave = tid >> 6;
    const uint32_t n = n_dev ? min(*n_dev, n_host) : n_host;
    const uint32_t base = blockIdx.x * (uint32_t)kSplitTile;
    if (base >= n) return;
    if (REL && tid < kWave) depth_key_range(ctrl, tid, s_krange);
#pragma unroll
    for (int w = 0; w < 256 / kWave; ++w) s_h[w][tid] = 0u;
    constexpr int kVec = kSplitTile / (256 * 4);
    uint4 k[kVec];
    const bool full = base + (uint32_t)kSplitTile <= n;
    if (full)
#pragma unroll
        for (int i = 0; i < kVec; ++i) k[i] = reinterpret_cast<const uint4*>(kin + base)[i * 256 + tid];
    __syncthreads();
    DepthDigits dd{0u, 0xFFFFFFFFu, false};
    if constexpr (REL) {
        dd = depth_digits(s_krange);
        if (pass == 3 && dd.three) return;  // uniform: nothing left to sort
    }
    auto add = [&](uint32_t key) {
        if constexpr (REL) key = min(key - dd.kbase, dd.clamp);
        atomicAdd(&s_h[wave][(key >> shift) & (kRadixBins - 1)], 1u);
    };
    if (full) {
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
            add(k[i].x);
            add(k[i].y);
            add(k[i].z);
            add(k[i].w);
        }
    } else {
        for (uint32_t q = base + tid; q < n; q += 256u) add(kin[q]);
    }
    __syncthreads();
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < 256 / kWave; ++w) t += s_h[w][tid];
    cnt[(size_t)blockIdx.x * kRadixBins + tid] = t;
}

// In place, for each group of kSplitGroup blocks: cnt[block][digit] to the
// exclusive prefix over the group's blocks; the group's totals go to
// gcnt[group][digit].  Thread: a digit and a quarter of the blocks.
__global__ __launch_bounds__(1024) void radix_offsets_kernel(const uint32_t* __restrict__ n_dev, uint32_t n_host,
                                                             uint32_t* __restrict__ cnt, uint32_t* __restrict__ gcnt,
                                                             const Ctrl* __restrict__ ctrl, int pass) {
    constexpr int kParts = 1024 / kRadixBins, kRun = kSplitGroup / kParts;
    __shared__ uint32_t s_sum[kParts][kRadixBins];
    __shared__ uint32_t s_krange[2];
    const int tid = threadIdx.x;
    if (pass == 3) {  // a fourth depth pass: none when three suffice
        if (tid < kWave) depth_key_range(ctrl, tid, s_krange);
        __syncthreads();
        if (depth_digits(s_krange).three) return;
    }
    const uint32_t n = n_dev ? min(*n_dev, n_host) : n_host;
    const uint32_t nb = (n + kSplitTile - 1) / kSplitTile;
    if (blockIdx.x * (uint32_t)kSplitGroup >= nb) return;
    const int d = tid % kRadixBins, part = tid / kRadixBins;
    const uint32_t b0 = blockIdx.x * (uint32_t)kSplitGroup + part * kRun;
    uint32_t v[kRun], sum = 0;
#pragma unroll
    for (int i = 0; i < kRun; ++i) v[i] = b0 + i < nb ? cnt[(size_t)(b0 + i) * kRadixBins + d] : 0u;
#pragma unroll
    for (int i = 0; i < kRun; ++i) sum += v[i];
    s_sum[part][d] = sum;
    __syncthreads();
    uint32_t off = 0;
    for (int w = 0; w < part; ++w) off += s_sum[w][d];
    if (part == kParts - 1) gcnt[(size_t)blockIdx.x * kRadixBins + d] = off + sum;
#pragma unroll
    for (int i = 0; i < kRun; ++i) {
        if (b0 + i < nb) cnt[(size_t)(b0 + i) * kRadixBins + d] = off;
        off += v[i];
    }
}

// In place: gcnt[group][digit] to the first output position of the digit's
// items of that group.  One workgroup; thread: a digit and a quarter of the
// groups.
__global__ __launch_bounds__(1024) void radix_groups_kernel(const uint32_t* __restrict__ n_dev, uint32_t n_host,
                                                            uint32_t* __restrict__ gcnt,
                                                            const Ctrl* __restrict__ ctrl, int pass) {
    constexpr int kParts = 1024 / kRadixBins, kChunk = 16;
    __shared__ uint32_t s_sum[kParts][kRadixBins];
    __shared__ uint32_t s_tmp[1024 / kWave];
    __shared__ uint32_t s_krange[2];
    const int tid = threadIdx.x;
    if (pass == 3) {  // a fourth depth pass: none when three suffice
        if (tid < kWave) depth_key_range(ctrl, tid, s_krange);
        __syncthreads();
        if (depth_digits(s_krange).three) return;
    }
    const uint32_t n = n_dev ? min(*n_dev, n_host) : n_host;
    const uint32_t nb = (n + kSplitTile - 1) / kSplitTile, groups = (nb + kSplitGroup - 1) / kSplitGroup;
    const uint32_t run = (groups + kParts - 1) / kParts;
    const int d = tid % kRadixBins, part = tid / kRadixBins;
    const uint32_t g0 = min(groups, part * run), g1 = min(groups, g0 + run);
    uint32_t sum = 0, v[kChunk];
    for (uint32_t g = g0; g < g1; g += kChunk) {
#pragma unroll
        for (int k = 0; k < kChunk; ++k) v[k] = g + k < g1 ? gcnt[(size_t)(g + k) * kRadixBins + d] : 0u;
#pragma unroll
        for (int k = 0; k < kChunk; ++k) sum += v[k];
    }
    s_sum[part][d] = sum;
    __syncthreads();
    uint32_t total = 0, off = 0;
    for (int w = 0; w < kParts; ++w) {
        if (w < part) off += s_sum[w][d];
        total += s_sum[w][d];
    }
    const uint32_t base = block_exclusive_scan<1024>(part == 0 ? total : 0u, s_tmp);  // valid in the first 256 threads
    __syncthreads();
    if (part == 0) s_sum[0][d] = base;
    __syncthreads();
    off += s_sum[0][d];
    for (uint32_t g = g0; g < g1; g += kChunk) {
        if (run > kChunk) {  // (else the counts are still in registers)
#pragma unroll
            for (int k = 0; k < kChunk; ++k) v[k] = g + k < g1 ? gcnt[(size_t)(g + k) * kRadixBins + d] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kChunk; ++k) {
            if (g + k < g1) gcnt[(size_t)(g + k) * kRadixBins + d] = off;
            off += v[k];
        }
    }
}

template <bool REL>
__global__ __launch_bounds__(kSplitNt) void radix_scatter_kernel(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
    uint32_t* __restrict__ vout, const uint32_t* __restrict__ n_dev, uint32_t n_host, int shift,
    const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ gcnt, const Ctrl* __restrict__ ctrl,
    DepthRel rel) {
    constexpr int NT = kSplitNt, IPT = kSplitIpt, kWaves = NT / kWave;
    __shared__ uint32_t s_x[kSplitTile];
    __shared__ uint32_t s_wcnt[kWaves][kRadixBins];
    __shared__ uint32_t s_dstart[kRadixBins];
    __shared__ uint32_t s_off[kRadixBins];
    __shared__ uint32_t s_tmp[kWaves];
    __shared__ uint32_t s_krange[2];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const uint32_t n = n_dev ? min(*n_dev, n_host) : n_host;
    const uint32_t nb = (n + kSplitTile - 1) / kSplitTile, per = (nb + kXcds - 1) / kXcds;
    const uint32_t slot = blockIdx.x / kXcds, bid = (blockIdx.x % kXcds) * per + slot;
    if (slot >= per || bid >= nb) return;
    const uint32_t base = bid * (uint32_t)kSplitTile;
    uint32_t key[IPT], val[IPT], rank[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const uint32_t pos = base + wave * (kWave * IPT) + i * kWave + lane;
        key[i] = pos < n ? kin[pos] : 0u;
    }
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const uint32_t pos = base + wave * (kWave * IPT) + i * kWave + lane;
        val[i] = pos < n ? vin[pos] : 0u;
    }
    const bool owner = tid < kRadixBins;
    // where the block's items of this digit go
    uint32_t first = 0u;
    if (owner) first = cnt[(size_t)bid * kRadixBins + tid] + gcnt[(size_t)(bid / kSplitGroup) * kRadixBins + tid];
    if (REL && tid < kWave) depth_key_range(ctrl, tid, s_krange);
    for (int i = tid; i < kWaves * kRadixBins; i += NT) (&s_wcnt[0][0])[i] = 0;
    __syncthreads();
    DepthDigits dd{0u, 0xFFFFFFFFu, false};
    if constexpr (REL) {
        dd = depth_digits(s_krange);
        if (rel.pass == 3 && dd.three) return;  // uniform: nothing left to sort
        if (rel.pass == 2 && dd.three) {
            kout = rel.kout_final;
            vout = rel.vout_final;
        }
    }
    auto digit = [&](uint32_t k) -> uint32_t {
        if constexpr (REL) k = min(k - dd.kbase, dd.clamp);
        return (k >> shift) & (kRadixBins - 1);
    };
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const bool valid = base + wave * (kWave * IPT) + i * kWave + lane < n;
        const uint32_t d = digit(key[i]);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRadixBits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
        uint32_t old = 0;
        if (valid) old = s_wcnt[wave][d];
        const bool leader = valid && ((peers >> lane) == 1ull);
        if (leader) s_wcnt[wave][d] = old + (uint32_t)__popcll(peers);
        rank[i] = old + below;
    }
    __syncthreads();
    uint32_t total = 0;
    if (owner) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = s_wcnt[w][tid];
            s_wcnt[w][tid] = total;
            total += c;
        }
    }
    const uint32_t dstart = block_exclusive_scan<NT>(total, s_tmp);
    if (owner) {
        s_dstart[tid] = dstart;
        s_off[tid] = first - dstart;  // output position of the block's item q of this digit: s_off + q
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        if (base + wave * (kWave * IPT) + i * kWave + lane < n) {
            const uint32_t d = digit(key[i]);
            rank[i] += s_dstart[d] + s_wcnt[wave][d];
            s_x[rank[i]] = key[i];
        }
    }
    __syncthreads();
    const uint32_t cnt_here = min((uint32_t)kSplitTile, n - base);
    uint32_t o[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const uint32_t q = i * NT + tid;
        o[i] = n;
        if (q < cnt_here) {
            const uint32_t k = s_x[q];
            o[i] = s_off[digit(k)] + q;
            if (o[i] < n) kout[o[i]] = k;  // (always, unless the keys changed since they were counted)
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IPT; ++i)
        if (base + wave * (kWave * IPT) + i * kWave + lane < n) s_x[rank[i]] = val[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        if (o[i] < n) vout[o[i]] = s_x[i * NT + tid];
    }
}

hipError_t launch_split_pass(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout,
                             const uint32_t* n_dev, uint32_t n_host, int shift, uint32_t* cnt, const Ctrl* ctrl,
                             hipStream_t st, const DepthRel* rel) {
    if (n_host == 0) return hipSuccess;
    const unsigned nb = (unsigned)(((uint64_t)n_host + kSplitTile - 1) / kSplitTile);
    const unsigned grid = (nb + kXcds - 1) / kXcds * kXcds;
    const DepthRel r = rel ? *rel : DepthRel{0, nullptr, nullptr, nullptr};
    hipLaunchKernelGGL(rel ? radix_count_kernel<true> : radix_count_kernel<false>, dim3(nb), dim3(256), 0, st, kin,
                       n_dev, n_host, shift, cnt, ctrl, r.pass);
    uint32_t* gcnt = cnt + (size_t)nb * kRadixBins;
    hipLaunchKernelGGL(radix_offsets_kernel, dim3((nb + kSplitGroup - 1) / kSplitGroup), dim3(1024), 0, st, n_dev,
                       n_host, cnt, gcnt, ctrl, r.pass);
    hipLaunchKernelGGL(radix_groups_kernel, dim3(1), dim3(1024), 0, st, n_dev, n_host, gcnt, ctrl, r.pass);
    hipLaunchKernelGGL(rel ? radix_scatter_kernel<true> : radix_scatter_kernel<false>, dim3(grid), dim3(kSplitNt), 0,
                       st, kin, vin, kout, vout, n_dev, n_host, shift, cnt, gcnt, ctrl, r);
    return hipGetLastError();
}

// [start, end) of every tile that holds pairs, from the boundaries of the
// sorted pair keys (tiles without pairs keep the empty range written when the
// frame was projected).  The same pass clears the written marks of the pairs
// (four one-byte marks per word), which the render backward sets.  Bound by
// reading the keys: a thread takes four, in one 16-byte load, and the key
// before them from the lane below (one key per thread with its neighbours'
// took 66 us for 27.8M pairs, now 28).
__global__ __launch_bounds__(256) void tile_bounds_kernel(const uint32_t* __restrict__ keys,
                                                          const uint32_t* __restrict__ n_dev, uint32_t n_host,
                                                          uint32_t tiles, uint32_t* __restrict__ ranges,
                                                          uint32_t* __restrict__ written_words) {
    const uint32_t n = min(*n_dev, n_host), nw = (n + 3u) / 4u;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t stride = gridDim.x * 256u;
    for (uint32_t w0 = blockIdx.x * 256u + (threadIdx.x - lane); w0 < nw; w0 += stride) {  // uniform per wavefront
        const uint32_t w = w0 + lane, i = 4u * w;
        uint32_t k[5] = {0u, 0u, 0u, 0u, 0u};  // the key before, then the four
        if (i + 4u <= n) {
            const uint4 v = reinterpret_cast<const uint4*>(keys)[w];
            k[1] = v.x;
            k[2] = v.y;
            k[3] = v.z;
            k[4] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (i + j < n) k[1 + j] = keys[i + j];
        }
        k[0] = __shfl_up(k[4], 1);
        if (lane == 0 && w0 > 0u) k[0] = keys[i - 1u];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t p = i + j;
            if (p >= n) break;
            const uint32_t t = k[1 + j];
            // (a list that overflowed may hold slots that no pair was written to)
            if (p == 0u || k[j] != t) {
                if (t < tiles) ranges[2 * t] = p;
                if (p > 0u && k[j] < tiles) ranges[2 * k[j] + 1] = p;
            }
            if (p + 1u == n && t < tiles) ranges[2 * t + 1] = n;
        }
        if (w < nw) written_words[w] = 0u;
    }
}

// Launch order of the render workgroups: tiles by decreasing pair count.
// Workgroups are dispatched in index order and spread round-robin over the
// XCDs and CUs, so the heaviest tiles, which are spatially clustered, start
// first and on different compute units instead of queueing on the same ones,
// and the launch ends with the lightest.  Counts are exact up to 4095 (larger
// ones share the top bin).  Against power-of-two classes of the count (tiles
// of a class in index order), the exact order made the backward replayed on
// its own at the 200k view 5% faster and the forward 6%; inside the whole
// training step the difference was within run-to-run noise.  Order among
// equal counts is arbitrary; results do not depend on the order (every tile
// writes only its own pixels and pair slots).
constexpr int kSchedThreads = 1024;
constexpr int kSchedBins = 4096;

// Up to kSchedRegs tiles per thread are loaded once, all at once, and kept in
// registers (their ranges are read by two dependent phases: the count
// histogram and the scatter); more tiles loop over global memory.
constexpr int kSchedRegs = 8;
__global__ __launch_bounds__(kSchedThreads) void tile_schedule_kernel(const uint32_t* __restrict__ ranges,
                                                                     int tiles, uint32_t* __restrict__ schedule,
                                                                     uint32_t cap, int seg,
                                                                     uint32_t* __restrict__ seg_base,
                                                                     Ctrl* __restrict__ ctrl) {
    __shared__ uint32_t s_cnt[kSchedBins];  // bin b holds count kSchedBins - 1 - b (descending order)
    // segmented backward: the segments of each bin's tiles, then the bin's
    // cursor in the segment list
    __shared__ uint32_t s_seg[kSchedBins];
    __shared__ uint32_t s_tmp[kSchedThreads / kWave];
    constexpr int kPer = kSchedBins / kSchedThreads;
    const int tid = threadIdx.x;
    auto bin_of_w = [](uint32_t w) { return kSchedBins - 1 - (int)min(w, (uint32_t)(kSchedBins - 1)); };
    auto width = [&](int t) {
        const uint2 b = reinterpret_cast<const uint2*>(ranges)[t];
        const PairRange r = tile_range(b.x, b.y, cap);  // as the render kernels see it
        return r.re - r.rs;
    };
    // thread tid holds tiles tid + k * kSchedThreads (coalesced loads)
    const bool regs = tiles <= kSchedRegs * kSchedThreads;
    uint32_t w[kSchedRegs];
    if (regs) {
#pragma unroll
        for (int k = 0; k < kSchedRegs; ++k) {
            const int t = tid + k * kSchedThreads;
            w[k] = t < tiles ? width(t) : 0u;
        }
    }
    for (int b = tid; b < kSchedBins; b += kSchedThreads) s_cnt[b] = s_seg[b] = 0u;
    __syncthreads();
    auto count = [&](uint32_t wt) {
        atomicAdd(&s_cnt[bin_of_w(wt)], 1u);
        if (seg) atomicAdd(&s_seg[bin_of_w(wt)], tile_segments(wt));
    };
    if (regs) {
#pragma unroll
        for (int k = 0; k < kSchedRegs; ++k)
            if (tid + k * kSchedThreads < tiles) count(w[k]);
    } else {
        for (int t = tid; t < tiles; t += kSchedThreads) count(width(t));
    }
    __syncthreads();
    uint32_t c[kPer], g[kPer], sum = 0, gsum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        c[k] = s_cnt[tid * kPer + k];
        g[k] = s_seg[tid * kPer + k];
        sum += c[k];
        gsum += g[k];
    }
    uint32_t off = block_exclusive_scan<kSchedThreads>(sum, s_tmp);
    uint32_t goff = seg ? block_exclusive_scan<kSchedThreads>(gsum, s_tmp) : 0u;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        s_cnt[tid * kPer + k] = off;
        s_seg[tid * kPer + k] = goff;
        off += c[k];
        goff += g[k];
    }
    // The backward's segment list holds every 64-pair segment of every tile,
    // tiles by bin (heaviest first); the forward fills in each tile's entries
    // once it knows how far its pixels blend (the rest it marks empty).
    if (seg && tid == kSchedThreads - 1) ctrl->counters[kCounterSegTotal] = goff;
    __syncthreads();
    auto place = [&](int t, uint32_t wt) {
        schedule[atomicAdd(&s_cnt[bin_of_w(wt)], 1u)] = (uint32_t)t;
        if (seg) seg_base[t] = atomicAdd(&s_seg[bin_of_w(wt)], tile_segments(wt));
    };
    if (regs) {
#pragma unroll
        for (int k = 0; k < kSchedRegs; ++k)
            if (tid + k * kSchedThreads < tiles) place(tid + k * kSchedThreads, w[k]);
    } else {
        for (int t = tid; t < tiles; t += kSchedThreads) place(t, width(t));
    }
}

// The block shapes in use: (threads, items per thread, depth pass).
#define DQO_RADIX_SHAPES(X) X(kDepthNt, 2, true) X(kDepthNt, 4, true) X(kPairNt, kPairIptShort, false) \
                            X(kPairNtLong, kPairIptLong, false)

bool radix_resident(int nt, int ipt, int64_t items) {
    const int64_t blocks = (items + (int64_t)nt * ipt - 1) / ((int64_t)nt * ipt);
    int res = 0;
#define DQO_RADIX_RES(NT_, IPT_, REL_) \
    if (nt == NT_ && ipt == IPT_) res = resident_blocks<radix_pass_kernel<NT_, IPT_, REL_>, NT_>();
    DQO_RADIX_SHAPES(DQO_RADIX_RES)
#undef DQO_RADIX_RES
    return blocks <= res;
}

hipError_t launch_radix_pass(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout,
                             const uint32_t* n_dev, uint32_t n_host, int shift, const uint32_t* ghist,
                             int hist_stride, int hist_copies, uint64_t* lb, uint32_t* counter, Ctrl* ctrl,
                             hipStream_t st, int nt, int ipt, const DepthRel* rel) {
    if (n_host == 0) return hipSuccess;
    const DepthRel r = rel ? *rel : DepthRel{0, nullptr, nullptr, nullptr};
    const uint32_t blocks = (uint32_t)(((int64_t)n_host + nt * ipt - 1) / (nt * ipt));
#define DQO_RADIX_CASE(NT_, IPT_, REL_)                                                                          \
    if (nt == NT_ && ipt == IPT_ && (rel != nullptr) == REL_) {                                                  \
        hipLaunchKernelGGL((radix_pass_kernel<NT_, IPT_, REL_>), dim3(blocks), dim3(NT_), 0, st, kin, vin, kout, \
                           vout, n_dev, n_host, shift, ghist, hist_stride, hist_copies, lb, counter, ctrl, r);   \
        return hipGetLastError();                                                                                \
    }
    DQO_RADIX_SHAPES(DQO_RADIX_CASE)
#undef DQO_RADIX_CASE
    return hipErrorInvalidValue;
}

// Per-tile depth order.  The pairs were emitted in item order and stably
// sorted by tile, so each tile's range holds its items in index order; one
// workgroup per tile sorts them by the item's depth key, ties by item index:
// the order a stable sort of every item by depth followed by the stable tile
// sort gives.  Up to kTileSortLds pairs: a bitonic network over the 64-bit
// values key << 32 | item, padded to P = 256 E (E = 1..16 values per thread,
// held in registers in blocked order: value e = thread E + r).  Its stages
// with a partner distance j < E run inside a thread, those with j < 64 E
// across the lanes of a wavefront (shuffles), and only those with j >= 64 E
// (three at P = 4096) through LDS with barriers.  Longer ranges: four stable
// 8-bit passes over global memory by the workgroup, through tmp (slow; meant
// for rare long tiles).  Tiles are taken in the launch order of the render
// (longest first), so the longest sorts start first.
constexpr int kTileSortThreads = 256;
constexpr int kTileSortLds = 4096;

__device__ __forceinline__ uint64_t keep_lo_hi(uint64_t mine, uint64_t other, bool keep_min) {
    const bool lt = mine < other;
    return (lt == keep_min) ? mine : other;
}

template <int E>
__device__ __forceinline__ void tile_bitonic(uint64_t (&x)[16], uint64_t* s_x, int tid, uint32_t P) {
    const int lane = tid & (kWave - 1);
    for (uint32_t k = 2u; k <= P; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0u; j >>= 1) {
            if (j < (uint32_t)E) {
#pragma unroll
                for (int r = 0; r < E; ++r) {
                    if ((r & (int)j) == 0) {
                        const uint32_t e = (uint32_t)tid * E + r;
                        const bool up = (e & k) == 0u;
                        const uint64_t a = x[r], b = x[r | (int)j];
                        const bool swap = (a > b) == up;
                        x[r] = swap ? b : a;
                        x[r | (int)j] = swap ? a : b;
                    }
                }
            } else if (j < (uint32_t)(kWave * E)) {
                const int d = (int)(j / (uint32_t)E);
#pragma unroll
                for (int r = 0; r < E; ++r) {
                    const uint64_t y = (uint64_t)__shfl_xor((unsigned long long)x[r], d);
                    const uint32_t e = (uint32_t)tid * E + r;
                    x[r] = keep_lo_hi(x[r], y, ((e & j) == 0u) == ((e & k) == 0u));
                }
            } else {
#pragma unroll
                for (int r = 0; r < E; ++r) s_x[tid * E + r] = x[r];
                __syncthreads();
#pragma unroll
                for (int r = 0; r < E; ++r) {
                    const uint32_t e = (uint32_t)tid * E + r;
                    x[r] = keep_lo_hi(x[r], s_x[e ^ j], ((e & j) == 0u) == ((e & k) == 0u));
                }
                __syncthreads();
            }
        }
    }
    (void)lane;
}

__global__ __launch_bounds__(kTileSortThreads) void tile_sort_kernel(const uint32_t* __restrict__ ranges,
                                                                    const uint32_t* __restrict__ schedule,
                                                                    const uint32_t* __restrict__ dkeys, uint32_t M,
                                                                    uint32_t cap, uint32_t lds_max, int tiles,
                                                                    const uint32_t* __restrict__ n_dev,
                                                                    uint32_t* __restrict__ pvals,
                                                                    uint32_t* __restrict__ tmp) {
    __shared__ uint64_t s_k[kTileSortLds];
    __shared__ uint32_t s_off[kRadixBins];
    __shared__ uint32_t s_wcnt[kTileSortThreads / kWave][kRadixBins];
    __shared__ uint32_t s_scan[kTileSortThreads / kWave];
    if (*n_dev > cap) return;  // the list overflowed: its ranges mean nothing
    const int tid = threadIdx.x;
    const uint32_t tile = min(schedule[blockIdx.x], (uint32_t)(tiles - 1));
    const PairRange range = tile_range(ranges[2 * tile], ranges[2 * tile + 1], cap);
    const uint32_t rs = range.rs, re = range.re;
    const uint32_t n = re - rs;
    if (n <= 1u) return;
    if (n <= min(lds_max, (uint32_t)kTileSortLds)) {
        int E = 1;
        while ((uint32_t)(kTileSortThreads * E) < n) E <<= 1;
        const uint32_t P = (uint32_t)(kTileSortThreads * E);
        uint64_t x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint32_t e = (uint32_t)tid * E + r;
            x[r] = ~0ull;  // padding sorts last
            if (r < E && e < n) {
                const uint32_t item = min(pvals[rs + e], M - 1);
                x[r] = ((uint64_t)dkeys[item] << 32) | item;
            }
        }
        switch (E) {
            case 1: tile_bitonic<1>(x, s_k, tid, P); break;
            case 2: tile_bitonic<2>(x, s_k, tid, P); break;
            case 4: tile_bitonic<4>(x, s_k, tid, P); break;
            case 8: tile_bitonic<8>(x, s_k, tid, P); break;
            default: tile_bitonic<16>(x, s_k, tid, P); break;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint32_t e = (uint32_t)tid * E + r;
            if (r < E && e < n) pvals[rs + e] = (uint32_t)x[r];
        }
        return;
    }
    // Long range: stable LSD passes, 256 items per round in index order,
    // ranked inside each wavefront by match ballots.
    const int lane = tid & (kWave - 1), wave = tid >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t* src = pvals + rs;
    uint32_t* dst = tmp + rs;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = pass * kRadixBits;
        for (int w = 0; w < kTileSortThreads / kWave; ++w)
            if (tid < kRadixBins) s_wcnt[w][tid] = 0u;
        if (tid < kRadixBins) s_off[tid] = 0u;
        __syncthreads();
        for (uint32_t i = tid; i < n; i += kTileSortThreads)
            atomicAdd(&s_off[(dkeys[min(src[i], M - 1)] >> shift) & (kRadixBins - 1)], 1u);
        __syncthreads();
        {
            const uint32_t c = tid < kRadixBins ? s_off[tid] : 0u;
            const uint32_t ex = block_exclusive_scan<kTileSortThreads>(c, s_scan);
            __syncthreads();
            if (tid < kRadixBins) s_off[tid] = ex;
            __syncthreads();
        }
        for (uint32_t c0 = 0; c0 < n; c0 += kTileSortThreads) {
            const uint32_t i = c0 + (uint32_t)tid;
            const bool valid = i < n;
            const uint32_t item = valid ? src[i] : 0u;
            const uint32_t d = valid ? (dkeys[min(item, M - 1)] >> shift) & (kRadixBins - 1) : 0u;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < kRadixBits; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bb = __ballot(bit);
                peers &= bit ? bb : ~bb;
            }
            const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
            if (valid && (peers >> lane) == 1ull) s_wcnt[wave][d] = (uint32_t)__popcll(peers);
            __syncthreads();
            if (valid) {
                uint32_t before = 0;
                for (int w = 0; w < wave; ++w) before += s_wcnt[w][d];
                dst[s_off[d] + before + below] = item;
            }
            __syncthreads();
            if (tid < kRadixBins) {
                uint32_t total = 0;
                for (int w = 0; w < kTileSortThreads / kWave; ++w) {
                    total += s_wcnt[w][tid];
                    s_wcnt[w][tid] = 0u;
                }
                s_off[tid] += total;
            }
            __syncthreads();
        }
        uint32_t* t = src;
        src = dst;
        dst = t;
    }
    // four passes: the result is back in pvals
}

bool pair_sort_split(int64_t capacity) {
    return !radix_resident(kPairNt, kPairIptShort, capacity) && !radix_resident(kPairNtLong, kPairIptLong, capacity);
}

hipError_t launch_pair_sort(const StatePtrs& s, int tiles_total, hipStream_t st) {
    const uint32_t cap = (uint32_t)s.capacity;
    const uint32_t* n_dev = &s.ctrl->num_pairs;
    // short blocks while that grid is resident, else long ones, else the split pass
    const bool short_ok = radix_resident(kPairNt, kPairIptShort, cap);
    const bool split = pair_sort_split(cap);
    const int nt = short_ok ? kPairNt : kPairNtLong, ipt = short_ok ? kPairIptShort : kPairIptLong;
    // the fused emission has done pass 0 (its output is in the other buffer)
    const int p0 = s.fused_emit ? 1 : 0;
    int src = s.pair_first_buf ^ p0;
    for (int p = p0; p < s.pair_passes; ++p) {
        uint32_t *ki = s.pair_keys[src], *vi = s.pair_vals[src], *ko = s.pair_keys[src ^ 1], *vo = s.pair_vals[src ^ 1];
        hipError_t e =
            split ? launch_split_pass(ki, vi, ko, vo, n_dev, cap, p * kRadixBits, s.digit_counts, s.ctrl, st)
                  : launch_radix_pass(ki, vi, ko, vo, n_dev, cap, p * kRadixBits, &s.ctrl->hist_pair[0][p][0],
                                      kMaxPairPasses * kRadixBins, s.hist_copies_pair,
                                      s.lb_pair + (size_t)p * lb_blocks(s.pair_blocks) * kRadixBins,
                                      &s.ctrl->counters[kCounterPair + p], s.ctrl, st, nt, ipt);
        if (e != hipSuccess) return e;
        src ^= 1;
    }
    if (tiles_total > 0) {
        // four pairs per thread, every key load in flight at once
        const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(1 << 20, ((int64_t)cap + 1023) / 1024));
        hipLaunchKernelGGL(tile_bounds_kernel, dim3(grid), dim3(256), 0, st, s.pair_keys[0], n_dev, cap,
                           (uint32_t)tiles_total, s.ranges,
                           (uint32_t*)s.written);
        hipLaunchKernelGGL(tile_schedule_kernel, dim3(1), dim3(kSchedThreads), 0, st, s.ranges, tiles_total,
                           s.schedule, cap, segmented_backward(s, tiles_total) || suffix_backward(s) ? 1 : 0,
                           s.seg_base, s.ctrl);
        if (s.tile_sort)
            hipLaunchKernelGGL(tile_sort_kernel, dim3((unsigned)tiles_total), dim3(kTileSortThreads), 0, st, s.ranges,
                               s.schedule, s.depth_keys[0], (uint32_t)s.items, cap, (uint32_t)s.tile_sort_lds,
                               tiles_total, n_dev, s.pair_vals[0], s.pair_vals[1]);
        return hipGetLastError();
    }
    return launch_clear_written(s, st);
}

}  // namespace dqo
