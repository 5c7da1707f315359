// Index arithmetic of a tile's pair range and of its backward segments, shared
// by the sort, the render kernels and the host (plain constexpr functions, so
// that the indices can be checked without a GPU).
#pragma once
#include <stdint.h>

namespace dqo {

constexpr int kSegLen = 64;        // pairs per backward segment of a tile
constexpr int kSegMax = 255;       // segments per tile (the last one takes the rest of the range)
constexpr uint32_t kNoBoundary = 0xFFFFFFFFu;  // segment-list entry of a tile's last segment: no restart

// A tile's pairs [rs, re), rs <= re <= cap, from its stored bounds.  A list
// that overflowed has slots that no pair was written to, so a tile can show up
// in several runs and its bounds come from different ones, end before start
// included.  Whatever reserves, writes or walks a tile's pairs goes through
// here and so sees the same range.
struct PairRange {
    uint32_t rs, re;
};
constexpr PairRange tile_range(uint32_t start, uint32_t end, uint32_t cap) {
    const uint32_t re = end < cap ? end : cap;
    return {start < re ? start : re, re};
}

// Segments of a range (0 for an empty one); the last one takes the rest of the
// range when it has more than kSegMax.
constexpr uint32_t tile_segments(uint32_t range) {
    const uint32_t n = range / kSegLen + (range % kSegLen != 0u ? 1u : 0u);
    return n < (uint32_t)kSegMax ? n : (uint32_t)kSegMax;
}

// Entries of the segment list that hold a segment: the total reserved can pass
// the list's end where ranges overlap (a list that overflowed).
constexpr uint32_t listed_segments(uint32_t reserved, uint32_t list_cap) {
    return reserved < list_cap ? reserved : list_cap;
}

// The boundary state at pair position b (a multiple of kSegLen past its
// tile's first position rs) is record rs / kSegLen + (b - rs) / kSegLen: the
// records of different tiles never meet (a tile of n pairs has fewer than
// n / kSegLen boundaries and the next starts n positions later), and they
// stay below capacity / kSegLen + 1.
constexpr uint32_t boundary_record(uint32_t rs, uint32_t k) { return rs / kSegLen + k; }

// The walk of segment seg of a range whose pixels blend up to position
// tile_last: pairs [s0, hi), within the segment's [s0, s1); past: pixels blend
// behind s1.  Empty (hi == s0 == rs) behind tile_last and for a segment that
// the range does not have, whatever its index.
struct SegmentWalk {
    uint32_t s0, s1, hi;
    bool past;
};
constexpr SegmentWalk segment_walk(PairRange r, uint32_t seg, int32_t tile_last) {
    const uint32_t nseg = tile_segments(r.re - r.rs);
    if (seg >= nseg) return {r.rs, r.rs, r.rs, false};
    const uint32_t s0 = r.rs + seg * (uint32_t)kSegLen;
    const uint32_t s1 = seg + 1u == nseg ? r.re : s0 + (uint32_t)kSegLen;
    if (tile_last < (int32_t)s0) return {r.rs, r.rs, r.rs, false};
    const uint32_t end = (uint32_t)tile_last + 1u;
    return {s0, s1, end < s1 ? end : s1, end > s1};
}

}  // namespace dqo
