"""The index arithmetic of the backward's segment list (csrc/segments.hpp, the
same functions as in the kernels, compiled here for the host) on the pair list
of a frame that overflowed: a tile may lie in several runs of the list, and its
stored start and end come from any of them, end before start included.  What
the sort reserves is what the suffix pass writes, and every entry that the
segments' launch takes, written or not, walks inside the pair list."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_02223_amd", "csrc")
SHIM = r"""
#include "segments.hpp"
using namespace dqo;
extern "C" {
void range_of(uint32_t a, uint32_t b, uint32_t cap, uint32_t* o) {
    const PairRange r = tile_range(a, b, cap); o[0] = r.rs; o[1] = r.re; }
uint32_t segments_of(uint32_t n) { return tile_segments(n); }
uint32_t listed_of(uint32_t n, uint32_t cap) { return listed_segments(n, cap); }
uint32_t record_of(uint32_t rs, uint32_t k) { return boundary_record(rs, k); }
void walk_of(uint32_t rs, uint32_t re, uint32_t seg, int32_t last, uint32_t* o) {
    const SegmentWalk w = segment_walk({rs, re}, seg, last); o[0] = w.s0; o[1] = w.s1; o[2] = w.hi; o[3] = w.past; }
}
"""


@pytest.fixture(scope="module")
def seg(tmp_path_factory):
    d = tmp_path_factory.mktemp("segments")
    (d / "shim.cpp").write_text(SHIM)
    lib = str(d / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", CSRC, "-o", lib, str(d / "shim.cpp")],
                   check=True)
    L = ctypes.CDLL(lib)
    u = ctypes.c_uint32

    class Seg:
        @staticmethod
        def range(a, b, cap):
            o = (u * 2)()
            L.range_of(u(a), u(b), u(cap), o)
            return int(o[0]), int(o[1])

        @staticmethod
        def walk(rs, re, s, last):
            o = (u * 4)()
            L.walk_of(u(rs), u(re), u(s), ctypes.c_int32(last), o)
            return int(o[0]), int(o[1]), int(o[2]), bool(o[3])

        segments = staticmethod(lambda n: L.segments_of(u(n)))
        listed = staticmethod(lambda n, cap: L.listed_of(u(n), u(cap)))
        record = staticmethod(lambda rs, k: L.record_of(u(rs), u(k)))

    return Seg


def _bounds(rng, tiles, cap, inverted):
    """Stored (start, end) of every tile: runs of an overflowed list whose
    bounds were written in any order; without inversion those of a whole list."""
    cuts = np.sort(rng.integers(0, cap + 1, tiles - 1))
    b = np.stack([np.r_[0, cuts], np.r_[cuts, cap]], 1)
    if inverted:
        other = b[rng.permutation(tiles)]   # the end that another run left
        swap = rng.random(tiles) < 0.5
        b[swap, 1] = other[swap, 1]
        stale = rng.random(tiles) < 0.1     # bounds of an earlier, longer list
        b[stale] += rng.integers(0, cap, (stale.sum(), 2))
    return b


@pytest.mark.parametrize("inverted", [False, True])
@pytest.mark.parametrize("tiles,cap", [(336, 9000), (1024, 1500), (7, 20000), (1, 100), (300, 64 * 300)])
def test_every_listed_entry_walks_inside_the_list(seg, tiles, cap, inverted):
    rng = np.random.default_rng(tiles + cap + inverted)
    for _ in range(10):
        b = _bounds(rng, tiles, cap, inverted)
        rngs = [seg.range(x, y, cap) for x, y in b.tolist()]
        assert all(0 <= rs <= re <= cap for rs, re in rngs)
        list_cap = tiles + cap // 64 + 1
        # the sort's places (any order of the tiles), then the suffix pass's entries
        base = total = 0
        places = {}
        for t in rng.permutation(tiles).tolist():
            places[t] = total
            total += seg.segments(rngs[t][1] - rngs[t][0])
        if not inverted:
            assert total <= list_cap
        entries = rng.integers(0, 1 << 32, (list_cap, 2), dtype=np.uint64)   # uninitialised memory
        written = np.zeros(list_cap, bool)
        for t, (rs, re) in enumerate(rngs):
            for j in range(seg.segments(re - rs)):
                if places[t] + j < list_cap:
                    entries[places[t] + j] = t, j
                    written[places[t] + j] = True
        units = seg.listed(total, list_cap)
        assert units <= list_cap and written[:units].all()
        # every entry, also those that nothing wrote: the walk stays in the list
        last = [int(rng.integers(rs, re)) if re > rs and rng.random() < 0.9 else -1 for rs, re in rngs]
        walked = {}
        for x, s in entries.tolist():
            t = min(x, tiles - 1)
            rs, re = rngs[t]
            s0, s1, hi, past = seg.walk(rs, re, s, last[t])
            assert rs <= s0 <= hi <= s1 <= re
            if hi > s0:
                assert s0 == rs + 64 * s and hi <= last[t] + 1 and past == (last[t] >= s1)
                walked.setdefault(t, set()).add((s0, hi))
            if past:
                assert seg.record(rs, s + 1) < cap // 64 + 1
        if not inverted:   # a whole list: the segments cover [start, last blended] once
            for t, (rs, re) in enumerate(rngs):
                w = sorted(walked.get(t, ()))
                want = max(0, last[t] + 1 - rs)
                assert sum(h - s for s, h in w) == want and all(a[1] == c[0] for a, c in zip(w, w[1:]))


def test_indices_that_wrap_are_refused(seg):
    # 64 * 0x3f800000 wraps to 0xe0000000: negative as a signed position
    for s in (0x3f800000, 0xffffffff, 0x03ffffff, 1 << 26, 4):
        s0, s1, hi, past = seg.walk(1000, 1200, s, 1150)
        assert s0 == hi == 1000 and not past
    assert seg.walk(1000, 1200, 2, 1150) == (1128, 1192, 1151, False)
    assert seg.walk(1000, 1200, 3, 1199) == (1192, 1200, 1200, False)
    # the last of 255 segments takes the rest of a long range
    assert seg.segments(20000) == 255 and seg.walk(0, 20000, 254, 19999) == (254 * 64, 20000, 20000, False)
    assert seg.walk(0, 20000, 253, 19999) == (253 * 64, 254 * 64, 254 * 64, True)
    assert seg.segments(0xffffffff) == 255 and seg.segments(0) == 0 and seg.segments(64) == 1 and seg.segments(65) == 2
