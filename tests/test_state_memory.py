"""The state buffer does not grow by the suffix states where they fit in memory
that a render backward leaves idle (the depth passes' buffers and the per-item
sums: 16 bytes and ten values an item), and only frames that use a segment
list hold one.  Layouts only: nothing is launched."""
import ctypes

import pytest

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes


def _total(tile, K, n, cap, W, H, dtype=B.F32, V=1):
    cams = B.make_cameras([scenes.camera(width=W, height=H)] * V)
    d = B.FrameDesc(n=n, n_views=V, K=K, pair_capacity=cap, dtype=dtype)
    L = B.Layout()
    assert B.lib().dqo_state_layout(B.Context(tile_w=tile[0], tile_h=tile[1]).h, ctypes.byref(d), cams,
                                    ctypes.byref(L)) == 0
    return L.total, L.tiles_x * L.tiles_y * V


@pytest.mark.parametrize("n,ratio", [(100_000, 4), (100_000, 12), (3000, 200)])
@pytest.mark.parametrize("dtype", [B.F32, B.F64])
@pytest.mark.parametrize("tile", [(8, 8), (16, 8), (16, 16), (32, 8)])
def test_suffix_states_share_memory(tile, dtype, n, ratio):
    cap, ts = n * ratio, 8 if dtype == B.F64 else 4
    px = tile[0] * tile[1]
    with_states, tiles = _total(tile, 3, n, cap, 160, 120, dtype)
    assert tiles * px // 64 <= 4096
    if px == 64:   # without channels the same frame has no suffix states
        without, slack = _total(tile, 0, n, cap, 160, 120, dtype)[0], 4096
    else:          # too many parts for them: the same but for what the tiles hold
        without, many = _total(tile, 3, n, cap, 2048, 2048, dtype)
        assert many * px // 64 > 4096
        without, slack = without - 32 * (many - tiles), 32 * many + 4096
    states = (cap // 64 + 1) * 2 * px * ts
    idle = n * (16 + 10 * ts)
    lists = 8 * (tiles + cap // 64 + 1) + 4 * tiles * px // 64
    assert with_states - without <= max(0, states - idle) + lists + slack
