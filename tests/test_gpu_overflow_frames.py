"""GPU: a frame whose pair list overflowed runs through forward and backward
(as a training loop does until it next reads the status), reports the
overflow, and leaves nothing behind: the same state's next frame, whose list
is long enough, gives bitwise the results of a fresh state.  More than 256
tiles, so a second pair pass meets the pairs that the first one dropped."""
import pytest
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [B.DEPTH_ORDER_GLOBAL, B.DEPTH_ORDER_TILE])
@pytest.mark.parametrize("tile,probs", [((16, 16), False), ((16, 16), True), ((8, 8), True), ((8, 8), False)])
def test_overflowed_frame_then_a_whole_one(tile, probs, order):
    n, W, H, K = 8000, 333, 251, 3
    sc = scenes.single_view_scene(seed=5, n=n)
    cam = scenes.camera(fx=110.0 * W / 128, fy=110.0 * W / 128, cx=W / 2, cy=H / 2, width=W, height=H)
    p, ids = to_dev(sc["params"]), torch.tensor(sc["ids"], device="cuda")
    few = p.clone()
    few[2, n // 2:] = -5.0   # behind the camera: half the pairs
    ctx = lambda: B.Context(tile_w=tile[0], tile_h=tile[1], depth_order=order)  # noqa: E731
    g = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    up = dict(d_color=r(1, 3, H, W), d_depth=r(1, H, W), d_t_final=r(1, H, W))
    if probs:
        up["d_probs"] = r(1, K, H, W)
    ref = B.Rasterizer([cam], n, K, ctx=ctx(), capacity=1 << 20)
    assert ref.frame.layout.tiles_x * ref.frame.layout.tiles_y > 256
    want = ref.forward(few, ids, probs=probs)
    want_g = ref.backward(few, want, up)
    _, _, need = ref.frame.read_status()
    ref.bin(p, ids)
    _, _, total = ref.frame.read_status()
    cap = max(need, total * 9 // 10)
    assert need <= cap < total
    fr = B.Rasterizer([cam], n, K, ctx=ctx(), capacity=cap)
    for _ in range(3):
        img = fr.forward(p, ids, probs=probs, grow=False)
        fr.backward(p, img, up)
    rc, st, pairs = fr.frame.read_status()
    assert rc == B.ECAPACITY and st == B.STATUS_OVERFLOW and pairs == total and fr.frame.capacity == cap
    fr.frame.clear_status()
    img = fr.forward(few, ids, probs=probs, grow=False)
    got = fr.backward(few, img, up)
    rc, st, pairs = fr.frame.read_status()
    assert rc == 0 and st == 0 and pairs == need
    for k in ("color", "depth", "t_final", "last") + (("probs",) if probs else ()):
        assert torch.equal(img[k], want[k]), k
    assert torch.equal(got, want_g)
