"""GPU: a channel gradient counts only where the object contributes.  The
gradient of log P is infinite or NaN where P is zero; such entries leave the
Gaussians' gradients bitwise as a zero there does, for every way through the
backward: the suffix pass (8x8 and larger tiles of few parts), strips, chunks
and whole 8x8 tiles."""
import numpy as np
import pytest
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("tile,V,W,H", [((8, 8), 1, 125, 91), ((16, 16), 1, 125, 91), ((16, 8), 2, 515, 389),
                                        ((16, 16), 3, 515, 389), ((8, 8), 2, 515, 389)])
def test_gradients_of_absent_objects_do_not_spread(tile, V, W, H, dtype):
    n, K = 6000, 4
    sc = scenes.single_view_scene(seed=9, n=n)
    cam = scenes.camera(fx=110.0 * W / 128, fy=110.0 * W / 128, cx=W / 2, cy=H / 2, width=W, height=H)
    p, ids = to_dev(sc["params"], dtype), torch.tensor(sc["ids"] % K, device="cuda")
    r = B.Rasterizer([cam] * V, n, K, ctx=B.Context(tile_w=tile[0], tile_h=tile[1]), dtype=dtype)
    img = r.forward(p, ids, probs=True)
    g = torch.Generator(device="cuda").manual_seed(2)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=dtype)  # noqa: E731
    up = dict(d_color=rand(V, 3, H, W), d_depth=rand(V, H, W), d_t_final=rand(V, H, W), d_probs=rand(V, K, H, W))
    absent = img["probs"] == 0
    assert absent.float().mean() > 0.2 and (~absent).float().mean() > 0.2
    up["d_probs"][absent] = 0.0
    want = r.backward(p, img, up)
    assert torch.isfinite(want).all() and want.abs().max() > 0
    for bad in (np.inf, -np.inf, np.nan):
        up["d_probs"][absent] = bad
        assert torch.equal(r.backward(p, img, up), want), bad
