"""GPU: tiles of one to four 64-pixel parts.  Every tile shape renders the
8x8 images (ragged sizes, windows), and the gradients agree with the 8x8 ones
with and without instance channels, where the backward runs through the suffix
pass (up to 4096 parts; ranges of many segments) and where it walks whole
tiles, by strips or, with channels and more than 8192 parts, in chunks.  The shapes differ in FP32 summing order only: the parity tolerance."""
import numpy as np
import pytest
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes
from tests.gpu_util import FWD_RTOL, GRAD_RTOL, close, to_dev

pytestmark = pytest.mark.gpu

TILES = [(8, 8), (16, 8), (16, 16), (32, 8), (8, 32)]


def _setup(n, W, H, V, K, tile, windows=None):
    sc = scenes.single_view_scene(seed=n, n=n)
    cam = scenes.camera(fx=110.0 * W / 128, fy=110.0 * W / 128, cx=W / 2, cy=H / 2, width=W, height=H)
    p = to_dev(sc["params"])
    ids = torch.tensor(sc["ids"] % K, device="cuda")
    r = B.Rasterizer([cam] * V, n, K, ctx=B.Context(tile_w=tile[0], tile_h=tile[1]), windows=windows)
    return r, p, ids


def _upstream(V, H, W, K, probs):
    g = torch.Generator(device="cuda").manual_seed(7)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    up = dict(d_color=r(V, 3, H, W), d_depth=r(V, H, W), d_t_final=r(V, H, W))
    if probs:
        up["d_probs"] = r(V, K, H, W)
    return up


# 125x91 at 30k Gaussians: ranges of many segments, windows leave parts empty;
# 515x389: 3,185 parts a view, so one view goes through the suffix pass, two
# are above its limit, and three take the chunked walk with channels
@pytest.mark.parametrize("probs", [False, True])
@pytest.mark.parametrize("n,W,H,V,windows", [(30000, 125, 91, 1, [(3, 5, 120, 91)]), (20000, 515, 389, 1, None), (20000, 515, 389, 2, None),
                                             (6000, 515, 389, 3, None)])
def test_tile_shapes_agree(n, W, H, V, windows, probs):
    K = 5
    ref = None
    up = _upstream(V, H, W, K, probs)
    for tile in TILES:
        r, p, ids = _setup(n, W, H, V, K, tile, windows)
        img = r.forward(p, ids, probs=probs)
        g = r.backward(p, img, up)
        assert torch.equal(g, r.backward(p, img, up)), tile   # deterministic, nothing left behind
        if ref is None:
            ref = img, g
        # (a splat's mean is rounded relative to its tile's corner, so shapes agree to rounding)
        for k in ("color", "depth", "t_final") + (("probs",) if probs else ()):
            close(img[k].cpu().numpy(), ref[0][k].cpu().numpy(), FWD_RTOL, what=f"{tile} {k}")
        close(g.cpu().numpy(), ref[1].cpu().numpy(), GRAD_RTOL, what=f"{tile} against 8x8")


def test_channel_gradients_leave_the_stored_states():
    """A backward with instance-channel gradients (the suffix pass) between a
    forward and its plain segmented backward changes nothing of the latter."""
    r, p, ids = _setup(30000, 128, 96, 1, 5, (8, 8))
    img = r.forward(p, ids)
    up, up_p = _upstream(1, 96, 128, 5, False), _upstream(1, 96, 128, 5, True)
    before = r.backward(p, img, up)
    r.backward(p, img, up_p)
    assert torch.equal(before, r.backward(p, img, up))


def test_marked_pairs_contribute_nowhere():
    """A pair marked by the forward of a 16x16 tile is below the contribution
    threshold at every pixel of the whole tile, not of one part alone."""
    r, p, ids = _setup(4000, 128, 96, 1, 3, (16, 16))
    r.forward(p, ids)
    f = r.frame
    _, _, P = f.read_status()
    keys = f.buf("pair_keys", torch.int32, P).cpu().numpy()
    vals = f.buf("pair_vals", torch.int32, P).cpu().numpy().view(np.uint32)
    spl = f.buf("splats", torch.float32, 4000 * B.SPLAT_WORDS).view(4000, B.SPLAT_WORDS).cpu().numpy().astype(np.float64)
    marked = np.nonzero(vals >> 31)[0]
    assert marked.size
    v, u = np.mgrid[0:16, 0:16] + 0.5
    tx = f.layout.tiles_x
    for i in marked[:: max(1, marked.size // 500)]:
        s = spl[vals[i] & 0x7FFFFFFF]
        dx, dy = keys[i] % tx * 16 + u - s[0], keys[i] // tx * 16 + v - s[1]
        Q = s[2] * dx * dx + 2 * s[3] * dx * dy + s[4] * dy * dy
        assert not ((Q <= 9) & (s[5] * np.exp(-0.5 * Q) >= 1 / 255)).any()
