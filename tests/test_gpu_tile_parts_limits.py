"""GPU: the backward of tiles of several 64-pixel parts where its branches
end.  FP64 frames through the suffix pass, strips and chunks (their 74 KB of
LDS at 16x16 pixels) against 8x8 tiles; ranges longer than the 255 segments
that the suffix pass lists, whose last entry takes the rest in several batches,
against the same Gaussians in a frame of so many parts that tiles are walked
whole; a depth sort of so many items that the groups' prefix goes in rounds."""
import gc

import numpy as np
import pytest
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes
from tests.gpu_util import FWD_RTOL, GRAD_RTOL, close, to_dev

pytestmark = pytest.mark.gpu

# shapes differ in summing order only: the FP32 gradients' 1e-3 times the ratio
# of the roundings (2^-29) is 2e-12, and FP64 leaves no threshold undecided
RTOL64 = 1e-9


@pytest.mark.parametrize("probs", [False, True])
@pytest.mark.parametrize("V", [1, 2, 3])   # 3,300 parts a view: suffix pass; strips; chunks with channels
def test_tile_shapes_agree_in_fp64(V, probs):
    n, W, H, K = 6000, 515, 389, 5
    sc = scenes.single_view_scene(seed=n, n=n)
    cam = scenes.camera(fx=110.0 * W / 128, fy=110.0 * W / 128, cx=W / 2, cy=H / 2, width=W, height=H)
    p, ids = to_dev(sc["params"], torch.float64), torch.tensor(sc["ids"] % K, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(7)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float64)  # noqa: E731
    up = dict(d_color=r(V, 3, H, W), d_depth=r(V, H, W), d_t_final=r(V, H, W))
    if probs:
        up["d_probs"] = r(V, K, H, W)
    ref = None
    for tile in ((8, 8), (16, 8), (16, 16), (8, 32)):
        rs = B.Rasterizer([cam] * V, n, K, ctx=B.Context(tile_w=tile[0], tile_h=tile[1]), dtype=torch.float64)
        img = rs.forward(p, ids, probs=probs)
        grad = rs.backward(p, img, up)
        if ref is None:
            ref = img, grad
        for k in ("color", "depth", "t_final") + (("probs",) if probs else ()):
            close(img[k].cpu().numpy(), ref[0][k].cpu().numpy(), RTOL64, what=f"{tile} {k}")
        close(grad.cpu().numpy(), ref[1].cpu().numpy(), RTOL64, what=f"{tile} against 8x8")


@pytest.mark.parametrize("tile,probs", [((16, 16), False), ((16, 16), True), ((16, 8), True), ((8, 8), True)])
def test_ranges_beyond_the_listed_segments(tile, probs):
    """n faint dots inside one tile, seen in an image of that tile alone and in
    one of 9,604 parts."""
    n, K, big, F = 17000, 3, 784, 100.0
    rng = np.random.default_rng(1)
    z = rng.uniform(1.0, 3.0, n)
    p = np.zeros((14, n), np.float32)
    margin = 2.0   # the 3-sigma box of 0.55 pixels stays inside the tile
    u, v = (rng.uniform(margin, t - margin, n) for t in tile)
    p[0], p[1], p[2] = u * z / F, v * z / F, z
    p[3:6] = np.log(0.01 * z / F)
    p[6] = 1.0
    p[10] = np.log(0.015 / 0.985)
    p[11:] = rng.uniform(0.1, 0.9, (3, n))
    params, ids = to_dev(p), torch.tensor(rng.integers(0, K, n).astype(np.int32), device="cuda")
    g = torch.Generator(device="cuda").manual_seed(4)
    keys = ["d_color", "d_depth", "d_t_final"] + (["d_probs"] if probs else [])
    shape = dict(d_color=(1, 3), d_depth=(1,), d_t_final=(1,), d_probs=(1, K))
    up = {k: torch.randn(*shape[k], tile[1], tile[0], generator=g, device="cuda") for k in keys}
    out = []
    for W, H in (tile, (big, big)):
        cam = dict(width=W, height=H, fx=F, fy=F, cx=0.0, cy=0.0, R=np.eye(3), t=np.zeros(3))
        r = B.Rasterizer([cam], n, K, ctx=B.Context(tile_w=tile[0], tile_h=tile[1]))
        img = r.forward(params, ids, probs=probs)
        ranges = r.frame.buf("ranges", torch.int32).view(-1, 2)
        assert int(ranges[0, 1] - ranges[0, 0]) == n > 255 * 64 + 64
        last = img["last"][0, :tile[1], :tile[0]]
        assert int(last.max()) > 255 * 64 and int((last > 254 * 64).sum()) > 4   # pixels blend into the tail
        full = {k: torch.zeros(*shape[k], H, W, device="cuda") for k in keys}
        for k in keys:
            full[k][..., :tile[1], :tile[0]] = up[k]
        out.append((img["color"][..., :tile[1], :tile[0]], r.backward(params, img, full)))
    close(out[0][0].cpu().numpy(), out[1][0].cpu().numpy(), FWD_RTOL, what="colour")
    close(out[0][1].cpu().numpy(), out[1][1].cpu().numpy(), GRAD_RTOL, what="gradients")


def test_depth_order_of_more_than_64_groups():
    """68.8M items: 8,399 blocks in 66 groups of 128, of which a thread of the
    groups' prefix takes a quarter, more than the 16 that it holds at once."""
    n, V = 4_300_000, 16
    assert -(-(-(-n * V // 8192)) // 128) > 64
    g = torch.Generator(device="cuda").manual_seed(2)
    p = torch.zeros(14, n, device="cuda")
    # depths with ties over two octaves of the key's second byte; far outside the image: no pairs
    p[2] = 1.0 + torch.randint(0, 1 << 20, (n,), generator=g, device="cuda") * 2.0 ** -19
    p[0] = 1e4 * p[2]
    p[3:6] = -5.0
    p[6] = 1.0
    cam = dict(width=64, height=64, fx=50.0, fy=50.0, cx=32.0, cy=32.0, R=np.eye(3), t=np.zeros(3))
    try:
        f = B.Frame(B.Context(tile_w=8, tile_h=8, depth_order=B.DEPTH_ORDER_GLOBAL), [cam] * V, n, 0, 1024)
        f.project_cull_bin(p, torch.zeros(n, dtype=torch.int32, device="cuda"))
        rc, st, pairs = f.read_status()
        assert rc == 0 and st == 0 and pairs == 0
        want = torch.sort(p[2].view(torch.int32).repeat(V), stable=True)
        assert torch.equal(f.buf("depth_keys", torch.int32, n * V), want.values)
        assert torch.equal(f.buf("depth_order", torch.int32, n * V), want.indices.to(torch.int32))
    finally:
        f = want = None
        gc.collect()
        torch.cuda.empty_cache()
