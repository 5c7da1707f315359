"""GPU: only the items inside their view's segment are projected, sorted and
emitted.  Views with empty, one-Gaussian, overlapping and whole segments must
render bitwise like their own Gaussians alone, under both depth orders, with
the pair list of a stable sort by (tile, depth, item), and their gradients sum
over the views (FP32 sums in another order: the parity tolerance)."""
import numpy as np
import pytest
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes
from tests.gpu_util import GRAD_RTOL, close, pair_items, to_dev

pytestmark = pytest.mark.gpu


def _render(p, ids, cams, segments, order, tile=(8, 8)):
    ctx = B.Context(tile_w=tile[0], tile_h=tile[1], depth_order=order)
    r = B.Rasterizer(cams, p.shape[1], 3, ctx=ctx, segments=segments)
    img = r.forward(p, ids)
    return r, img


@pytest.mark.parametrize("order", [B.DEPTH_ORDER_GLOBAL, B.DEPTH_ORDER_TILE])
@pytest.mark.parametrize("n,segments", [(1500, [(0, 0), (7, 1), (100, 1400), (0, 1500)]),
                                        (700, [(0, 700), (300, 400)]), (600, [(0, 0), (600, 0)])])
def test_segments_render_their_own_gaussians(order, n, segments):
    sc = scenes.single_view_scene(seed=n, n=n)
    cam, V = sc["cams"][0], len(segments)
    p, ids = to_dev(sc["params"]), torch.tensor(sc["ids"], device="cuda")
    r, img = _render(p, ids, [cam] * V, segments, order)
    f = r.frame
    _, _, P = f.read_status()
    M = n * V
    cnt = f.buf("counts", torch.int32, M).cpu().numpy().reshape(V, n)
    rect = f.buf("rects", torch.int16, 4 * M).view(M, 4).cpu().numpy().astype(np.int64)
    spl = f.buf("splats", torch.float32, M * B.SPLAT_WORDS).view(M, B.SPLAT_WORDS).cpu().numpy()
    assert P == cnt.sum()
    for v, (lo, c) in enumerate(segments):
        out = np.r_[0:lo, lo + c:n]
        assert (cnt[v, out] == 0).all() and (rect.reshape(V, n, 4)[v, out] == [0, 0, -1, -1]).all()
    # the pair list: every tile of every rectangle, sorted by (tile, depth key, item)
    tx, ty = f.layout.tiles_x, f.layout.tiles_y
    tiles, items = [], []
    for i in np.nonzero(cnt.reshape(-1))[0]:
        x0, y0, x1, y1 = rect[i]
        yy, xx = np.meshgrid(np.arange(y0, y1 + 1), np.arange(x0, x1 + 1), indexing="ij")
        tiles.append((i // n) * tx * ty + yy.ravel() * tx + xx.ravel())
        items.append(np.full(yy.size, i))
    if P:
        tiles, items = np.concatenate(tiles), np.concatenate(items)
        o = np.lexsort((items, spl[items, 6], tiles))
        np.testing.assert_array_equal(f.buf("pair_keys", torch.int32, P).cpu().numpy(), tiles[o])
        np.testing.assert_array_equal(pair_items(f.buf("pair_vals", torch.int32, P).cpu().numpy()), items[o])
    g = torch.Generator(device="cuda").manual_seed(1)
    grads = {k: torch.randn(img[s].shape, generator=g, device="cuda") for k, s in
             (("d_color", "color"), ("d_depth", "depth"), ("d_t_final", "t_final"))}
    got = r.backward(p, img, grads)
    want = torch.zeros_like(p)
    for v, (lo, c) in enumerate(segments):
        if c == 0:
            assert (img["color"][v] == 0).all() and (img["t_final"][v] == 1).all() and (img["last"][v] == -1).all()
            continue
        ps = p[:, lo:lo + c].contiguous()
        rs, one = _render(ps, ids[lo:lo + c].contiguous(), [cam], None, order)
        for k in ("color", "depth", "t_final"):
            assert torch.equal(img[k][v], one[k][0]), (v, k)
        want[:, lo:lo + c] += rs.backward(ps, one, {k: t[v:v + 1].contiguous() for k, t in grads.items()})
    close(got.cpu().numpy(), want.cpu().numpy(), GRAD_RTOL, what="gradients over segments")
