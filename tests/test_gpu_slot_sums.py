"""GPU: the slot sums of an item do not depend on the first slot of the items
after its wave of 64.  A scan whose wait gave up can leave any first slot
there; it is written from the host here, into the state buffer."""
import pytest
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stray", [0, 5, 0x7fffffff, -1])
@pytest.mark.parametrize("order", [B.DEPTH_ORDER_GLOBAL, B.DEPTH_ORDER_TILE])
def test_slots_end_with_the_wave(order, stray):
    n, K = 2000, 3
    sc = scenes.single_view_scene(seed=4, n=n)
    p, ids = to_dev(sc["params"]), torch.tensor(sc["ids"], device="cuda")
    r = B.Rasterizer(sc["cams"], n, K, ctx=B.Context(tile_w=8, tile_h=8, depth_order=order))
    img = r.forward(p, ids)
    g = torch.Generator(device="cuda").manual_seed(1)
    up = {k: torch.randn(img[s].shape, generator=g, device="cuda") for k, s in
          (("d_color", "color"), ("d_depth", "depth"), ("d_t_final", "t_final"))}
    want = r.backward(p, img, up)
    f = r.frame
    seq = torch.arange(n, device="cuda")
    if order == B.DEPTH_ORDER_GLOBAL:
        seq = f.buf("depth_order", torch.int32, n).long()
    counts, offsets = f.buf("counts", torch.int32, n), f.buf("offsets", torch.int32, n)
    waves = [w for w in range(64, n, 64) if counts[seq[w]] > 0 and want[:, seq[w - 1]].abs().max() > 0]
    assert len(waves) >= 4
    for w in waves[:4]:
        kept = offsets[seq[w]].clone()
        offsets[seq[w]] = stray
        f.render_backward(img, up)
        got = torch.empty_like(p)
        f.project_backward(p, got)
        offsets[seq[w]] = kept
        before = seq[max(0, w - 64):w]
        assert torch.equal(got[:, before], want[:, before]), w
