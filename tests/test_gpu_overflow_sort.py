"""GPU: bin() enqueues the sort before it knows whether the pair list
overflowed.  A list that is far too short, one pair too short and exactly long
enough must all end in the same pair list and image, under both depth orders
and on a stream of the caller's."""
import pytest
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [B.DEPTH_ORDER_GLOBAL, B.DEPTH_ORDER_TILE])
@pytest.mark.parametrize("n,tile", [(2000, (8, 8)), (20000, (16, 16))])
def test_short_lists_grow_to_the_same_result(n, tile, order):
    sc = scenes.single_view_scene(seed=n, n=n)
    p, ids = to_dev(sc["params"]), torch.tensor(sc["ids"], device="cuda")
    ctx = lambda: B.Context(tile_w=tile[0], tile_h=tile[1], depth_order=order)  # noqa: E731
    ref = B.Rasterizer(sc["cams"], n, 3, ctx=ctx(), capacity=1 << 20)
    img = ref.forward(p, ids, probs=True)
    _, _, P = ref.frame.read_status()
    assert P > 1000
    want = {k: ref.frame.buf(k, torch.int32)[:P].clone() for k in ("pair_keys", "pair_vals")}
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    for cap, stream in ((1, None), (P // 2, st), (P - 1, None), (P, st)):
        r = B.Rasterizer(sc["cams"], n, 3, ctx=ctx(), capacity=cap)
        torch.cuda.synchronize()
        out = r.forward(p, ids, probs=True, stream=stream)
        torch.cuda.synchronize()
        rc, status, npairs = r.frame.read_status()
        assert rc == 0 and status == 0 and npairs == P and r.frame.capacity >= P
        for k, v in want.items():
            assert torch.equal(r.frame.buf(k, torch.int32)[:P], v), (cap, k)
        for k in ("color", "depth", "t_final", "probs"):
            assert torch.equal(out[k], img[k]), (cap, k)
