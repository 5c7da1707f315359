"""GPU: radix passes whose grid does not fit on the device at once (counts per
block of 8192, prefix over groups of 128 blocks, scatter).  Every Gaussian is
a dot inside one tile, so the pair list is known exactly: one pair per item,
in (tile, depth bits, item) order, with exact tile ranges."""
import numpy as np
import pytest
import torch

from paper_2503_02223_amd import binding as B
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu

W, H, F = 640, 480, 500.0
TX = W // 8


def _dots(n, z0, z1, seed=0):
    """n dots of 0.01 pixels at tile centres, depths in [z0, z1] with many ties."""
    rng = np.random.default_rng(seed)
    tile = rng.integers(0, TX * (H // 8), n)
    z = np.float32(z0) + np.float32(z1 - z0) * (rng.integers(0, max(2, n // 3), n) / max(2, n // 3)).astype(np.float32)
    p = np.zeros((14, n), np.float32)
    p[0] = (tile % TX * 8 + 4 - W / 2) * z / F
    p[1] = (tile // TX * 8 + 4 - H / 2) * z / F
    p[2] = z
    p[3:6] = np.log(0.01 * z / F)
    p[6] = 1.0
    p[10] = 2.0
    cam = dict(width=W, height=H, fx=F, fy=F, cx=W / 2, cy=H / 2, R=np.eye(3), t=np.zeros(3))
    return p, tile, cam


def _check(n, z0, z1, capacity):
    p, tile, cam = _dots(n, z0, z1)
    r = B.Rasterizer([cam], n, 0, capacity=capacity,
                     ctx=B.Context(tile_w=8, tile_h=8, depth_order=B.DEPTH_ORDER_GLOBAL))
    r.bin(to_dev(p), torch.zeros(n, dtype=torch.int32, device="cuda"), grow=False)
    f = r.frame
    torch.cuda.synchronize()
    rc, st, P = f.read_status()
    assert rc == 0 and st == 0 and P == n
    do = f.buf("depth_order", torch.int32, n).cpu().numpy().astype(np.int64)
    np.testing.assert_array_equal(do, np.argsort(p[2].view(np.uint32), kind="stable"))
    order = do[np.argsort(tile[do], kind="stable")]
    np.testing.assert_array_equal(f.buf("pair_vals", torch.int32, n).cpu().numpy(), order)
    np.testing.assert_array_equal(f.buf("pair_keys", torch.int32, n).cpu().numpy(), tile[order])
    rng = f.buf("ranges", torch.int32).cpu().numpy().reshape(-1, 2)
    cnt = np.bincount(tile, minlength=rng.shape[0])
    np.testing.assert_array_equal(rng[:, 1] - rng[:, 0], cnt)
    np.testing.assert_array_equal(rng[cnt > 0, 0], (np.cumsum(cnt) - cnt)[cnt > 0])


@pytest.mark.parametrize("n", [1, 8191, 8192, 8193, 128 * 8192, 128 * 8192 + 1])
def test_pairs_in_a_large_pair_list(n):
    _check(n, 1.0, 3.0, 1 << 24)


@pytest.mark.parametrize("n", [3, 4097, 1 << 18])
def test_pairs_in_a_resident_pair_list(n):
    _check(n, 1.0, 3.0, n + 1000)


@pytest.mark.parametrize("z1", [1.9, 300.0])   # three depth passes suffice; four are needed
@pytest.mark.parametrize("n", [(1 << 18) - 1, 5_000_001])
def test_depth_order_of_many_items(n, z1):
    _check(n, 1.0, z1, n + 1000)
