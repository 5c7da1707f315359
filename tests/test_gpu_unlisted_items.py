"""GPU: the state's per-item buffers hold every (view, Gaussian) item, those
outside their view's segment too: no tiles, an empty record, a culled item's
depth key, a place at the end of the depth order (which stays a permutation),
and the first slot that the scan over the whole order gives.  So after other
segments on the same state, and after a frame without any."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu

N = 700
LISTS = [[(0, 0), (7, 1), (100, 500), (0, N)], [(0, N), (300, 400), (0, 0), (N, 0)], [(0, 0)] * 4, None,
         [(650, 50), (0, 650), (3, 3), (10, 0)]]


def _check(f, segments, order, V):
    _, _, P = f.read_status()
    M = N * V
    listed = np.ones((V, N), bool)
    if segments is not None:
        listed[:] = False
        for v, (lo, c) in enumerate(segments):
            listed[v, lo:lo + c] = True
    listed = listed.reshape(-1)
    spl = f.buf("splats").view(f.tdtype).view(M, B.SPLAT_WORDS).double().cpu().numpy()
    cnt = f.buf("counts", torch.int32, M).cpu().numpy().astype(np.int64)
    rect = f.buf("rects", torch.int16, 4 * M).view(M, 4).cpu().numpy()
    off = f.buf("offsets", torch.int32, M).cpu().numpy().astype(np.int64)
    keys = f.buf("depth_keys", torch.int32, M).cpu().numpy().view(np.uint32)
    assert (spl[~listed] == 0).all() and (cnt[~listed] == 0).all() and (rect[~listed] == [0, 0, -1, -1]).all()
    key = np.where(listed & (spl[:, 6] > 0), spl[:, 6].astype(np.float32).view(np.uint32), np.uint32(0xffffffff))
    if order == B.DEPTH_ORDER_GLOBAL:
        do = f.buf("depth_order", torch.int32, M).cpu().numpy().astype(np.int64)
        np.testing.assert_array_equal(np.sort(do), np.arange(M))
        np.testing.assert_array_equal(keys, key[do])
        assert (np.diff(keys.astype(np.int64)) >= 0).all()
        np.testing.assert_array_equal(do[listed.sum():], np.nonzero(~listed)[0])
    else:
        do = np.arange(M)
        np.testing.assert_array_equal(keys, key)
    np.testing.assert_array_equal(off[do], np.cumsum(cnt[do]) - cnt[do])
    assert cnt.sum() == P


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("order", [B.DEPTH_ORDER_GLOBAL, B.DEPTH_ORDER_TILE])
def test_every_item_has_its_entries(order, dtype):
    sc = scenes.single_view_scene(seed=3, n=N)
    p, ids = to_dev(sc["params"], dtype), torch.tensor(sc["ids"], device="cuda")
    p[2, ::9] = -1.0   # culled ones among the listed
    V = 4
    f = B.Frame(B.Context(tile_w=8, tile_h=8, depth_order=order), sc["cams"] * V, N, 3, 1 << 16, dtype=dtype)
    for name in ("splats", "rects", "counts", "offsets", "depth_keys", "depth_order"):
        f.buf(name).fill_(0x5A5A5A5A)
    for segments in LISTS + LISTS[:1]:
        arr = None if segments is None else (ctypes.c_int64 * (2 * V))(*np.asarray(segments).ravel().tolist())
        f.desc.segments = ctypes.cast(arr, ctypes.POINTER(ctypes.c_int64)) if segments is not None else None
        for _ in range(2):   # the second frame finds the unlisted items as it needs them
            f.project_cull_bin(p, ids)
            f.sort()
            _check(f, segments, order, V)
            p[2] += 0.05
