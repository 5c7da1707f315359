"""GPU: the passes over whole images that are split into runs of pixels (mask
boxes, densification, crop initialization and labels) at sizes around the
splits: strips of 8 rows, rounds of 512 pixels, several rounds per run, views
whose masks start at any byte.  The column of every new Gaussian and every
integer is exact; values come from the oracles."""
import numpy as np
import pytest
import torch

from oracle import learned as OL
from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import learned as L
from paper_2503_02223_amd import scenes
from tests.gpu_util import to_dev
from tests.test_gpu_incremental import _check_params, _dens_inputs, _oracle_densify, _run_densify

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,H,W,K", [(1, 1, 1, 1), (2, 7, 255, 3), (1, 8, 257, 64), (3, 33, 600, 5)])
def test_id_boxes_strips(V, H, W, K):
    rng = np.random.default_rng(H * W)
    idm = rng.integers(-2, K + 2, (V, H, W)).astype(np.int32)   # ids outside [0, K) are no object
    idm[rng.uniform(size=idm.shape) < 0.9] = -1
    boxes, bo, bv = (t.cpu().numpy() for t in B.id_boxes(B.Context(), torch.tensor(idm, device="cuda"), K))
    for v in range(V):
        for k in range(K):
            ys, xs = np.nonzero(idm[v] == k)
            i = v * K + k
            assert bv[i] == v and bo[i] == (k if xs.size else -1)
            want = [xs.min(), ys.min(), xs.max() + 1, ys.max() + 1] if xs.size else [0, 0, 0, 0]
            np.testing.assert_array_equal(boxes[i], want)


@pytest.mark.parametrize("V,H,W", [(1, 1, 3), (3, 64, 32), (2, 41, 151), (2, 369, 401)])
def test_densify_runs(V, H, W):
    rng = np.random.default_rng(H)
    masks, tc, td, tid = _dens_inputs(rng, V, H, W)
    tc, td = tc.astype(np.float32).astype(np.float64), td.astype(np.float32).astype(np.float64)
    cams = scenes.ring_cameras(V, width=W, height=H)
    p_o, id_o, per_view = _oracle_densify(masks, tc, td, tid, cams)
    n = p_o.shape[1]
    p, ids, counts = _run_densify(cams, masks, tc, td, tid, 2, n + 4, torch.float32)
    assert counts[0] == n and list(counts[1:]) == per_view
    np.testing.assert_array_equal(ids[2:2 + n], id_o)
    _check_params(p[:, 2:2 + n], p_o, torch.float32)
    assert (ids[:2] == -99).all() and (ids[2 + n:] == -99).all() and (p[:, 2 + n:] == 123.0).all()


@pytest.mark.parametrize("Bn,H,W", [(1, 16, 16), (3, 32, 48), (2, 208, 176)])
def test_crop_runs(Bn, H, W):
    rng = np.random.default_rng(W)
    crops = rng.uniform(0.2, 1.0, (Bn, 5, H, W)).astype(np.float32)
    crops[:, 4] = rng.uniform(size=(Bn, H, W)) < 0.4
    crops[:, 3][rng.uniform(size=(Bn, H, W)) < 0.1] = 0.0
    cam = scenes.camera(fx=110, fy=110, cx=W / 2, cy=H / 2, width=W, height=H)
    counts = L.valid_counts(crops)
    off = np.concatenate([[0], np.cumsum(counts)])
    x = to_dev(crops)
    params, ids, off_dev = L.init_gaussians(B.Context(), x, [cam] * Bn, off, obj_id=3)
    got = params.cpu().numpy().astype(np.float64)
    want = np.concatenate([OL.plain_init(crops[b], cam)[0] for b in range(Bn)], 1)
    assert got.shape == want.shape and (ids.cpu().numpy() == 3).all()
    _check_params(got, want, torch.float32)
    # labels of perturbed Gaussians, in FP32 of values of order 1 (three log-scales averaged)
    conv = (want + rng.normal(0, 0.1, want.shape)).astype(np.float32)
    lab = L.init_labels(B.Context(), x, [cam] * Bn, off_dev, to_dev(conv)).cpu().numpy()
    for b in range(Bn):
        ref = OL.labels(crops[b], cam, conv[:, off[b]:off[b + 1]].astype(np.float64))
        assert np.abs(lab[b] - ref).max() < 1e-5
