"""GPU: the quadric kernels at the box counts where their wavefront changes
shape: sums over 8, 16, 32 and 64 lanes and two boxes per lane (loss and
gradient, 1e-9 relative as elsewhere), and one to four equations per lane
(fit; boxes exact to rounding, so the quadric is recovered to 1e-8)."""
import numpy as np
import pytest
import torch

import oracle as O
from oracle import refine as RF
from paper_2503_02223_amd import binding as B
from tests.test_gpu_refine import _dev, _obj_boxes, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views", [1, 8, 9, 16, 17, 33, 64, 65, 130])
def test_loss_and_gradient_at_lane_counts(views):
    pb = _problem(views, n_obj=2, n_views=views, drop=0.0)
    theta = np.stack([RF.pack(*s) for s in pb["start"]])
    boxes, bo, bv, Ps, wh = _dev(pb)
    out = B.quadric_iou_grad(B.Context(), boxes, bo, bv, Ps, torch.tensor(theta, device="cuda"), img_wh=wh)
    loss, grad = out["loss"].cpu().numpy(), out["grad"].cpu().numpy()
    checked = 0
    for k in range(2):
        ob, ov = _obj_boxes(pb, k)
        if RF.kink_margin(theta[k], ob, pb["Ps"], ov, pb["wh"]) < 1e-6:
            continue
        J, g = np.real(RF.loss(theta[k], ob, pb["Ps"], ov, pb["wh"])), RF.grad(theta[k], ob, pb["Ps"], ov, pb["wh"])
        assert abs(loss[k] - J) <= 1e-9 * max(1.0, abs(J))
        assert np.abs(grad[k] - g).max() <= 1e-9 * np.abs(g).max()
        checked += 1
    assert checked


@pytest.mark.parametrize("views", [3, 16, 17, 33, 64])
def test_fit_at_row_counts(views):
    pb = _problem(100 + views, n_obj=3, n_views=views, drop=0.0, noise_px=0.0)
    boxes, bo, bv, Ps, wh = _dev(pb)
    fit = B.fit_dual_quadric(B.Context(), boxes, bo, bv, Ps, 3, img_wh=wh)
    ref = O.fit_dual_quadric(pb["boxes"], pb["bo"], pb["bv"], pb["Ps"], 3, img_wh=pb["wh"])
    st = fit["status"].cpu().numpy()
    np.testing.assert_array_equal(st, ref["status"])
    for k in np.nonzero(st == 0)[0]:
        assert np.abs(fit["Q"][k].cpu().numpy() - ref["Q"][k]).max() < 1e-8
        assert np.abs(fit["axes"][k].cpu().numpy() - ref["axes"][k]).max() < 1e-8
