"""GPU: the network's convolutions where a workgroup walks a run of tiles.  One
workgroup per CU at the widest layer, 256 CUs: a single tile, one tile more
than workgroups (runs of two, the last of one) and runs of three whose last is
short, each tile an image of its own so that a run crosses images.  Output and
gradients against the oracle, to the dot-product bound of four BF16 steps per
term that the network's other tests derive."""
import numpy as np
import pytest
import torch

from oracle import learned as OL
from paper_2503_02223_amd import crops as CR
from paper_2503_02223_amd import learned as L
from tests.gpu_util import to_dev
from tests.test_gpu_learned import _abs_layers, _close_net, _layers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 257, 515])
def test_runs_of_tiles_match_oracle(count):
    full = CR.make_crops(21, (count + 63) // 64)
    tiles = full.reshape(full.shape[0], full.shape[1], 8, 16, 8, 16).transpose(0, 2, 4, 1, 3, 5)
    # (from a tile of the first crop's centre on, which has valid pixels)
    tiles = np.ascontiguousarray(np.roll(tiles.reshape(-1, full.shape[1], 16, 16), -27, axis=0)[:count])
    layers = _layers(4)
    layers32 = [(np.float32(w).astype(np.float64), np.float32(b).astype(np.float64)) for w, b in layers]
    labels = np.random.default_rng(5).normal(0, 0.5, size=(count, 5, 16, 16)).astype(np.float32)
    chan_w = [2.0, 0.5, 4.0, 4.0, 4.0]
    net = L.Net(theta=L.pack_layers(layers))
    rg = to_dev(tiles)
    out = net.forward(rg)
    net.loss_backward(rg, out, to_dev(labels), chan_w)
    torch.cuda.synchronize()
    got_out = out.cpu().numpy()
    acts, outs = [], []
    for b in range(count):
        a, o = OL.net_forward(OL.net_input(tiles[b]), layers32)
        acts.append(a)
        outs.append(o)
        _close_net(got_out[b], o, OL.conv3x3(a[3], OL.bf16(np.abs(layers32[3][0])), np.zeros(6)), f"output {b}")
    ok = np.stack([OL.valid_pixels(c) for c in tiles])
    _, g_out = OL.net_loss(np.stack(outs), labels, ok, chan_w)
    grads, bounds = None, None
    add = lambda u, v: v if u is None else [(x[0] + y[0], x[1] + y[1]) for x, y in zip(u, v)]
    for b in range(count):
        grads = add(grads, OL.net_backward(acts[b], layers32, g_out[b]))
        bounds = add(bounds, OL.net_backward(acts[b], _abs_layers(layers32), np.abs(g_out[b])))
    got = L.unpack_theta(net.grad.cpu().numpy())
    for l in range(4):
        _close_net(got[l][0], grads[l][0], bounds[l][0], f"dW layer {l + 1}")
        _close_net(got[l][1], grads[l][1], bounds[l][1], f"db layer {l + 1}")
