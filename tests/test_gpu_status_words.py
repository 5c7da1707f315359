"""GPU: the pinned words behind Rasterizer.bin are shared by every Rasterizer
of the process, so what mode the first one was made or used under (inference
mode, a default device, a graph capture) must not show in the next, and a copy
of a Rasterizer keeps the words that it shares."""
import copy
import gc

import pytest
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import scenes
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture
def scene():
    sc = scenes.single_view_scene(seed=1, n=500)
    p, ids = to_dev(sc["params"]), torch.tensor(sc["ids"], device="cuda")
    want = B.Rasterizer(sc["cams"], 500, 3).forward(p, ids)["color"].clone()
    kept, B._status_words = B._status_words, []   # the next one allocates a block
    yield (lambda: B.Rasterizer(sc["cams"], 500, 3)), p, ids, want
    B._status_words = kept


def _uses(make, p, ids, want):
    assert torch.equal(make().forward(p, ids)["color"], want)


def test_made_under_inference_mode(scene):
    make, p, ids, want = scene
    with torch.inference_mode():
        r = make()
        assert torch.equal(r.forward(p, ids)["color"], want)
    assert torch.equal(r.forward(p, ids)["color"], want)
    _uses(*scene)


def test_made_under_a_default_device(scene):
    make, p, ids, want = scene
    with torch.device("cuda"):
        _uses(*scene)
    _uses(*scene)


def test_made_inside_a_capture(scene):
    """A Rasterizer made while a graph is being captured (its state cleared in
    the graph) allocates no status words: it cannot wait for them there."""
    make, p, ids, want = scene
    make().forward(p, ids, grow=False)   # kernels loaded
    torch.cuda.synchronize()
    B._status_words = []
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        r = make()
        img = r.forward(p, ids, grow=False)
    for _ in range(3):
        img["color"].zero_()
        g.replay()
        assert torch.equal(img["color"], want)
    assert not B._status_words
    _uses(*scene)


def test_a_copy_keeps_the_words(scene):
    make, p, ids, want = scene
    r = make()
    assert torch.equal(r.forward(p, ids)["color"], want)
    c = copy.copy(r)
    del r
    gc.collect()
    free = {w.data_ptr() for w in B._status_words}
    assert torch.equal(c.forward(p, ids)["color"], want)
    assert c._status.words.data_ptr() not in free and len(free) == 255
    del c
    gc.collect()
    assert len(B._status_words) == 256
