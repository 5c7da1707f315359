"""GPU: mask boxes of id maps with more rows than one launch takes strips for
(2^27 rows are 2^32 threads at a strip of 8 rows each) and with long rows."""
import pytest
import torch

from paper_2503_02223_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [((1 << 27) + 1000, 1), ((1 << 19) + 9, 3), (9, 1 << 20)])
def test_boxes_of_large_maps(H, W):
    idm = torch.full((1, H, W), -1, dtype=torch.int32, device="cuda")
    idm[0, H - 1, W - 1] = 0
    idm[0, 5, 0] = 1
    idm[0, H - 2, W // 2] = 1
    boxes, bo, _ = B.id_boxes(B.Context(), idm, 3)
    assert bo.tolist() == [0, 1, -1]
    assert boxes.tolist() == [[W - 1, H - 1, W, H], [0, 5, W // 2 + 1, H - 1], [0, 0, 0, 0]]
