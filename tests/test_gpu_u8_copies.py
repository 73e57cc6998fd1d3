"""8-bit launches with a histogram copy per lane (workgroups of more than 12
waves that walk at least 16 planes): interior waves load byte pairs, waves at
x = 0 and at the far edges single bytes; ragged rows and columns, both ranks,
both conventions, each rows-per-wave and look-ahead form."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(100, 1501, 203), (130, 1030, 64), (97, 1100, 129), (16500, 2051), (33000, 1024)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("rows,ahead", [("2", "1"), ("2", "2"), ("4", "2")])
def test_u8_lane_copies(monkeypatch, shape, rows, ahead):
    import paper_1705_02045_amd as ecc
    monkeypatch.setenv("ECC_INT_ROWS", rows)
    monkeypatch.setenv("ECC_INT_PD", ahead)
    img = gen.iid(shape, 8, seed=7)
    img.reshape(-1)[:: 5] = 255  # the largest offset, ties
    img.reshape(-1)[:: 7] = 0
    t = torch.from_numpy(img).cuda()
    assert np.array_equal(ecc.compute(t, "u8").cpu().numpy(), oracle.curve(img, m=256))
    # max_f(t) = 1 - min_{255 - f}(254 - t): the largest-value form by the smallest-value oracle
    want = np.empty(256, dtype=np.int64)
    low = oracle.curve(255 - img, m=256)
    want[255] = 1
    want[:255] = 1 - low[254::-1]
    assert np.array_equal(ecc.compute_max_entry(t, "u8").cpu().numpy(), want)
