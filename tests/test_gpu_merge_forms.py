"""Merges of 256-bin count rows on both sides of 256 rows: one workgroup up to
it, column sums and a scan above.  With ECC_INT_PLAN=0 an image of n0 planes
of one row each gives ceil(n0 / 8) rows; both conventions (the largest-value
one lands reversed)."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("rows", [255, 256, 257, 320, 513, 1000])
def test_rows(monkeypatch, rows):
    import paper_1705_02045_amd as ecc
    monkeypatch.setenv("ECC_INT_PLAN", "0")
    img = gen.iid((8 * rows - 3, 100), 8, seed=rows)
    t = torch.from_numpy(img).cuda()
    for _ in range(2):  # the second call starts from the first one's status
        assert np.array_equal(ecc.compute(t, "u8").cpu().numpy(), oracle.curve(img, m=256))
        assert np.array_equal(ecc.compute_max_entry(t, "u8").cpu().numpy(), oracle.curve_max_entry(img, m=256))
