"""The box's faces of the dual complex at the edges of their kernel's units
(64 columns by 8 rows, one workgroup per 16 units up to the number of compute
units): counts are whole numbers, so the curves are equal exactly."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(7, 8, 63), (8, 9, 64), (9, 15, 65), (16, 17, 127), (2, 128, 129), (65, 2, 7), (2, 3, 70000),
          (1025, 1100, 2), (9, 8, 2, 65), (2, 64, 7, 9)]


@pytest.mark.parametrize("dtype", ["u8", "u14"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_box_faces(shape, dtype):
    import paper_1705_02045_amd as ecc
    print(f"\n[gpu] box faces {shape} {dtype}", flush=True)
    img = gen.iid(shape, 8, seed=31)
    m = ecc.THRESHOLDS[dtype]
    if dtype == "u14":
        img = (img.astype(np.uint16) * 64 + 63).astype(np.uint16)  # up to the largest value, 16383
    x = torch.from_numpy(img.view(np.int16) if dtype == "u14" else img).cuda()
    assert (ecc.compute_dual(x, dtype).cpu().numpy() == oracle.curve_dual(img, m=m)).all()
