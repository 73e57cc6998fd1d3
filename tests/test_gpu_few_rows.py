"""Volumes whose planes have a few rows: workgroups of as many rows of waves as
the plane has, or of one wide row."""
import numpy as np
import pytest

import gen
import oracle

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(300, 5, 2048), (290, 6, 2053), (700, 5, 385), (600, 9, 2048), (400, 10, 769),
                                   (900, 7, 600)], ids=str)
@pytest.mark.parametrize("bits", [8, 14])
def test_planes_of_few_rows(shape, bits):
    import paper_1705_02045_amd as ecc
    print(f"\n[gpu] few rows {shape} {bits}", flush=True)
    img = gen.iid(shape, bits, seed=11)
    t = torch.from_numpy(img.view(np.int16) if bits > 8 else img).cuda()
    got = ecc.compute(t, "u8" if bits == 8 else "u14").cpu().numpy()
    assert np.array_equal(got, oracle.curve(img, m=1 << bits))
