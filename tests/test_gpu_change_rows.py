"""4-D images of 16 bits are counted in 8 to 64 rows that workgroups share (a row
per 8192 voxels): sizes around the steps, few and many values, resident and in
chunks, against the oracle."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [(2, 2, 2, 2), (8, 16, 16, 32), (13, 17, 16, 19), (30, 31, 29, 33)], ids=str)
@pytest.mark.parametrize("values", ["two", "sixteen", "all"])
def test_shared_rows(shape, values):
    import paper_1705_02045_amd as ecc
    img = gen.iid(shape, 16, seed=sum(shape))
    if values == "two":
        img = np.where(img < 30000, 0, 65535).astype(np.uint16)
    elif values == "sixteen":
        img = (img & np.uint16(15)).astype(np.uint16)
    want = oracle.curve(img, m=65536)
    t = torch.from_numpy(img.view(np.int16)).cuda()
    for _ in range(2):  # the second call starts from the first one's rows
        assert np.array_equal(ecc.compute(t, "u16").cpu().numpy(), want)
    st = ecc.Stream(shape, "u16")
    st.push(t[:1])
    st.push(t[1:])
    assert np.array_equal(st.finish(), want)
