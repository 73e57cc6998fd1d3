"""Merges of count rows around the block sizes of their kernels: at most 256
rows of 256 columns in one workgroup, other rows 64 at a time in one launch
and the scan of 1024 columns per workgroup in a second."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# n0 x 100 planes: from 8 planes on a workgroup walks 8 (rows = ceil(n0 / 8))
CASES = [("u8", n0) for n0 in (2040, 2048, 2049, 2056, 4100)] + [("u14", n0) for n0 in (1, 504, 512, 513, 2050)] + [
    ("u16", n0) for n0 in (1, 513, 2050)]


@pytest.mark.parametrize("dtype,n0", CASES, ids=str)
def test_merge_rows(dtype, n0):
    import paper_1705_02045_amd as ecc
    bits = {"u8": 8, "u14": 14, "u16": 16}[dtype]
    img = gen.iid((n0, 100), bits, seed=n0)
    t = torch.from_numpy(img if bits == 8 else img.view(np.int16)).cuda()
    for _ in range(2):  # the second call starts from the first one's status
        assert np.array_equal(ecc.compute(t, dtype).cpu().numpy(), oracle.curve(img, m=1 << bits))
    if dtype != "u16":
        assert np.array_equal(ecc.compute_max_entry(t, dtype).cpu().numpy(), oracle.curve_max_entry(img, m=1 << bits))
