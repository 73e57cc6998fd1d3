"""Launches whose workgroups are planned (whole rounds of the CUs, several
tiles per workgroup, narrower tiles for odd widths): shapes at the edges of
those rules, against the oracle."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# planes just above and below whole rounds, widths of 5, 9, 10, 11 and 17
# segments of 64 columns, more tiles in a plane than workgroups
SHAPES = [(8, 1024, 70), (9, 515, 520), (33, 130, 641), (17, 66, 1030), (40, 300, 300), (25, 1027, 1090),
          (10, 2100, 33), (513, 40, 300)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("dtype", ["u8", "u14", "u16"])
def test_planned_tilings(shape, dtype):
    import paper_1705_02045_amd as ecc
    bits = {"u8": 8, "u14": 14, "u16": 16}[dtype]
    img = gen.value_noise(shape, bits, 1 << max(0, bits - 8), seed=sum(shape))
    t = torch.from_numpy(img if bits == 8 else img.view(np.int16)).cuda()
    want = oracle.curve(img, m=1 << bits)
    assert np.array_equal(ecc.compute(t, dtype).cpu().numpy(), want)
    out = torch.zeros(1 << bits, dtype=torch.int64, device="cuda")
    ecc.compute_async_noalloc(t, out, dtype)
    assert np.array_equal(out.cpu().numpy(), want)
