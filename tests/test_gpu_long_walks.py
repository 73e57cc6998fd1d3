"""Images of nearly 2^31 planes (the most that an image may have): the walks of
the last tile end at the image's end.  All planes are 7 but the first and the
last ones, which are noise: planes of 7 between them are one contractible
piece, so the curve is that of the same ends with one plane of 7 between (the
oracle's)."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N0 = 2 ** 31 - 1 - 4


@pytest.mark.parametrize("plane,dtype", [((2, 2), "u8"), ((2,), "u8"), ((3,), "u14")], ids=str)
def test_last_planes_are_counted(plane, dtype):
    import paper_1705_02045_amd as ecc
    print(f"\n[gpu] {N0} planes of {plane} {dtype}", flush=True)
    head, tail = (gen.iid((300, *plane), 8, seed=k) for k in (3, 4))
    # (one plane of 7 between the ends: a product with an interval around it)
    small = np.concatenate([head, np.full((1, *plane), 7, np.uint8), tail])
    kind = torch.uint8 if dtype == "u8" else torch.int16
    t = torch.full((N0, *plane), 7, dtype=kind, device="cuda")
    t[:300].copy_(torch.from_numpy(head).to(kind))
    t[-300:].copy_(torch.from_numpy(tail).to(kind))
    want = oracle.curve(small if dtype == "u8" else small.astype(np.uint16), m=ecc.THRESHOLDS[dtype])
    assert np.array_equal(ecc.compute(t, dtype).cpu().numpy(), want)
