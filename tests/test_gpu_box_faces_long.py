"""The dual complex of a volume whose faces have more rows than one launch's
units can number.  The planes past the first thousand are zero: they only
extend the complex along its last, zero plane, which changes no Euler
characteristic, so the curve is that of the first planes (the oracle's)."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_two_launches_of_faces():
    import paper_1705_02045_amd as ecc
    n0 = 1_950_000_000
    print(f"\n[gpu] dual of {n0} x 2 x 2", flush=True)
    head = gen.iid((1000, 2, 2), 8, seed=9)
    head[-1] = 0
    t = torch.zeros((n0, 2, 2), dtype=torch.uint8, device="cuda")
    t[:1000].copy_(torch.from_numpy(head))
    assert np.array_equal(ecc.compute_dual(t, "u8").cpu().numpy(), oracle.curve_dual(head, m=256))
