"""Float images of many distinct values (over 16384) most of whose changes fall on
few of them, which are summed in LDS slots (2048 per workgroup): clipped, mostly
zero, with more frequent values than slots, and with no frequent one."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [(250000,), (500, 501), (60, 64, 65), (22, 23, 24, 21)], ids=str)
@pytest.mark.parametrize("kind", ["clipped", "sparse", "frequent", "even"])
def test_hot_values(shape, kind):
    import paper_1705_02045_amd as ecc
    print(f"\n[gpu] {kind} {shape}", flush=True)
    rng = np.random.default_rng(len(shape))
    img = rng.standard_normal(shape).astype(np.float32)
    if kind == "clipped":
        img = np.clip(img, -0.4, 0.4)
    elif kind == "sparse":
        img = np.where(rng.random(shape) < 0.9, np.float32(0), np.abs(img)).astype(np.float32)
    elif kind == "frequent":
        img = np.where(rng.random(shape) < 0.8, rng.integers(-2500, 2500, shape).astype(np.float32), img)
    rk, rc = oracle.curve_float(img)
    assert rk.size > 16384
    gk, gc = ecc.compute(torch.from_numpy(np.ascontiguousarray(img)).cuda(), dtype="f32")
    assert np.array_equal(gk.cpu().numpy().view(np.uint32), rk.view(np.uint32))
    assert np.array_equal(gc.cpu().numpy(), rc)
