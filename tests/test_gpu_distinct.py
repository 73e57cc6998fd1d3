"""The distinct values of float images by bits (up to 32 sign and binade-pair
groups, the keys' top bytes) and by the sort (more), at the line between them
and with the keys' lowest 9 bits evenly spread, skewed and constant."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def check(img):
    import paper_1705_02045_amd as ecc
    rk, rc = oracle.curve_float(img)
    gk, gc = ecc.compute(torch.from_numpy(np.ascontiguousarray(img)).cuda(), dtype="f32")
    assert np.array_equal(gk.cpu().numpy().view(np.uint32), rk.view(np.uint32))
    assert np.array_equal(gc.cpu().numpy(), rc)


@pytest.mark.parametrize("groups", [1, 2, 31, 32, 33, 64])
@pytest.mark.parametrize("low", ["spread", "constant", "skewed"])
def test_distinct_groups(groups, low):
    """groups top bytes; the lowest 9 bits of the keys random, all zero (one
    bucket, shared by many workgroups), or zero for nine voxels in ten."""
    shape = (7, 61, 601)
    rng = np.random.default_rng(groups)
    frac = rng.integers(0, 1 << 23, size=shape, dtype=np.uint32)
    if low == "constant":
        frac &= np.uint32(0xFFFFFE00)
    elif low == "skewed":
        frac = np.where(rng.random(shape) < 0.9, frac & np.uint32(0xFFFFFE00), frac).astype(np.uint32)
    g = rng.integers(0, groups, size=shape).astype(np.uint32)
    # group i: sign i & 1, exponent 10 + 4 (i >> 1): one top byte each
    bits = ((g & 1) << 31) | ((10 + 4 * (g >> 1)) << 23) | frac
    img = bits.astype(np.uint32).view(np.float32)
    assert np.isfinite(img).all()
    check(img)


@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 8191, 8192, 8193, 16385])
def test_distinct_sizes(n):
    """Lengths at the key tiles' and the curve tiles' edges."""
    check(gen.value_noise_f32((n,), sigma=0.3, seed=n))
