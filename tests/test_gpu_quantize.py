"""The quantised curve's first pass at the edges of its four-wide loads
(lengths around multiples of four, buffers that start between two of them),
and a NaN at its ends: exact counts, and the next call is not disturbed."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BINS = ["u8", "u14", "u16"]


def bins_of(img, m):
    """[0, 1) in m bins; m is a power of two, so the product is exact."""
    return np.clip(np.floor(img * np.float32(m)), 0, m - 1).astype(np.uint8 if m == 256 else np.uint16)


@pytest.mark.parametrize("bins", BINS)
@pytest.mark.parametrize("start", [0, 1, 3])
@pytest.mark.parametrize("shape", [(1,), (3,), (4,), (5,), (7, 147), (2, 3, 1025), (4, 256)], ids=str)
def test_lengths_and_starts(shape, start, bins):
    import paper_1705_02045_amd as ecc
    print(f"\n[gpu] quantise {shape} from {start} {bins}", flush=True)
    n = int(np.prod(shape))
    img = np.random.default_rng(n).uniform(-0.1, 1.1, n).astype(np.float32)
    buf = torch.from_numpy(np.concatenate([np.full(start, np.nan, np.float32), img])).cuda()
    got = ecc.compute_quantized(buf[start:].view(*shape), 0.0, 1.0, bins).cpu().numpy()
    m = ecc.THRESHOLDS[bins]
    assert (got == oracle.curve(bins_of(img.reshape(shape), m), m=m)).all()


@pytest.mark.parametrize("bins", BINS)
@pytest.mark.parametrize("shape", [(4099,), (3, 4, 5, 6)], ids=str)
def test_nan_at_the_ends(shape, bins):
    import paper_1705_02045_amd as ecc
    print(f"\n[gpu] quantise NaN {shape} {bins}", flush=True)
    img = np.random.default_rng(5).uniform(0, 1, shape).astype(np.float32)
    m = ecc.THRESHOLDS[bins]
    ref = oracle.curve(bins_of(img, m), m=m)
    for at in (0, img.size - 1):
        bad = img.copy()
        bad.reshape(-1)[at] = np.nan
        with pytest.raises(ecc.EccError) as ei:
            ecc.compute_quantized(torch.from_numpy(bad).cuda(), 0.0, 1.0, bins)
        assert ei.value.code == ecc.ECC_E_NAN
        assert (ecc.compute_quantized(torch.from_numpy(img).cuda(), 0.0, 1.0, bins).cpu().numpy() == ref).all()
