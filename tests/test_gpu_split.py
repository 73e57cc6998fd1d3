"""Float keys by their lowest 9 bits within tiles of 16384: lengths at the
tiles' edges, buffers that start between two 16-byte loads, runs that are
empty, crowded in some tiles only, and more tiles than one round of the
waves takes (736).  Distinct values and curves equal the oracle's exactly."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def check(img, start=0):
    import paper_1705_02045_amd as ecc
    rk, rc = oracle.curve_float(img)
    buf = torch.from_numpy(np.concatenate([np.zeros(start, np.float32), img.reshape(-1)])).cuda()
    gk, gc = ecc.compute(buf[start:].view(*img.shape), dtype="f32")
    assert np.array_equal(gk.cpu().numpy().view(np.uint32), rk.view(np.uint32))
    assert np.array_equal(gc.cpu().numpy(), rc)


def values(n, seed, crowded=()):
    """n floats in [0.25, 2); the tiles in `crowded` have their lowest 9 bits zero."""
    rng = np.random.default_rng(seed)
    bits = rng.integers(0x3E800000, 0x40000000, size=n, dtype=np.uint32)
    for t in crowded:
        bits[t * 16384:(t + 1) * 16384] &= np.uint32(0xFFFFFE00)
    return bits.view(np.float32)


@pytest.mark.parametrize("start", [0, 1])
@pytest.mark.parametrize("n", [2, 511, 16383, 16384, 16385, 32768, 49153])
def test_split_edges(n, start):
    print(f"\n[gpu] split {n} from {start}", flush=True)
    check(values(n, n), start)


@pytest.mark.parametrize("crowded", [(), (0, 1, 735, 736), tuple(range(100, 200))], ids=["even", "ends", "block"])
def test_split_many_tiles(crowded):
    n = 737 * 16384 + 5
    print(f"\n[gpu] split {n}, {len(crowded)} crowded tiles", flush=True)
    check(values(n, 7, crowded))


@pytest.mark.parametrize("k", [1, 2, 16383, 16384, 16385])
def test_few_values(k):
    """k distinct values: up to 16384 the changes are added in LDS."""
    print(f"\n[gpu] {k} values", flush=True)
    rng = np.random.default_rng(k)
    img = rng.integers(0, k, size=70 * 30 * 40)
    img[rng.permutation(img.size)[:k]] = np.arange(k)  # every value occurs
    check((img - k // 2).astype(np.float32).reshape(70, 30, 40))
