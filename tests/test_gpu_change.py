"""The change kernel's tiles (rows and planes per lane, 62 emitting lanes per
wave, walks along axis 0) at their edges, against the oracle."""
import pathlib
import re
import shutil
import subprocess

import numpy as np
import pytest

import gen
import oracle

torch = pytest.importorskip("torch")

ROOT = pathlib.Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_1705_02045_amd" / "csrc"
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def check(img):
    import paper_1705_02045_amd as ecc
    rk, rc = oracle.curve_float(img)
    gk, gc = ecc.compute(torch.from_numpy(np.ascontiguousarray(img, dtype=np.float32)).cuda(), dtype="f32")
    assert np.array_equal(gk.cpu().numpy().view(np.uint32), rk.view(np.uint32))
    assert np.array_equal(gc.cpu().numpy(), rc)


# lanes: 1, 62 to 66, 124 to 128 flattened positions; rows per lane: 4 with
# one line axis, 2 with two; walks of one plane, and of odd and even lengths
EDGES = [(62,), (63,), (64,), (65,), (66,), (124,), (126,), (127,), (3, 61), (8, 64), (9, 65), (16, 127),
         (2, 1000), (17, 3), (3, 4, 31), (8, 5, 13), (9, 3, 64), (1, 8, 63), (5, 9, 21), (2, 16, 16), (11, 2, 2),
         (3, 2, 2, 31), (2, 3, 5, 13), (9, 2, 4, 32), (8, 5, 3, 21), (4, 7, 2, 64), (3, 4, 9, 7), (2, 2, 2, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", EDGES, ids=str)
@pytest.mark.parametrize("kind", ["noise", "ties", "special"])
def test_change_tile_edges(shape, kind):
    rng = np.random.default_rng(len(shape) * 1000 + sum(shape))
    if kind == "noise":
        img = gen.value_noise_f32(shape, sigma=0.2, seed=5)
    elif kind == "ties":
        img = rng.integers(-2, 3, size=shape).astype(np.float32)
    else:
        img = rng.choice(np.array([-0.0, 0.0, 1e-42, -1e-42, 3.5, np.inf, -np.inf], dtype=np.float32), size=shape)
    check(img)


# 4-D integer images: shapes at the tiles' edges, every dtype and convention
EDGES_4D = [(2, 2, 2, 2), (3, 4, 5, 31), (8, 2, 3, 62), (9, 5, 4, 13), (17, 3, 2, 21), (4, 7, 6, 64), (10, 9, 11, 12)]
CONVENTIONS = [("u8", "min"), ("u8", "max"), ("u8", "dual"), ("u14", "min"), ("u14", "max"), ("u14", "dual"),
               ("u16", "min")]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", EDGES_4D, ids=str)
@pytest.mark.parametrize("dtype,convention", CONVENTIONS, ids=str)
def test_change_4d_integers(shape, dtype, convention):
    import paper_1705_02045_amd as ecc
    m = ecc.THRESHOLDS[dtype]
    rng = np.random.default_rng(sum(shape) + m)
    # the lowest and highest values among others, with ties
    img = rng.choice(np.array([0, 1, m // 2, m - 2, m - 1]), size=shape)
    img = np.where(rng.random(shape) < 0.6, img, rng.integers(0, m, size=shape))
    img = img.astype(np.uint8 if dtype == "u8" else np.uint16)
    t = torch.from_numpy(img if dtype == "u8" else img.view(np.int16)).cuda()
    if convention == "min":
        got, want = ecc.compute(t, dtype), oracle.curve(img, m=m)
    elif convention == "max":
        got, want = ecc.compute_max_entry(t, dtype), oracle.curve_max_entry(img, m=m)
    else:
        got, want = ecc.compute_dual(t, dtype), oracle.curve_dual(img, m=m)
    assert np.array_equal(got.cpu().numpy(), want)


def test_no_subtraction_with_a_lane_shift():
    """v_subrev_u32 with a lane shift on its first source shifted the second
    on the card: the change kernel's build holds no such subtraction."""
    if not pathlib.Path(HIPCC).exists():
        pytest.skip("hipcc not available")
    cmd = [HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature",
           "-Xclang", "-packed-fp32-ops", "-I", str(ROOT / "include"), "-I", str(CSRC), "--offload-device-only",
           "-S", "-o", "-", str(CSRC / "ecc_change.hip")]
    asm = subprocess.run(cmd, check=True, capture_output=True, text=True).stdout
    assert re.search(r"v_\w+_dpp", asm)
    assert not re.findall(r"v_sub\w*_dpp.*", asm)
