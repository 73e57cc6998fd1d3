"""Every form of the 8-bit kernel with a histogram copy per lane that a launch
can take (one and two in-plane axes, two and four rows per wave, one and two
planes of look-ahead, both conventions): that the launches of these shapes take
it (without a GPU) and that their curves are the oracle's."""
import numpy as np
import pytest

import gen
import oracle
from test_host_paths import program, run  # noqa: F401 (a fixture)

torch = pytest.importorskip("torch")

# shape, stored tiling ("": the rule's), in-plane axes, rows, look-ahead
FORMS = [((16200, 2051), "", 1, 2, 1), ((12000, 1793), "", 1, 2, 1), ((97, 1100, 129), "", 2, 2, 1),
         ((600, 700, 300), "", 2, 2, 2), ((300, 1000, 203), "4 4 16", 2, 4, 2), ((301, 1003, 129), "4 4 16", 2, 4, 2)]


def tiling_file(path, shape, params):
    n1 = shape[1] if len(shape) == 3 else 1
    path.write_text(f"ecc-tiling-v1 1 {len(shape) - 1} {n1} {shape[-1]} {shape[0]} {params} 0.1\n")
    return str(path)


@pytest.mark.parametrize("convention", ["min", "max"])
@pytest.mark.parametrize("shape,params,axes,rows,ahead", FORMS, ids=str)
def test_form_taken(program, tmp_path, convention, shape, params, axes, rows, ahead):  # noqa: F811
    tilings = tiling_file(tmp_path / "t.txt", shape, params) if params else "-"
    line = run(program, "kernel_of", tilings, convention, "x".join(map(str, shape)))[-1]
    transform = 0 if convention == "min" else 1
    assert f"kernelIhLi256ELi{axes}ELi{rows}ELi0ELi{ahead}ELi{transform}ELi6E" in line[-1], line


def test_one_copy_for_large_pictures(program):  # noqa: F811
    """With one in-plane axis and 2^25 voxels or more a single histogram counts."""
    lines = run(program, "kernel_of", "-", "min", "16384x2047", "16384x2048", "8192x8192", "16384x16000")
    assert ["Li6E" in line[-1] for line in lines] == [True, False, False, False], lines


@pytest.mark.gpu
@pytest.mark.parametrize("shape,params,axes,rows,ahead", FORMS, ids=str)
def test_form_counts(tmp_path, shape, params, axes, rows, ahead):
    import paper_1705_02045_amd as ecc
    print(f"\n[gpu] 8-bit copies {shape} {params}", flush=True)
    img = gen.iid(shape, 8, seed=7)
    img.reshape(-1)[::5] = 255  # the largest offset, ties
    img.reshape(-1)[::7] = 0
    t = torch.from_numpy(img).cuda()
    ecc.autotune_reset()
    try:
        if params:
            assert ecc.autotune_load(tiling_file(tmp_path / "t.txt", shape, params)) == 1
        assert np.array_equal(ecc.compute(t, "u8").cpu().numpy(), oracle.curve(img, m=256))
        assert np.array_equal(ecc.compute_max_entry(t, "u8").cpu().numpy(), oracle.curve_max_entry(img, m=256))
    finally:
        ecc.autotune_reset()
