"""The library's host side without a GPU: what it allocates, launches, gives
back and reports, seen by the HIP runtime calls that host_paths.c defines."""
import os
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
LIB = pathlib.Path(os.environ.get("ECC_LIB_DIR", ROOT / "paper_1705_02045_amd"))
ROCM = pathlib.Path(shutil.which("hipcc") or "/opt/rocm/bin/hipcc").resolve().parents[1]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not (ROCM / "include" / "hip" / "hip_runtime_api.h").exists():
        ROCM_INC = pathlib.Path("/opt/rocm/include")
    else:
        ROCM_INC = ROCM / "include"
    out = tmp_path_factory.mktemp("host") / "host_paths"
    subprocess.run(["gcc", "-O1", "-std=gnu11", "-w", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", str(ROCM_INC),
                    "-I", str(ROOT / "include"), str(ROOT / "tests" / "host_paths.c"), str(LIB / "libecc.so"),
                    f"-Wl,-rpath,{LIB}", "-Wl,--allow-shlib-undefined", "-o", str(out)], check=True)
    return out


def run(program, *args):
    r = subprocess.run([str(program), *args], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return [line.split() for line in r.stdout.splitlines()]


def records(lines, key):
    """The "key value" pairs of the lines that start with key."""
    return [dict(zip(line[1::2], map(int, line[2::2]))) for line in lines if line[0] == key]


ECC_OK, ECC_E_RANGE, ECC_E_NAN, ECC_E_NOMEM = 0, -2, -3, -6


def test_float_call_leaves_no_status_behind(program):
    """A float call that fails after its kernels were launched clears the
    status word that they set and waits for them: the next call on the stream
    is not disturbed."""
    lines = run(program, "float_exits")
    failed = records(lines, "float")
    assert {c["rc"] for c in failed} <= {ECC_E_NOMEM, ECC_E_NAN}
    assert sum(c["rc"] == ECC_E_NOMEM for c in failed) >= 6
    assert all(c["status"] == 0 for c in failed), failed
    assert all(c["rc"] == ECC_OK for c in records(lines, "next")), lines


def test_dual_call_leaves_no_status_behind(program):
    """The dual curve of a 4-D image that fails after its volume was launched:
    the status word is clear and the caller's stream has been waited for."""
    lines = run(program, "dual_exits")
    failed = records(lines, "dual")
    assert {c["rc"] for c in failed} == {ECC_E_NOMEM, ECC_E_RANGE}
    assert any(c["rc"] == ECC_E_NOMEM and c["launched"] for c in failed)
    assert all(c["status"] == 0 for c in failed), failed
    assert all(c["waits"] for c in failed if c["launched"]), failed
    assert all(c["rc"] == ECC_OK for c in records(lines, "next")), lines


def test_kept_blocks_give_way(program):
    """The device blocks that finished streams left are bounded, and given
    back when another call finds no memory; a call that fails all the same
    leaves no error of the runtime behind."""
    lines = run(program, "kept_blocks")
    assert records(lines, "begin") == [{"rc": ECC_OK}]
    kept = [int(line[2]) for line in lines if line[1] == "kept"]
    assert 0 < kept[0] <= 256 << 20 and 32 << 20 <= kept[1] <= 256 << 20
    assert records(lines, "call") == [{"rc": ECC_OK}]
    assert records(lines, "none") == [{"rc": ECC_E_NOMEM, "error": 0}]


def test_small_float_image_on_a_nearly_full_card(program):
    """The bits of the distinct values take some MiB however small the image;
    where they find no memory the keys are sorted instead."""
    assert records(run(program, "float_nearly_full"), "float") == [{"rc": ECC_OK}]


def test_batch_memory_is_within_the_footprints(program):
    """What a run's planned tiles make it allocate is at most 32 MiB more than
    ecc_job_footprint counts for its images (admission adds those up), and no
    more than that where the card has no more."""
    lines = run(program, "batch_rows")
    assert len(lines) == 18
    for line in lines:
        r = dict(zip(line[1::2], map(int, line[2::2])))
        assert r["rc"] == ECC_OK and r["bytes"] <= r["bound"], line


def test_batch_tuner_reports_the_depth_in_use(program):
    """After ecc_batch_autotune a run cuts an image into tiles of
    max(min_planes, n0 / split) planes, with the values that it returned."""
    tuned = records(run(program, "batch_tuned"), "tuned")
    assert len(tuned) == 3
    for t in tuned:
        depth = max(t["min_planes"], -(-t["n0"] // t["split"]))
        assert t["rc"] == ECC_OK and t["tiles"] == -(-t["n0"] // depth), t


def test_loaded_tilings_are_taken_as_they_are(program, tmp_path):
    """A stored tiling's workgroups follow from its parameters (200 planes of
    300 x 300 in at least tiles_per_cu * 256 tiles, walks of 8 planes or more);
    only the rule's own parameters are planned."""
    lines = run(program, "tilings", str(tmp_path / "tiling.txt"))
    rule = records(lines, "rule")[0]["grid"]
    want = []
    for rows, per_cu, wx in ((2, 16, 16), (2, 8, 8), (4, 4, 8)):
        w = min(wx, 5)  # 300 columns are 5 segments of 64
        tiles = -(-5 // w) * -(-(-(-300 // rows)) // (16 // w))
        walk = max(8, -(-200 // min(200, -(-256 * per_cu // tiles))))
        all_tiles = tiles * -(-200 // walk)
        per = -(-all_tiles // (256 * per_cu)) if all_tiles > 256 * per_cu else 1
        want.append(-(-all_tiles // per))
    loaded = records(lines, "loaded")
    assert all(x["rc"] == 1 for x in loaded)
    assert [x["grid"] for x in loaded] == [rule, *want], (rule, want)
    assert rule not in want


def test_4d_chunks_are_cut_below_2_30_values(program):
    """The change kernel counts in int32: a launch has less than 2^30 values."""
    pushes = records(run(program, "stream_4d"), "push")
    assert len(pushes) == 6
    for p in pushes:
        assert p["rc"] == ECC_OK and p["launches"] * ((1 << 30) - 1) >= p["values"], p


def test_dual_of_volumes_with_very_long_faces(program):
    """Faces of more rows than one launch's units can number go to several."""
    duals = records(run(program, "dual_long"), "dual")
    assert [d["rc"] for d in duals] == [ECC_OK] * 5
    assert [d["launches"] > 1 for d in duals] == [True, True, True, False, False]


def test_narrow_8_bit_launches_are_split_finely(program):
    """8-bit workgroups of up to four waves: about four tiles per CU where that
    gives walks of 16 planes or more."""
    shapes = [(1000000, 8), (100000, 130), (2000000, 2), (200000, 2, 2), (100000, 4, 4), (20000, 4, 64), (16384, 64)]
    lines = run(program, "kernel_of", "-", "min", *["x".join(map(str, s)) for s in shapes])
    for shape, line in zip(shapes, lines):
        r = dict(zip(line[1:5:2], map(int, line[2:5:2])))
        walk = -(-shape[0] // 1024)
        assert r["rc"] == ECC_OK and r["grid"] == -(-shape[0] // walk), line


def test_float_images_of_narrow_planes_take_no_more_memory(program):
    """Two key buffers, the records' slots (8 bytes, twice the voxels where rows
    of two fill lanes of four), some per mille of tables, and the bits."""
    for f in records(run(program, "float_memory"), "float"):
        assert f["rc"] == ECC_OK and f["bytes"] <= 28 * f["voxels"] + (32 << 20), f


def test_wide_16_bit_planes_fill_the_cus(program, tmp_path):
    """Planes of somewhat more tiles than CUs are cut into several tiles per
    workgroup, so that three in four CUs or more have work (16-bit passes: one
    workgroup per CU)."""
    lines = run(program, "grids_u16", "2000x700x700", "256x700x750", "500x1000x700", "1000x600x800", "1024x1024x1024")
    grids = [int(line[4]) for line in lines]
    assert all(192 <= g <= 256 for g in grids), lines


def test_planes_of_few_rows_leave_no_row_of_waves_idle(program):
    """Three rows of waves: workgroups of 4 x 3 waves (8 x 2 left a quarter of
    them idle); two rows and four fill 8 x 2."""
    shapes = ["10000x5x2048", "2810x6x5418", "10000x4x2048", "10000x8x2048"]
    lines = run(program, "kernel_of", "-", "min", *shapes)
    assert [int(line[line.index("waves") + 1]) for line in lines] == [12, 12, 16, 16], lines
