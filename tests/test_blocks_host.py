"""Host checks (no GPU) of what set-up packs for the triangle kernels' blocks,
through the driver tests/host/blocks2d.cpp."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2105_02127_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    tmp = str(tmp_path_factory.mktemp("blocks2d"))
    exe = os.path.join(tmp, "blocks2d")
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-ffp-contract=off",
                    os.path.join(ROOT, "tests", "host", "blocks2d.cpp"), "-o", exe],
                   check=True, capture_output=True)
    return tmp, exe


def _write(tmp, tag, m):
    with open(os.path.join(tmp, tag + ".txt"), "w") as fh:
        fh.write(f"{m.xy.shape[0]} {m.tri.shape[0]} {m.period[0]} {m.period[1]}\n")
    np.ascontiguousarray(m.xy, np.float64).tofile(os.path.join(tmp, tag + ".xy"))
    np.ascontiguousarray(m.tri, np.int32).tofile(os.path.join(tmp, tag + ".tri"))


def _run(exe, *args):
    r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-2000:]
    return r.stdout


def _mesh(driver, m, order, variant=0, characteristic=0):
    tmp, exe = driver
    _write(tmp, "m", m)
    w = _run(exe, "mesh", tmp, "m", order, variant, characteristic).split()
    return dict(zip(w[::2], map(int, w[1::2])))


def test_block_layouts_do_not_overlap(driver):
    # every order, wavefront count, member count, one and two buffers; in
    # characteristic variables the Gram matrices lie over the members just read,
    # and at order 3 (about 200 members per block) they are the longer of the two
    assert "ok" in _run(driver[1], "layout")


@pytest.mark.parametrize("order", [3, 4, 5, 6])
@pytest.mark.parametrize("kind", ["periodic", "box", "strip"])
def test_characteristic_block_layouts_of_meshes(driver, order, kind):
    m = {"periodic": lambda: inputs.jittered_periodic_mesh(30, 2),
         "box": lambda: inputs.jittered_box_mesh(31, 23, 3),
         "strip": lambda: inputs.jittered_box_mesh(400, 12, 4, lx=400.0, ly=12.0)}[kind]()
    s = _mesh(driver, m, order, characteristic=1)
    assert s["lds"] <= 160 * 1024


def test_inline_assembly_names_m0():
    # a copy to LDS sets m0; unnamed, the compiler may keep something else there
    for name in ("kernels.hpp", "kernels3.hpp"):
        src = open(os.path.join(ROOT, "paper_2105_02127_amd", "csrc", name)).read()
        for asm in re.findall(r"asm volatile\((.*?)\);", src, flags=re.S):
            text, _, operands = asm.rpartition(":")
            if re.search(r"s_mov_b32 m0|\bm0,", asm):
                assert '"m0"' in operands, asm


def test_setup_stores_no_operators(driver):
    # order 6: the device arrays take 3.0 KB a cell, the operators would take 8.3 KB
    m = inputs.jittered_periodic_mesh(150, 3)
    s = _mesh(driver, m, 6)
    assert s["peak_kb"] * 1024 < 8000 * m.n_cell, s


@pytest.mark.parametrize("order", [3, 6])
def test_tiles_of_runs(driver, order):
    # the packing that set-up falls back to where bisected tiles do not fit
    tmp, exe = driver
    _write(tmp, "r", inputs.jittered_box_mesh(20, 17, 5))
    for line in _run(exe, "solve", tmp, "r", order, 7, "runs").splitlines():
        assert float(line.split()[-1]) <= 1.0, line


# (angle, growth): radii 1 : e^growth over a sector of that angle; 0: a jittered
# periodic mesh; -1: a box stretched eightfold
@pytest.mark.parametrize("order", [3, 4, 5, 6])
@pytest.mark.parametrize("angle,growth", [(4.0, 6.0), (4.0, 4.0), (1.5, 8.0), (1.5, 4.0), (0, 0), (-1, 0)])
def test_least_squares_of_the_block_data(driver, order, angle, growth):
    """Coefficients from the records, slots and normal inverses, or the operators of
    kept cells, in the kernels' arithmetic, against 128 bits.  The bar: set-up
    keeps the operators of a cell unless the bound of each stencil's normal matrix
    is below 2e-13 or below 10 (large: 30) times what an operator formed in FP64
    costs; errors are a fifth (a tenth) of the bound at most, so each stencil's
    face values are within 2e-13 plus twice the operator's worst.  Over a mesh the
    worst face value stays below the operators' worst."""
    if angle > 0:
        m = inputs.graded_sector_mesh(64, 3, angle, growth)
    elif angle == 0:
        m = inputs.jittered_periodic_mesh(32, 3)
    else:
        m = inputs.jittered_box_mesh(32, 32, 3, lx=1.0, ly=0.125)
    tmp, exe = driver
    _write(tmp, "s", m)
    out = _run(exe, "solve", tmp, "s", order, 11 if angle > 0 else 3)
    print(out)
    for line in out.splitlines():
        w = line.split()
        assert float(w[-1]) <= 1.0, out
        assert float(w[6]) <= float(w[8]), out
