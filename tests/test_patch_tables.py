"""The tables of the patch kernels on the CPU: every owner of every grid pair meets its neighbors, each once, and no other point."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_11157_amd", "csrc")

# short and long arcs, whole circles (lengths that are and are not multiples of four), fewer columns than a patch or a workgroup
# has, more walked rows than a table, row counts that leave a segment incomplete, classes of a finer grid on either side, a grid without its pole row
SHAPES = [(0, 17, 32, 17, 32, 0.39), (0, 33, 64, 33, 64, 0.13), (0, 18, 35, 18, 35, 0.5), (0, 9, 12, 9, 12, 3.1), (1, 9, 7, 9, 7, 0.9),
          (1, 6, 4, 6, 4, 1.2), (0, 37, 72, 37, 72, 0.2), (1, 24, 50, 24, 50, 1.4), (0, 33, 64, 17, 32, 0.4), (0, 17, 32, 33, 64, 0.4),
          (0, 19, 57, 9, 19, 0.6), (0, 9, 11, 19, 33, 0.7), (2, 20, 40, 20, 40, 0.5), (3, 21, 44, 11, 22, 0.8), (0, 129, 256, 129, 256, 0.0982), (0, 300, 6, 300, 6, 2.9), (0, 150, 4, 75, 4, 3.1),
          # on either side of what 16 bits hold: the longest circle, and rows that stay classes of a finer latitude
          (1, 2, 32764, 2, 32764, 0.003), (1, 3, 40000, 3, 20000, 0.003), (1, 3, 20000, 3, 40000, 0.003), (1, 2, 32766, 2, 16383, 0.003)]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("patch") / "patch_tables")
    subprocess.run(["hipcc", "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "patch_tables_driver.cpp"),
                    os.path.join(CSRC, "s2_grid.cpp"), os.path.join(CSRC, "s2_trace.cpp"), "-o", exe], check=True, capture_output=True, timeout=600)
    return exe


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_every_owner_meets_its_neighbors_once(driver, shape):
    r = subprocess.run([driver] + [str(x) for x in shape], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.split()[:2] == ["0", "0"], (r.returncode, r.stdout, r.stderr[-500:])


@pytest.mark.parametrize("shape", [(1, 12, 27, 12, 27, 3.14159), (1, 20, 42, 20, 42, 3.14159), (1, 32, 63, 32, 63, 3.14159), (1, 32, 64, 32, 64, 3.14159),
                                   (1, 32, 63, 64, 126, 3.14159), (1, 64, 126, 32, 63, 3.14159)], ids=str)
def test_whole_circles_are_walked_about_once(driver, shape):
    # a patch of 4 x 4 owners needs the 3 step columns more by which its owners lie apart and begins at a multiple of four (a patch of
    # 1 x 16: 15 step); nothing more where chunks fill the circle
    r = subprocess.run([driver] + [str(x) for x in shape], capture_output=True, text=True, timeout=300)
    ratio = shape[1] // shape[3] or 1, shape[3] // shape[1] or 1
    for more, step in zip(r.stdout.split()[2:], ratio):
        assert float(more) <= (3 * step + 6) / 4, r.stdout
        assert float(more) == 0 or min(shape[2], shape[4]) * step % 4
