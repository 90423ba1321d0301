"""The tables of the forward by columns on the CPU: every owner meets its neighbors, each once, and the order does not depend on its column."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_11157_amd", "csrc")

# two to four classes, short and long arcs, whole circles, a last segment that is incomplete, more rows than a part holds, a grid without its
# pole row, columns that no multiple of a workgroup's sixteen fills
SHAPES = [(0, 17, 72, 33, 144, 0.4), (1, 12, 76, 20, 228, 0.9), (0, 9, 80, 17, 320, 3.1), (0, 33, 128, 65, 256, 0.12), (0, 90, 72, 100, 144, 2.6),
          (2, 20, 72, 40, 144, 0.5), (3, 21, 84, 42, 168, 0.6), (0, 129, 256, 257, 512, 0.0491)]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("columns") / "column_tables")
    subprocess.run(["hipcc", "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "column_tables_driver.cpp"),
                    os.path.join(CSRC, "s2_grid.cpp"), os.path.join(CSRC, "s2_trace.cpp"), "-o", exe], check=True, capture_output=True, timeout=600)
    return exe


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_every_owner_meets_its_neighbors_once_in_its_own_order(driver, shape):
    r = subprocess.run([driver] + [str(x) for x in shape], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "0\n", (r.returncode, r.stdout, r.stderr[-500:])


@pytest.mark.parametrize("shape", [(0, 17, 72, 17, 72, 0.4), (0, 33, 144, 17, 72, 0.4), (0, 17, 68, 33, 136, 0.4), (0, 17, 74, 33, 148, 0.4)], ids=str)
def test_other_grids_have_none(driver, shape):
    r = subprocess.run([driver] + [str(x) for x in shape], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "none\n", (r.returncode, r.stdout, r.stderr[-500:])
