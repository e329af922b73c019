"""Index arithmetic of the matrix-core engine compiled for the host (tests/host):
its row accesses on grids near the 32-bit limits (row_io.hip), the tiles and
barriers of its waves (wave_run.hip), and the row blocks of every axis in its size
class (axis_classes.hip)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _build(name, tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp(name) / name)
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2003_13569_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", name + ".hip"), "-o", exe],
                   check=True, capture_output=True, text=True)
    return exe


@pytest.fixture(scope="module")
def row_io(tmp_path_factory):
    return _build("row_io", tmp_path_factory)


# wave_run: every tile once, as many barriers from every wave of a block;
# axis_classes: every position once, no row block of padding alone
@pytest.mark.parametrize("name", ["wave_run", "axis_classes"])
def test_index_arithmetic_of_the_engine(name, tmp_path_factory):
    res = subprocess.run([_build(name, tmp_path_factory)], capture_output=True, text=True,
                         timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr


# last axes of up to 16 blocks whose FP32 offsets fit 32 bits, with a tile across
# the species boundary (inner extent not a multiple of 16): FP64 offsets past 2^32
# in the first three
@pytest.mark.parametrize("ny,nx,nz", [(1023, 1023, 401), (901, 900, 351), (1023, 1022, 477),
                                      (513, 511, 289), (5, 3, 67)])
def test_rows_of_fp64_arrays_beside_fp32_fields(row_io, ny, nx, nz):
    res = subprocess.run([row_io, str(ny), str(nx), str(nz)], capture_output=True, text=True,
                         timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
