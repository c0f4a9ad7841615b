"""What the spline form leaves out (``left_out`` in ``tetra_spline.h``), built for the host with g++: a pair of equal
energies and points without one in every placement of a block of cubes; and the number of states' grid index and
volumes (``tetra_nos_device.h``). No GPU needed.

Bound: as for the spline form itself (a kept tetrahedron loses 2e-4 of its own density at worst, a tenth of that in
the sum over a block)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, oracle_lib, name):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and the ROCm headers")
    exe = str(tmp_path / name)
    odir = os.path.dirname(oracle_lib.build())
    res = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                          os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1710_10789_amd", "csrc"),
                          os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", exe, "-L", odir,
                          "-ltetra_oracle", f"-Wl,-rpath,{odir}"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    print(out.stdout)
    return {line.split()[0]: line.split()[1:] for line in out.stdout.strip().split("\n")}


def test_ties_beside_points_without_energy(tmp_path, oracle_lib):
    placements, bad, err = _run(tmp_path, oracle_lib, "spline_edges_check")["ties"]
    assert int(placements) > 10000 and int(bad) == 0 and float(err) <= 2e-5


def test_number_of_states_index_and_volumes(tmp_path, oracle_lib):
    """No index may be wrong; the volume form has no cancellation and the oracle's, in FP64 as well, a few digits of
    it (1e-16 times the inverse of the smallest of 20,000 random gaps, about 1e-5)."""
    rows = _run(tmp_path, oracle_lib, "nos_index_check")
    assert int(rows["index"][0]) == 40000 and int(rows["index"][1]) == 0
    assert float(rows["volumes"][0]) <= 1e-10


def test_spline_form_at_the_smallest_limit(tmp_path, oracle_lib):
    """A kept tetrahedron's loss goes with the inverse of the limit: 2e-3 of its own density at a tenth of it, and a
    tenth of that in the sum over a block."""
    rows = _run(tmp_path, oracle_lib, "spline_limit_check")
    assert int(rows["block"][0]) == 60 and int(rows["block"][1]) > 100
    assert float(rows["block"][2]) <= 2e-4 and float(rows["states"][0]) <= 2e-4
