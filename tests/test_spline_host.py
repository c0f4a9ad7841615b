"""The spline form of the tetrahedron sums (``tetra_spline.h``: neighbours, coefficients of a grid point from
the reciprocals of its energy differences, with and without left-out tetrahedra, fourth differences of
truncated powers) built for the host with g++ and checked against the FP64 oracle's tetrahedra on blocks
of cubes with random, equal and nearly equal energies. No GPU needed.

Bound: the terms of a tetrahedron that is kept cancel to 2e-4 of its own density at worst (the limit of
``kDegenerate``, with a gap just above it); summed over a block's 162 tetrahedra of similar density the
error stays below a tenth of that. A wrong neighbour, ring or sign gives O(1)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_spline_form_against_the_oracle(tmp_path, oracle_lib):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and the ROCm headers")
    exe = str(tmp_path / "spline_check")
    odir = os.path.dirname(oracle_lib.build())
    res = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                          os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1710_10789_amd", "csrc"),
                          os.path.join(ROOT, "tests", "host", "spline_check.cpp"), "-o", exe, "-L", odir,
                          "-ltetra_oracle", f"-Wl,-rpath,{odir}"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    print(out.stdout)
    rows = {line.split()[0]: line.split()[1:] for line in out.stdout.strip().split("\n")}
    blocks, left, err = int(rows["block"][0]), int(rows["block"][1]), float(rows["block"][2])
    assert blocks == 60 and left > 100 and err <= 2e-5
    assert float(rows["states"][0]) <= 2e-5
    assert int(rows["division"][0]) == 0
