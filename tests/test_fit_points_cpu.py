"""The calibration fit walks its points without leaving 32 bits, up to the most that its entry
point takes: the kernel's own code, compiled for the host."""
import os
import subprocess

import pytest

from paper_1505_05655_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fit") / "fit_points")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    res = subprocess.run(
        ["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-Wno-unknown-pragmas",
         "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", build.INCLUDE, "-I",
         build.CSRC, os.path.join(HERE, "fit_points.cpp"), build.LIB,
         f"-Wl,-rpath,{os.path.dirname(build.LIB)}", f"-L{rocm}/lib", f"-Wl,-rpath,{rocm}/lib",
         "-lamdhip64", "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return out


@pytest.mark.parametrize("points", [1, 7, 8, 9, 1000, 2147483640, 2147483641, 2147483647])
def test_every_point_is_taken_once(program, points):
    res = subprocess.run([program, str(points)], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.returncode
    # Targets of 1 and samples of 0: the sum of the targets over the number of points.
    assert res.stdout.split() == ["1", "0", "0", "0"]
