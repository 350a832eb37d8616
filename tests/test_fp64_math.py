"""The device's fp64 elementary functions (csrc/fp64_math.hpp), built for the host
with estimates worse than the hardware's: over all 2^23 uniforms a photon can
draw, the azimuth's sine and cosine and the optical depth round to libm's fp32
values; the others are within two ulps of fp64 (2^-52 each) of the true value."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(HERE, "..", "paper_2201_13191_amd", "csrc", "fp64_math.hpp")


def test_fp64_math(tmp_path):
    src = open(HEADER).read().replace("#include <hip/hip_runtime.h>", "")
    (tmp_path / "m.hpp").write_text(src)
    exe = tmp_path / "check"
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-mfma", "-w",
                    f'-DFP64_MATH_HEADER="{tmp_path / "m.hpp"}"',
                    os.path.join(HERE, "fp64_math_check.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert [int(v) for v in out[:3]] == [0, 0, 0]
    assert all(float(v) <= 2 * 2.0 ** -52 for v in out[3:]), out
