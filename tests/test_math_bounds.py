"""The bounds that qed_math.h states, on the CPU (math_check.cpp: its functions with the hardware's
estimates replaced by values off by up to their documented error).  In units of 2^-53 of the
result, one rounding is at most 1; beside it rsqrt takes half the rounding of x y, and the others'
inner steps are below 0.05: log2 of a mantissa is a table value rounded at 2^-54 and a sum rounded
there; log2_affine adds the product's rounding (half an ulp at 4096 is its unit) and 4095/27 times
the logarithm's."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BOUNDS = {"rsqrt": 1.5, "rcp": 1.05, "exp": 1.05, "pow23": 1.05, "log2": 1.05,
          "affine": 2.0 + 1.05 * 4095.0 / 27.0 / 4096.0, "sqrt": 1.0, "div": 1.0, "edges": 4.0}


def test_errors_stay_within_the_stated_bounds(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not on PATH")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("")
    exe = tmp_path / "math_check"
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", str(tmp_path),
                    "-I", os.path.join(ROOT, "paper_1412_6426_amd", "csrc"),
                    os.path.join(ROOT, "tests", "math_check.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe), "400000"], capture_output=True, text=True, check=True).stdout
    rows = {r.split()[0]: (float(r.split()[1]), int(r.split()[2])) for r in out.splitlines()}
    assert set(rows) == set(BOUNDS)
    for name, (worst, wrong) in rows.items():
        assert worst <= BOUNDS[name], (name, worst)
        assert wrong == 0, name  # sqrt and the quotient: correctly rounded at every argument
