"""The FP64 functions of the kernels (csrc/f64_math.h) on the CPU, compiled for the
host with reciprocal and root estimates of 22 bits, against long double: root mean
square and largest error in ulp. A correctly rounded result is off by 0.289 and
0.5; the deviates of a Box-Muller pair made with correctly rounded functions by
0.532."""
import platform
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent

# function: (largest root mean square, largest error)
BARS = {"log": (0.31, 1.0), "log_u": (0.31, 1.0), "sqrt": (0.2895, 0.501), "div": (0.2895, 0.501),
        "sin": (0.30, 1.0), "cos": (0.30, 1.0), "exp": (0.32, 1.1), "deviate": (0.55, 3.0)}


def test_errors_in_ulp(tmp_path):
    if not shutil.which("g++") or platform.machine() != "x86_64":
        pytest.skip("g++ with an 80-bit long double not available")
    text = (ROOT / "paper_2011_13695_amd" / "csrc" / "f64_math.h").read_text()
    (tmp_path / "f64_math_host.h").write_text(text.replace("#include <hip/hip_runtime.h>", ""))
    exe = tmp_path / "driver"
    subprocess.run(["g++", "-std=c++17", "-O2", "-mfma", "-ffp-contract=off", "-Wno-unknown-pragmas", f"-I{tmp_path}",
                    str(ROOT / "tests" / "sanitize" / "f64_driver.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=120).stdout
    got = {a: (float(b), float(c)) for a, b, c in (line.split() for line in out.splitlines())}
    print(got)
    for name, (rms, most) in BARS.items():
        assert got[name][0] <= rms and got[name][1] <= most, (name, got[name])
