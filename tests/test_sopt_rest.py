"""The ticket loop of the s-search on the CPU: the text of k_sopt_rest, compiled
for the host with a thread per wave (sanitize/sopt_rest_driver.cpp), has to end
with all its waves also in a block that starts while the last pass publishes the
end of the search, whichever of its waves sees it first, and to serve every share
of every pass in a block that starts in time."""
import re
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent


def kernel_text():
    s = (ROOT / "paper_2011_13695_amd" / "csrc" / "sopt.hip").read_text()
    at = re.search(r"template <typename T, int BITS>\n__global__[^;{]*? k_sopt_rest\(", s).start()
    i = s.index("{", at)
    depth = 0
    for j in range(i, len(s)):
        depth += (s[j] == "{") - (s[j] == "}")
        if depth == 0:
            return s[at:j + 1]
    raise AssertionError("k_sopt_rest does not end")


@pytest.mark.parametrize("scenario", [0, 1, 2])
def test_every_wave_ends(scenario, tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    (tmp_path / "kernel.h").write_text(kernel_text())
    exe = tmp_path / "driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", f'-DKERNEL="{tmp_path / "kernel.h"}"',
                    str(ROOT / "tests" / "sanitize" / "sopt_rest_driver.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), str(scenario)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
