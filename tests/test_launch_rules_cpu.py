"""Index and choice rules that the kernels share with their host code, checked on the host
(helpers/launch_rules.cpp, under the sanitizers): that no index leaves its array."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent


def test_launch_rules(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("host compiler not available")
    exe = tmp_path / "launch_rules"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + str(ROOT / "paper_2510_23419_amd" / "csrc"), "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", str(ROOT / "tests" / "helpers" / "launch_rules.cpp"), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "rules ok" in r.stdout, r.stdout + r.stderr
