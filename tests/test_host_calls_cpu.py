"""The host side of the library on the CPU, against a HIP runtime of the test's own that
notes every call and can fail a launch (tests/helpers/host_calls.cpp): what a call
leaves behind when a launch fails, what the tuner times, when steps are captured."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2203_11043_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_calls") / "host_calls")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-rdynamic",
                    "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "helpers", "host_calls.cpp"), "-o", exe,
                    "-L", PACKAGE, "-lgccd", "-Wl,-rpath," + PACKAGE,
                    "-Wl,--allow-shlib-undefined"], check=True)
    return exe


@pytest.mark.parametrize("case", ["join", "autotune", "graphs"])
def test_host_calls(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
