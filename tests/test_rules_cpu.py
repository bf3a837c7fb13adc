"""The rules by which plans and calls choose their launches, checked on the CPU
at the sizes where they were measured (tests/c/rules_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "c", "rules_check.cpp")
CSRC = os.path.join(ROOT, "paper_1511_00175_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    out = tmp_path_factory.mktemp("rules") / "rules_check"
    build = ["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-D__HIP_PLATFORM_AMD__",
             "-isystem", f"{ROCM}/include", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}", SRC, "-o", str(out)]
    r = subprocess.run(build, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.mark.parametrize("rule", ["copies", "packed", "shapes", "short_steps", "split_plans", "noalloc", "resident", "sgd"])
def test_rule(exe, rule):
    r = subprocess.run([str(exe), rule], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "as measured" in r.stdout
