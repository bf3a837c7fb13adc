"""The rule that gives short plans to the split kernel, and the association of
its runs, checked on the CPU for every worker count under AddressSanitizer and
UndefinedBehaviorSanitizer (tests/c/shape_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "c", "shape_check.cpp")
CSRC = os.path.join(ROOT, "paper_1511_00175_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_split_shapes_are_valid(tmp_path):
    exe = tmp_path / "shape_check"
    build = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror", "-ffp-contract=off",
             "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__",
             "-isystem", f"{ROCM}/include", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}", SRC, "-o", str(exe)]
    r = subprocess.run(build, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all shapes valid" in r.stdout
