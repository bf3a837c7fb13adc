"""The overlap check that every call runs on its buffers (csrc/fc_alias.h),
compared on the CPU with the rule applied to every pair of buffers, under
AddressSanitizer and UndefinedBehaviorSanitizer (tests/c/alias_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "c", "alias_check.cpp")
CSRC = os.path.join(ROOT, "paper_1511_00175_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_verdicts_match_the_pairwise_rule(tmp_path):
    exe = tmp_path / "alias_check"
    build = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror", "-fsanitize=address,undefined",
             "-fno-sanitize-recover=all", f"-I{CSRC}", SRC, "-o", str(exe)]
    r = subprocess.run(build, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all verdicts agree" in r.stdout
