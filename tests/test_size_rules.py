"""The size rules that the kernels and the host side share (olive_internal.hpp), checked on the
CPU by tests/size_rules_check.cpp under UndefinedBehaviorSanitizer.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = "/opt/rocm/llvm/bin/clang++"


def test_size_rules(tmp_path):
    if not os.path.exists(CXX):
        pytest.skip("ROCm compilers not found")
    exe = str(tmp_path / "size_rules_check")
    subprocess.run([CXX, "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__",
                    "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2609_36246_amd", "csrc"),
                    os.path.join(ROOT, "tests", "size_rules_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr
