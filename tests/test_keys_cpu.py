"""The keys that selections rank tokens by, and the digit that two kernels must
agree on, for z and d in range and far out of it: tests/c/keys_check.cpp."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_keys_and_first_digits(tmp_path):
    exe = str(tmp_path / "keys_check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-Wno-format-security",
                           "-Wno-format-extra-args", "-I", os.path.join(ROOT, "paper_2604_02945_amd", "csrc"),
                           os.path.join(ROOT, "tests", "c", "keys_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
