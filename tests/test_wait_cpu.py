"""The host's wait for a kernel's word ends when the device fails, and does not
end while the stream is busy: tests/c/wait_check.cpp plays clock, word and stream."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_wait_ends_with_the_word_or_the_device(tmp_path):
    exe = str(tmp_path / "wait_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2604_02945_amd", "csrc"),
                           os.path.join(ROOT, "tests", "c", "wait_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.count("ok ") == 8
