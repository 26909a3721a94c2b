"""The counted build's choice (which columns, what key range) and its tiling,
compiled with g++ (no GPU) under AddressSanitizer and
UndefinedBehaviorSanitizer."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2102_02440_amd", "csrc")


def test_count_arithmetic(tmp_path):
    exe = str(tmp_path / "count_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-Wall",
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", CSRC,
                           os.path.join(HERE, "host", "count_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "ok" in out.stdout
