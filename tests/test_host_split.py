"""How a fused scan's workgroups are shared out to the slice groups whose
columns are not counted, compiled with g++ (no GPU) under AddressSanitizer and
UndefinedBehaviorSanitizer: every chunk of every live group by exactly one
workgroup."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2102_02440_amd", "csrc")


def test_live_split(tmp_path):
    exe = str(tmp_path / "split_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-Wall",
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", CSRC,
                           os.path.join(HERE, "host", "split_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "ok" in out.stdout
