"""The chunk count of a two-phase flush is evaluated by every workgroup that
needs it, and all have to agree: compiled with and without fused multiply-adds
(no GPU) it is the same number everywhere, and within what the slab and the
survivors allow."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2102_02440_amd", "csrc")


def test_chunks_do_not_depend_on_the_compilation(tmp_path):
    printed = []
    for k, flags in enumerate((["-O1", "-ffp-contract=off"],
                               ["-O3", "-mfma", "-ffp-contract=fast"],
                               ["-O2", "-mfma", "-ffast-math"])):
        exe = str(tmp_path / ("chunks_check%d" % k))
        subprocess.check_call(["g++", "-std=c++17", "-Wall", *flags, "-I", CSRC,
                               os.path.join(HERE, "host", "chunks_check.cpp"), "-o", exe])
        out = subprocess.run([exe], capture_output=True, text=True)
        print(flags, out.stdout)
        assert out.returncode == 0, out.stdout + out.stderr
        printed.append(out.stdout)
    assert "too" in printed[0]
    assert len(set(printed)) == 1
