"""A kernel with barriers may not let its waves read, each for itself, a word
that other workgroups of the same launch store: some would leave and the
barriers of the others would no longer hold.  The decision is compiled with
g++ (no GPU) with threads as waves and ThreadSanitizer; the counting kernels'
source is looked at for such reads."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2102_02440_amd", "csrc")


def test_block_decision(tmp_path):
    exe = str(tmp_path / "stop_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-pthread",
                           "-fsanitize=thread", "-I", CSRC,
                           os.path.join(HERE, "host", "stop_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "ok" in out.stdout


def test_partition_reads_the_flag_in_one_lane():
    """count_partition_kernel, whose workgroups store the column's flag, and
    the functions it is made of: the flag is loaded by one lane only."""
    src = open(os.path.join(CSRC, "count_kernels.hip")).read()
    src = re.sub(r"//[^\n]*", "", src)
    first = src.index("partition_tiles(const CountArgs")
    body = src[first:src.index("void count_plan_kernel")]
    assert "count_partition_kernel" in body
    assert not re.search(r"(\.|->)bad\b", body)
    reads = re.findall(r"[^;{}]*column_bad\([^;{}]*", body)
    assert len(reads) == 2
    # the loop's read stands in a block of lane 0, the entry's in block_reads
    assert re.search(r"if \(tid == 0\) \{[^}]*column_bad", body)
    assert re.search(r"block_reads\(&s_bad, threadIdx\.x == 0,\s*\[&\] \{ return column_bad", body)
