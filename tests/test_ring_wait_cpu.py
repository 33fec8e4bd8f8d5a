"""Host check of the many-row GEMM's wait counts (ring_wait_count in ring.h) against the order in which
the kernel's two loops issue their copies and loads, over more ring shapes than the kernel is built for."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2510_05421_amd", "csrc")


def test_every_stage_has_landed_when_the_ring_reads_it(tmp_path):
    exe = tmp_path / "ring_wait_check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, os.path.join(HERE, "ring_wait_check.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout
