"""The persistent GEMM's order of asynchronous loads, waits and LDS reads, replayed on the host (no GPU needed)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_read_of_the_ring_is_covered_by_a_wait(tmp_path):
    exe = str(tmp_path / "gemm_schedule")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", os.path.join(HERE, "gemm_schedule_driver.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and ", 0 reads not covered" in r.stdout, r.stdout[-3000:]
