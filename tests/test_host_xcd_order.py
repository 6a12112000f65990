"""The order in which blocks take rows and merge groups (paper_2507_17769_amd/csrc/xcd_order.h), checked on the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_block_orders_visit_everything_once_and_spread_over_the_xcds(tmp_path):
    exe = str(tmp_path / "xcd_order_check")
    cmd = ["g++", "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-I", os.path.join(ROOT, "paper_2507_17769_amd", "csrc"),
           os.path.join(ROOT, "tests", "xcd_order_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "OK\n", r.stdout + r.stderr
