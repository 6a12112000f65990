"""The GEMM planner (paper_2507_17769_amd/csrc/gemm_plan.h) checked on the host: every plan over a grid of shapes, token counts
and options is one its kernel accepts, and a capped plan needs no more memory than the kernels without weights in registers."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_plan_is_valid_and_capped_plans_stay_within_the_other_kernels_memory():
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "gemm_plan_check")
        cmd = ["g++", "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-I", os.path.join(ROOT, "paper_2507_17769_amd", "csrc"),
               os.path.join(ROOT, "tests", "gemm_plan_check.cpp"), "-o", exe]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        r = subprocess.run([exe], capture_output=True, text=True)
        assert r.returncode == 0 and r.stdout.startswith("OK "), r.stdout + r.stderr
        assert int(r.stdout.split()[1]) > 100000
