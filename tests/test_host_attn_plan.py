"""The attention plan checked on the host over random mixtures of chunks and decodes, under AddressSanitizer and
UndefinedBehaviorSanitizer."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plans_cover_every_page_and_fit_the_device(tmp_path):
    csrc = os.path.join(ROOT, "paper_2507_17769_amd", "csrc")
    exe = str(tmp_path / "attn_plan_check")
    cmd = ["g++", "-O2", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", csrc, os.path.join(ROOT, "tests", "attn_plan_check.cpp"),
           os.path.join(csrc, "planner.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("OK "), r.stdout + r.stderr
