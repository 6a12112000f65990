"""The GEMM planner (paper_2507_17769_amd/csrc/gemm_plan.h) checked on the host: every plan over a grid of shapes, token counts
and options is one its kernel accepts, a capped plan needs no more memory than the kernels without weights in registers, and the
GPU tests that mean to run the weights-in-registers kernel do so."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PARTIAL, SWIGLU = 0, 1


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "gemm_plan_check")
    cmd = ["g++", "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-I", os.path.join(ROOT, "paper_2507_17769_amd", "csrc"),
           os.path.join(ROOT, "tests", "gemm_plan_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _plans(planner, queries):
    """[(M, N, K, kind, wreg option, capped)] -> [(kernel, row tiles, column groups, K splits, row blocks)] on 256 compute units."""
    r = subprocess.run([planner] + [str(int(x)) for q in queries for x in q], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return [(l.split()[0], *map(int, l.split()[1:])) for l in r.stdout.splitlines()]


def test_every_plan_is_valid_and_capped_plans_stay_within_the_other_kernels_memory(planner):
    r = subprocess.run([planner], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("OK "), r.stdout + r.stderr
    assert int(r.stdout.split()[1]) > 100000


def test_streaming_takes_two_k_shares_where_they_measured_faster(planner):
    # told by the K splits: eight of one share, at most six of two.  4096 columns put two blocks of one share on every compute unit
    # and gain from two up to runs of 16 k-blocks; fewer columns, and more, up to 24
    splits = lambda N, K: {p[3] for p in _plans(planner, [(T, N, K, PARTIAL, 1, 0) for T in (8, 64, 97, 144)])}
    assert splits(4096, 4096) == {3} and splits(2048, 6144) == {6} and splits(3072, 5632) == {4} and splits(5120, 5376) == {2}
    assert all(splits(4096, K) == {8} for K in (4608, 5632, 6144, 14336)) and splits(3072, 7168) == {8}


def test_gpu_tests_of_the_weights_in_registers_gemm_reach_it(planner):
    # test_weights_in_registers_gemm_row_blocks: by the automatic choice, gate/up up to 289 tokens, QKV and down from 257 on
    tokens = [97, 113, 129, 161, 209, 257, 289]
    assert all(p[0] == "wreg" for p in _plans(planner, [(T, 24576, 2048, SWIGLU, 0, 1) for T in tokens]))
    for N, K in ((4096, 2048), (2048, 12288)):
        assert all(p[0] == "wreg" for p in _plans(planner, [(T, N, K, PARTIAL, 0, 1) for T in (257, 289, 321)]))
    # test_weights_in_registers_gemm_every_block: all four projections, any block, one row block and three
    for tm in range(5, 11):
        for nc in (2, 4):
            for N, K, kind in ((1152, 1024, PARTIAL), (1024, 1024, PARTIAL), (4096, 1024, SWIGLU), (1024, 2048, PARTIAL)):
                assert _plans(planner, [(T, N, K, kind, 10 * tm + nc, 1) for T in (16 * tm - 15, 32 * tm + 1)]) == \
                    [("wreg", tm, nc, 1, 1), ("wreg", tm, nc, 1, 3)]
            # ... and its partly filled blocks: three column groups of QKV, 42 of gate/up
            for N, kind in ((192, PARTIAL), (2688, SWIGLU)):
                assert _plans(planner, [(16 * tm + 1, N, 1024, kind, 10 * tm + nc, 1)]) == [("wreg", tm, nc, 1, 2)]
    # test_static_step_8b_layer_runs_the_kernels_of_ps_step_also_where_scratch_is_short
    free, capped = _plans(planner, [(673, 4096, 6144, PARTIAL, 0, cap) for cap in (0, 1)])
    assert free[0] == capped[0] == "wreg" and capped[3] < free[3]
    assert [p[0] for p in _plans(planner, [(97, 28672, 4096, SWIGLU, 0, 1), (294, 4096, 14336, PARTIAL, 0, 1)])] == ["wreg"] * 2


def test_bench_names_the_kernels_that_serve_the_default_workload(planner):
    import bench
    shapes = {"QKV": (10240, 8192, PARTIAL), "O": (8192, 8192, PARTIAL), "gate/up + SwiGLU": (57344, 8192, SWIGLU), "down": (8192, 28672, PARTIAL)}
    names = {"tiled": "gemm_sk_kernel", "wreg": "gemm_wreg_kernel", "wstream": "gemm_wstream_kernel"}
    by_kernel = {}
    for proj, p in zip(shapes, _plans(planner, [(1280, *s, 0, 0) for s in shapes.values()])):
        by_kernel.setdefault(names[p[0]], []).append(proj)
    want = " and ".join(f"{k} ({', '.join(v)})" for k, v in by_kernel.items())
    assert bench.CFG4_GEMM_KERNELS.startswith(want + ":"), want
