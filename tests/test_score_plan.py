"""The sharing-out of kvp_score_tokens (csrc/score_plan.h, host arithmetic): a C++ program walks it over its range.  What a
plan writes has to fit the workspace size that callers are told, for every shape, and each shape has to run the kernel
that was measured to be the faster one there."""
import os
import subprocess

import pytest

import test_gpu_score_edges as edges
import test_gpu_score_large as large

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("score_plan") / "score_plan")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_14946_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "score_plan.cpp")], check=True)
    return exe


def _wide(exe, L, H, T, G, W):
    return subprocess.run([exe, *map(str, (L, H, G * H, W, T))], check=True, capture_output=True, text=True).stdout.strip() == "1"


def test_every_plan_fits_the_workspace_and_covers_every_key_once(plan):
    out = subprocess.run([plan], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    walks, sizes = map(int, out.stdout.split())
    assert walks > 2000 and sizes > 400_000


def test_short_rows_and_calls_of_few_units_run_the_chunked_kernel(plan):
    for G, W in [(1, 8), (1, 32), (4, 32), (7, 32), (8, 64)]:
        for L, H, T in [(80, 8, 256), (80, 8, 1024), (32, 8, 2048), (257, 8, 64), (8, 8, 4096), (1, 8, 16384), (2, 8, 8192)]:
            assert not _wide(plan, L, H, T, G, W), (L, H, T, G, W)
        assert _wide(plan, 32, 8, 32768, G, W)


def test_shapes_of_the_large_call_tests_run_the_throughput_kernel(plan):
    for L, H, T, G, W, _, _ in large.THROUGHPUT_SHAPES:
        assert _wide(plan, L, H, T, G, W), (L, H, T, G, W)
    for L, H, T, G, W, _, _ in large.SHAPES:
        assert not _wide(plan, L, H, T, G, W), (L, H, T, G, W)


def test_shapes_of_the_edge_tests_run_both_kernels(plan):
    assert [_wide(plan, *s) for s in edges.BOTH] == [True, True, False]
    assert _wide(plan, 2, 8, 49152, 4, 32) and _wide(plan, 2, 8, 49152, 8, 64) and not _wide(plan, 1, 8, 4096, 4, 32)
