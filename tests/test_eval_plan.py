"""The blocks of kvp_eval_configs' attention launch (csrc/eval_plan.h, host arithmetic): each segment has one block, and each
shape the arrangement that was measured to be the fastest there."""
import os
import subprocess

import pytest

import test_gpu_eval_compare as compare

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("eval_plan") / "eval_plan")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_14946_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "eval_plan.cpp")], check=True)
    return exe


def _run(exe, *args):
    out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    return out.stdout.split()


def test_every_segment_has_one_block(plan):
    walk, grouped, cell = map(int, _run(plan))
    assert walk > 30 and grouped > 1000 and cell > 100


@pytest.mark.parametrize("cells,streams,T,pv,levels,want", [
    (256, 2, 8192, "default", (2458, 8192), "grouped"),              # two codecs fill the chip: unequal segments
    (256, 3, 8192, "matrix", (2458, 8192), "grouped"),
    (256, 10, 8192, "default", (2048, 4096, 6144, 8192), "cell"),    # the utility sweep
    (64, 10, 5003, "matrix", (1251, 2502, 3753, 5003), "cell"),
    (256, 10, 300, "matrix", (75, 150, 225, 300), "walk"),           # short segments
    (256, 10, 300, "default", (75, 150, 225, 300), "cell"),
    (256, 10, 300, "fp32", (75, 150, 225, 300), "cell"),
    (128, 10, 300, "matrix", (75, 150, 225, 300), "walk"),           # three rounds of blocks for two and a half of work
    (112, 10, 300, "matrix", (75, 150, 225, 300), "cell"),           # three rounds for 2.2
    (256, 10, 300, "matrix", (75, 150, 225), "cell"),                # a quarter of the tokens kept by nobody
    (128, 4, 2048, "matrix", (1024,), "walk"),                       # only the reference's second segments do not fit
    (128, 4, 2048, "default", (1024,), "cell"),
    (2, 4, 10666, "default", (3200, 10666), "cell"),                 # unequal segments that all fit
])
def test_arrangement(plan, cells, streams, T, pv, levels, want):
    assert _run(plan, cells, streams, T, pv, *levels) == [want]


def test_the_comparison_tests_run_every_arrangement(plan):
    seen = set()
    for _, (L, H, T, G, W), codecs, keeps in compare.CASES:
        n = len(codecs) + (0 if (16, 0) in codecs else 1)
        for pv in ("default", "matrix", "fp32"):
            seen.add((pv, *_run(plan, L * H * -(-G * W // 128), n, T, pv, *keeps)))
    assert seen == {(pv, a) for pv in ("default", "matrix", "fp32") for a in ("grouped", "cell")} | {("matrix", "walk")}
