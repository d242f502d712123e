"""The sharing-out of kvp_score_tokens (csrc/score_plan.h, host arithmetic): a C++ program walks it over its range.  What a
plan writes has to fit the workspace size that callers are told, for every shape."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_plan_fits_the_workspace_and_covers_every_key_once():
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "score_plan")
        subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_14946_amd", "csrc"), "-o", exe,
                        os.path.join(ROOT, "tests", "score_plan.cpp")], check=True)
        out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    walks, sizes = map(int, out.stdout.split())
    assert walks > 2000 and sizes > 400_000
