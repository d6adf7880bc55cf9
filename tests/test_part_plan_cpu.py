"""The plan of block inference (part_plan.h) run on the CPU under address and
undefined-behaviour sanitizers: every slot written once and before it is read, and every
score equal to the definition's, for powers of two, highly composite and prime sizes, sizes
with a large prime factor (sub-sums), and several tensors in one plan."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("part") / "part_plan_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2606_13894_amd", "csrc"),
                    os.path.join(ROOT, "tests", "part_plan_check.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("sizes", [
    [1], [2], [3], [4], [840], [840 * 7], [97], [2047], [2048], [2049], [4096], [7919], [2 * 7919], [2 * 40009],
    [49155], [1 << 16], [3 << 15], [768 * 64], [999 * 50], [720720 // 4], [1092 * 99], [29 * 1733],
    [1733 * 96], [37 * 41 * 43], [6 * 16411], [11 * 13 * 17 * 19],
    [768, 3072, 1, 768 * 65, 4096, 97, 3 * 5 * 7 * 11 * 13],
], ids=lambda s: "+".join(map(str, s)))
@pytest.mark.parametrize("scale", [1, 10 ** 4])   # runs of one chunk, and of several
def test_plan_gives_the_scores(check, sizes, scale):
    r = subprocess.run([check] + [str(s) for s in sizes], capture_output=True, text=True,
                       env=dict(os.environ, PART_SCALE=str(scale)))
    assert r.returncode == 0, r.stdout + r.stderr
