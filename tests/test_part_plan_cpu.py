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


@pytest.mark.parametrize("budget", [0, 4000, 40000, 400000])
@pytest.mark.parametrize("sizes", [
    [840 * 7], [2 * 7919], [49155], [3 << 15], [720720 // 4], [29 * 1733], [11 * 13 * 17 * 19],
    [5 * 4097 * 3], [768, 3072, 1, 768 * 65, 4096, 97, 3 * 5 * 7 * 11 * 13, 768 * 65, 46189],
], ids=lambda s: "+".join(map(str, s)))
def test_plans_within_a_budget(check, sizes, budget):
    """Less room for stored sums: small divisors contrasted straight from the gradient, and
    several plans; the same scores."""
    r = subprocess.run([check] + [str(s) for s in sizes], capture_output=True, text=True,
                       env=dict(os.environ, PART_BUDGET=str(budget)))
    assert r.returncode == 0, r.stdout + r.stderr


# Parameter lists: elements of each tensor (GPT-2 small, 124M; Llama-3 1.5B, embeddings of
# 128256 x 2048; one tensor of many divisors; one whose factors beside 2 are large).
GPT2 = [50257 * 768, 1024 * 768] + 12 * [768, 768, 2304 * 768, 2304, 768 * 768, 768, 768, 768,
                                         3072 * 768, 3072, 3072 * 768, 768] + [768, 768]
LLAMA = [128256 * 2048] + 16 * [2048 * 2048, 512 * 2048, 512 * 2048, 2048 * 2048, 8192 * 2048,
                                8192 * 2048, 2048 * 8192, 2048, 2048] + [2048, 128256 * 2048]


@pytest.mark.parametrize("sizes", [GPT2, LLAMA, [128256 * 2048], [1081080], [9699690], [73513440],
                                   [151936 * 4096], [65537 * 4096], [32000 * 4096]],
                         ids=lambda s: f"{len(s)}x{s[0]}")
def test_stored_bytes(tmp_path, sizes):
    """What a call keeps on the device at a time: within the budget (half a byte an element and
    64 MiB), and the contrasts within another half. All sums of all tensors at once took 1.9
    bytes an element for the Llama-3 shapes and 20 for 73513440 elements."""
    src = tmp_path / "stored.cpp"
    src.write_text("""#include <cstdio>
#include <cstdlib>
#include "part_plan.h"
using namespace gefen;
int main(int argc, char** argv)
{
    std::vector<PartInput> in;
    int64_t total = 0, sums = 0, parts = 0;
    for (int a = 1; a < argc; ++a) in.push_back(PartInput{nullptr, std::atoll(argv[a]), 0}), total += in.back().n;
    for (const PartPlan& p : part_plans(in, part_budget(total)))
        sums = std::max(sums, p.sums), parts = std::max(parts, p.parts);
    std::printf("%lld %lld %lld\\n", (long long)total, 8 * (long long)sums, 8 * (long long)parts);
}
""")
    exe = str(tmp_path / "stored")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I",
                    os.path.join(ROOT, "paper_2606_13894_amd", "csrc"), str(src), "-o", exe],
                   check=True)
    total, sums, parts = map(int, subprocess.run([exe] + [str(s) for s in sizes], check=True,
                                                 capture_output=True, text=True).stdout.split())
    assert sums <= (64 << 20) + total // 2, (sums, total)
    assert parts <= (1 << 20) + total // 2, (parts, total)
