"""The dispatch rules of lsgd_rules.hpp (host C++, no GPU) at calls measured on
both sides of their lines: each row names a call and which kernel was the
faster one there."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1906_05936_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <string>
#include <iostream>
#include "lsgd_rules.hpp"
using namespace lsgd;
int main() {
    std::string rule;
    long long v[10];
    while (std::cin >> rule) {
        int k = 0;
        std::cin >> k;
        for (int i = 0; i < k; ++i) std::cin >> v[i];
        bool r = false;
        if (rule == "split") r = split_serves(v[0], (int)v[1], v[2], v[3], v[4]);
        else if (rule == "apart") r = copies_apart((int)v[0], (int)v[1], (int)v[2], v[3], v[4], v[5], v[6], v[7]);
        else if (rule == "two") r = stream_two_units(v[0], (int)v[1], (int)v[2], v[3], (int)v[4]);
        else if (rule == "plan") {
            r = split_serves_plan(PlanShape{v[0], v[1], v[2], v[3], (int)v[4], v[5] != 0, v[6] != 0, v[7] != 0, v[8]});
        } else if (rule == "lars") {
            r = split_serves_lars(PlanShape{v[0], v[1], v[2], v[3], (int)v[4], v[5] != 0, v[6] != 0, v[7] != 0, v[8]}, v[9]);
        } else if (rule == "copies") r = copy_replicas_per_group(v[0], v[1]) == (int)v[2];
        else if (rule == "plantwo") r = plan_two_units(PlanShape{v[0], v[1], v[2], v[3], (int)v[4], v[5] != 0, v[6] != 0, v[7] != 0, v[8]}, v[9], 256);
        else if (rule == "mean") r = mean_stream_form((int)v[0], v[1]) == (MeanForm)v[2];
        else return 1;
        std::printf("%d\n", (int)r);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "main")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + CSRC, str(d / "main.cpp"), "-o", exe], check=True)

    def run(rule, rows):
        text = "".join("%s %d %s\n" % (rule, len(r), " ".join(str(int(x)) for x in r)) for r in rows)
        return [x == "1" for x in subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()]

    return run


F32, BF16 = False, True

# (n, workers, bfloat16, compile-time kernel, copy bytes), split kernel faster?
SPLIT = [
    ((65_536, 4, F32, True, 0), False), ((131_072, 4, F32, True, 0), False), ((10_007, 4, F32, True, 0), True),
    ((1_000, 16, F32, True, 0), False), ((2_003, 16, F32, True, 0), True), ((65_536, 16, F32, True, 0), True),
    ((262_144, 16, F32, True, 0), True), ((262_145, 16, F32, True, 0), False), ((40_000, 8, F32, True, 0), True),
    ((11, 8, F32, True, 0), True), ((205, 12, F32, True, 16), True), ((100_003, 1, F32, True, 0), False), ((10_007, 2, F32, True, 0), True), ((165_830, 2, F32, True, 8), False),
    ((3_825, 8, F32, True, 92), True), ((1_671, 8, F32, True, 72), True), ((30_000, 5, F32, True, 4), True),
    ((30_000, 5, F32, True, 0), False), ((65_536, 4, F32, True, 16), False), ((20_001, 4, F32, True, 16), True),
    ((65_536, 4, BF16, True, 0), False), ((131_072, 16, BF16, True, 0), False), ((131_069, 16, BF16, True, 0), True),
    ((100_000, 10, BF16, True, 0), False), ((1_003, 4, BF16, True, 0), True), ((262_144, 128, BF16, True, 0), False),
    ((30_000, 8, BF16, True, 48), True), ((30_000, 8, BF16, True, 16), False), ((30_000, 4, BF16, True, 48), False),
    ((185_360, 128, BF16, True, 0), True), ((262_141, 128, BF16, True, 0), True), ((262_144, 64, BF16, True, 0), True),
    ((262_144, 40, BF16, False, 0), True), ((300_000, 40, BF16, False, 0), False),
    ((370_727, 64, F32, False, 0), True), ((524_288, 64, F32, False, 0), False), ((1_000_000, 30, F32, False, 0), False),
    ((1_000_000, 80, F32, False, 0), False), ((200_000, 9, F32, False, 0), True), ((300_000, 9, F32, False, 0), False),
    ((541_674, 20, F32, False, 20), True), ((446_528, 20, F32, False, 52), True), ((577_000, 30, F32, False, 0), False),
    ((381_120, 80, F32, False, 40), False),
]


def test_split_kernels(ask):
    got = ask("split", [r for r, _ in SPLIT])
    assert got == [want for _, want in SPLIT], [r for (r, w), g in zip(SPLIT, got) if w != g]


# (workers, gradient bytes, replica bytes, copy bytes, broadcast, n, stream, cached), copies in their own pass faster?
APART = [
    ((4, 4, 4, 40, False, 300_000, False, True), False), ((16, 4, 4, 40, False, 300_000, False, True), False),
    ((16, 4, 4, 56, False, 1_000_000, False, True), False), ((4, 4, 4, 40, False, 12_000_000, False, True), False),
    ((16, 4, 4, 48, False, 3_000_000, False, True), True), ((4, 4, 4, 56, False, 5_000_000, False, True), True),
    ((16, 4, 4, 56, False, 12_000_000, False, True), True), ((9, 4, 4, 56, False, 12_000_000, True, True), False),
    ((4, 2, 2, 48, False, 1_000_000, False, True), False), ((8, 2, 2, 48, False, 5_000_000, False, True), True),
    ((4, 2, 4, 32, False, 600_000, False, True), False), ((16, 2, 4, 32, False, 1_000_000, False, True), True),
    ((16, 2, 4, 40, False, 1_000_000, False, True), True), ((10, 2, 4, 32, False, 1_000_000, False, True), True),
    ((10, 2, 4, 24, False, 1_000_000, False, True), False), ((10, 2, 4, 24, False, 3_000_000, False, True), True),
    ((10, 2, 4, 16, False, 3_000_000, False, True), False), ((10, 2, 4, 16, False, 25_000_000, False, True), True),
    ((16, 4, 4, 32, False, 25_000_000, False, True), True), ((32, 4, 4, 32, False, 1_000_000, True, False), True),
    ((64, 4, 4, 4, False, 1_000_000, True, False), True),
    ((8, 4, 4, 60, True, 300_000, False, True), False), ((8, 4, 4, 60, True, 12_000_000, False, True), False),
    ((9, 4, 4, 40, True, 1_000_000, False, True), False), ((4, 4, 4, 44, True, 12_000_000, False, True), False),
    ((16, 4, 4, 60, True, 3_000_000, False, True), True), ((16, 4, 4, 60, True, 1_000_000, False, True), False),
    ((16, 4, 4, 0, False, 25_000_000, False, True), False),
]


def test_copies_apart(ask):
    got = ask("apart", [r for r, _ in APART])
    assert got == [want for _, want in APART], [r for (r, w), g in zip(APART, got) if w != g]


# (elements, workers), two-unit tiles faster? (flat, 256 compute units)
TWO_UNITS = [((25_557_032, 9), True), ((1_000_000, 9), False), ((500_000, 9), True), ((1_100_000, 9), True), ((25_557_032, 14), False), ((10_000_000, 14), True), ((1 << 19, 64), True),
             ((600_000, 64), False), ((1 << 20, 64), False), (((1 << 20) + 1, 64), True), ((1_100_000, 128), True),
             ((1_600_000, 64), False), ((2_400_000, 64), False), ((25_557_032, 64), False)]


def test_two_unit_tiles(ask):
    got = ask("two", [(-(-n // 4096), 2, N, n, 256) for (n, N), _ in TWO_UNITS])
    assert got == [want for _, want in TWO_UNITS], [r for (r, w), g in zip(TWO_UNITS, got) if w != g]


def shape(sizes, workers, bf16, compile_time, pow2_groups=True, copy_bytes=0):
    unit = 8 if bf16 else 4
    return (sum(sizes), sum(s > 0 for s in sizes), sum(-(-s // 2048) for s in sizes), sum(s % unit > 0 for s in sizes), workers,
            bf16, compile_time, pow2_groups, copy_bytes)


GROWING = [30_000 * k // 20 + 7 for k in range(1, 31)]   # 30 tensors of 7e5 elements in all
# plan and its step, split kernel faster?
PLAN_SPLIT = [
    (shape([200] * 20_000, 40, F32, False), True), (shape([700] * 3_000, 64, F32, False), True),
    (shape([900] * 2_000, 64, F32, False), False), (shape([1_500] * 1_000, 64, F32, False), False),
    (shape([200] * 20_000, 4, F32, True), True), (shape([1_000] * 5_000, 4, F32, True), True),
    (shape([200] * 20_000, 16, F32, True), False), (shape([200] * 20_000, 16, BF16, True), True),
    (shape([900] * 2_000, 64, BF16, True), True), (shape([2_048] * 2_000, 64, BF16, True), False),
    (shape(GROWING, 16, F32, True), True), (shape(GROWING, 16, BF16, True), True),
    (shape([333_333] * 3, 16, F32, True), False), (shape([333_333] * 3, 64, F32, False), False),
    (shape([333_333] * 3, 16, BF16, True), True), (shape([16_667] * 60, 16, F32, True), True),
    (shape([175_000] * 3, 4, F32, True), False), (shape([170_001] * 3, 4, F32, True), True), (shape([170_000] * 3, 4, F32, True), True),
    (shape([524_288], 16, F32, True), True), (shape([65_536], 4, F32, True), True), (shape([65_536], 16, F32, True), True),
    (shape([262_144], 16, BF16, True), False), (shape([131_069], 16, BF16, True), True),
    (shape([100_001, 100_001], 4, F32, True), True), (shape([100_000, 100_000], 4, F32, True), True), (shape([519_001, 5_000], 16, BF16, True), True),
    (shape([17_472] * 60, 4, F32, True), True), (shape([6_400] * 160, 2, F32, True), True), (shape([52_480] * 10, 2, F32, True), False),
    (shape([8_704] * 60, 4, BF16, True), False), (shape([8_703] * 60, 4, BF16, True), True), (shape([13_120] * 10, 64, BF16, True), True),
    (shape([524_288, 0], 16, F32, True), True), (shape([524_288], 9, BF16, False), True),
    (shape([272_215], 36, BF16, True, False), True), (shape([232_256] * 2, 20, BF16, True, False, 40), True),
    (shape([57_384] * 8, 24, BF16, True, False, 10), True), (shape([32_000] * 8, 64, BF16, True), False),
    (shape([16_000] * 12, 32, BF16, True), True), (shape([75_008] * 4, 32, BF16, True, True, 64), True), (shape([75_008] * 4, 32, BF16, True), False),
    (shape([88] * 350, 12, BF16, True, False), True), (shape([88] * 350, 16, BF16, True), False), (shape([88] * 350, 16, BF16, True, True, 64), True),
    (shape([420] * 112, 2, F32, True), False), (shape([420] * 112, 2, F32, True, True, 48), True), (shape([64] * 64, 16, F32, True), False),
    (shape([1_280] * 64, 5, F32, True), True), (shape([128] * 64, 5, F32, True), False),
    (shape([360_567, 360_568], 20, F32, False), True), (shape([271_045, 271_045], 28, F32, False), True),
    (shape([23_676] * 39, 54, F32, False), False), (shape([17_880] * 49, 99, F32, False), False), (shape([14_461] * 60, 70, F32, False), False),
    (shape([18_816] * 34, 64, F32, True), True), (shape([24_740] * 24, 100, BF16, False), True), (shape([200_001] * 5, 30, F32, False), True),
]


def test_plan_split_kernels(ask):
    got = ask("plan", [r for r, _ in PLAN_SPLIT])
    assert got == [want for _, want in PLAN_SPLIT], [r for (r, w), g in zip(PLAN_SPLIT, got) if w != g]


def test_plan_two_unit_tiles(ask):
    rows = [([1_500] * 1_000, 64, True), ([5_000] * 1_000, 40, True), ([20_000] * 600, 64, False), ([700_000] * 3, 64, True),
            ([1_000_000] * 3, 64, False), ([400_000] * 30, 9, True), ([3_000] * 1_000, 64, False), ([3_001] * 1_000, 64, True),
            ([9_001] * 1_000, 64, True), ([9_000] * 1_000, 64, False)]
    got = ask("plantwo", [shape(s, n, F32, False) + (sum(-(-x // 4096) for x in s),) for s, n, _ in rows])
    assert got == [want for _, _, want in rows]


# plan, merged and its LARS step, split kernels faster?
LARS_SPLIT = [
    (shape([524_288], 4, F32, True), False, False), (shape([524_288], 64, F32, True), False, True),
    (shape([8_738] * 60, 4, F32, True), True, True), (shape([16_667] * 60, 4, F32, True), True, False),
    (shape([16_667] * 60, 64, F32, True), True, True), (shape([333_333] * 3, 64, F32, True), False, False),
    (shape([62_500] * 16, 64, F32, True), True, True), (shape([174_762] * 3, 4, BF16, True), False, False),
    (shape([174_762] * 3, 16, BF16, True), False, True), (shape([300_001] * 3, 64, BF16, True), False, True), (shape([300_000] * 3, 64, BF16, True), False, False),
    (shape([8_704] * 60, 16, BF16, True), True, True), (shape([16_704] * 60, 16, BF16, True), True, False),
    (shape([1_000_001], 9, BF16, False), False, False), (shape([500_001], 9, BF16, False), False, True),
    (shape([6_272] * 160, 4, F32, True), True, True), (shape([131_072], 16, BF16, True), False, False),
    (shape([5_824] * 120, 20, BF16, True, False), True, True), (shape([17_000] * 32, 30, BF16, True, False), True, True),
    (shape([20_000] * 32, 30, BF16, True, False), True, False), (shape([62_501] * 16, 80, F32, False), True, False),
    (shape([131_072], 4, F32, True), True, True), (shape([700] * 3_000, 64, BF16, True), True, False),
]


def test_lars_split_kernels(ask):
    got = ask("lars", [r + (merged,) for r, merged, _ in LARS_SPLIT])
    assert got == [want for _, _, want in LARS_SPLIT], [r for (r, _, w), g in zip(LARS_SPLIT, got) if w != g]


def test_copy_pass_of_small_pieces(ask):
    rows = [([700] * 3_000, 4), ([200] * 20_000, 4), ([2_500] * 300, 2), ([200_000] * 60, 1), ([2_048] * 8, 1)]
    assert all(ask("copies", [(sum(x), sum(-(-n // 2048) for n in x), rk) for x, rk in rows]))


def test_mean_forms(ask):
    one, ahead, four = 0, 1, 2
    rows = [(9, 100_000, one), (128, 300_000, one), (9, 1_000_000, ahead), (20, 25_000_000, ahead), (64, 1_000_000, four),
            (32, 3_000_000, four), (64, 25_000_000, ahead)]
    assert all(ask("mean", rows))
