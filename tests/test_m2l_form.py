"""The rule between the plain and the reflection-reduced FP64 / FP32 M2L
(csrc/m2l_form.h), compiled for the host and compared with what was measured:
for each tree the form whose M2L took less time, at least 3 % apart."""
import os
import subprocess

import pytest

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2209_13121_amd", "csrc")
MAIN = """
#include <cstdio>
#include "m2l_form.h"
int main() {
  int p, fp64, ad;
  long long g16, g128;
  while (scanf("%d %d %d %lld %lld", &p, &fp64, &ad, &g16, &g128) == 5)
    printf("%d\\n", (int)fmm::sym::serves(p, fp64 != 0, ad != 0, g16, g128));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("m2l_form")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "main")
    subprocess.run(["g++", "-std=c++17", "-I", SRC, str(d / "main.cpp"), "-o", exe], check=True)

    def ask(rows):
        text = "".join(" ".join(str(int(v)) for v in r) + "\n" for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [v == "1" for v in out.split()]

    return ask


def groups(parents):
    """(16-parent, 128-parent) work-groups of that many divided parents on one level."""
    return 8 * ((parents + 15) // 16), 8 * ((parents + 127) // 128)


# order, FP64, divided parents, M2L us of the plain and of the reflection form
ADAPTIVE = [
    (4, 1, 585, 212, 136), (4, 1, 997, 208, 148), (4, 1, 2852, 215, 416), (4, 1, 3908, 221, 486), (4, 1, 4110, 379, 943),
    (4, 1, 19048, 936, 2540), (4, 0, 997, 142, 98), (4, 0, 2852, 147, 271), (4, 0, 4110, 267, 555), (4, 0, 19048, 677, 1535),
    (5, 1, 1145, 411, 253), (5, 1, 2852, 426, 504), (5, 1, 4110, 830, 1153), (5, 1, 15437, 1678, 2438),
    (5, 0, 1145, 271, 178), (5, 0, 2852, 282, 350), (5, 0, 4110, 518, 753), (5, 0, 15437, 1031, 1641),
    (6, 1, 1145, 586, 346), (6, 1, 2852, 608, 684), (6, 1, 4110, 1196, 1572), (6, 1, 15437, 2407, 3276),
    (6, 0, 1145, 322, 220), (6, 0, 2852, 334, 436), (6, 0, 4110, 653, 961), (6, 0, 15437, 1306, 2064),
    (7, 1, 2852, 826, 644), (7, 1, 4110, 1657, 1522), (7, 1, 15437, 3364, 3126), (7, 0, 2852, 454, 408),
    (7, 0, 4650, 851, 919), (7, 0, 12440, 1619, 1824), (7, 0, 19048, 2279, 2353), (8, 0, 9246, 2353, 2159), (9, 1, 9246, 6966, 4479),
    (12, 1, 585, 7792, 1138),
]
# order, FP64, depth, the same
UNIFORM = [(4, 1, 3, 152, 49), (4, 1, 4, 223, 129), (4, 1, 5, 406, 430), (4, 1, 6, 1963, 2129), (4, 1, 7, 14427, 15858),
           (5, 1, 5, 864, 543), (5, 0, 6, 2568, 1855), (6, 1, 6, 6128, 3782), (8, 1, 6, 13277, 6002)]


def test_adaptive_trees_take_the_form_that_was_faster(rule):
    got = rule([(p, fp64, 1, *groups(n)) for p, fp64, n, _, _ in ADAPTIVE])
    assert [(r[:3], r[4] < r[3]) for r in ADAPTIVE] == [(r[:3], g) for r, g in zip(ADAPTIVE, got)]


def test_uniform_trees_take_the_form_that_was_faster(rule):
    levels = [[groups(8 ** (m - 1)) for m in range(2, depth + 1)] for _, _, depth, _, _ in UNIFORM]
    got = rule([(p, fp64, 0, sum(a for a, _ in g), sum(b for _, b in g))
                for (p, fp64, *_), g in zip(UNIFORM, levels)])
    assert [(r[:3], r[4] < r[3]) for r in UNIFORM] == [(r[:3], g) for r, g in zip(UNIFORM, got)]


def test_low_orders_are_plain_and_high_orders_are_not(rule):
    g = [(16, 8), (1000, 128), (100000, 12500)]
    assert not any(rule([(p, f, a, *n) for p in range(4) for f in (0, 1) for a in (0, 1) for n in g]))
    assert all(rule([(p, f, a, *n) for p in range(8, 13) for f in (0, 1) for a in (0, 1) for n in g]))
