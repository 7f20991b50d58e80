"""The rule that sends transposing conversions to tiles of 128 x 128: what it sends can be launched, and the tests' statement of it, and
of the rule for the FP8 columns that it leaves, is the library's.  Host code, compiled here."""
import itertools
import os
import random
import shutil
import subprocess

import pytest

from paper_2603_02731_amd import build
from tests.rules import KINDS, own_rows, small_tiles

PROGRAM = r"""
#include <cstdio>
#include "col_small_rule.hpp"
#include "row_to_fp8_col_rule.hpp"
int main()
{
    long long M, K, E, kind, units;
    while (scanf("%lld %lld %lld %lld %lld", &M, &K, &E, &kind, &units) == 5)
        printf("%d %lld %d\n", (int)mxfp4::col_in_small_tiles(M, K, (int)E, (mxfp4::ColKind)kind, units),
               (long long)mxfp4::col_small_workgroups(M, K, (int)E),
               (int)mxfp4::fp8_col_in_segments(M, K, (int)E, kind == mxfp4::COL_REQUANT, units));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """[(kind, M, K, E, units)] -> [(small tiles, workgroups, FP8 in segments)]."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    folder = tmp_path_factory.mktemp("rule")
    (folder / "rule.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", build.CSRC, str(folder / "rule.cpp"), "-o", str(folder / "rule")],
                   check=True)

    def ask(cases):
        text = "".join(f"{M} {K} {E} {KINDS.index(kind)} {units}\n" for kind, M, K, E, units in cases)
        out = subprocess.run([str(folder / "rule")], input=text, check=True, capture_output=True, text=True).stdout.split()
        return [(bool(int(a)), int(b), bool(int(c))) for a, b, c in zip(out[0::3], out[1::3], out[2::3])]

    return ask


SIZES = [(M, 128 * w, E) for M, w, E in itertools.product((1, 32, 127, 128, 4096, 8192, 8193, 65535, 1 << 24), (1, 3, 56, 8192, 65535, 65536, 131072),
                                                          (0, 1, 64, 128, 255, 256, 257, 1024)) if E or M % 32 == 0]


@pytest.mark.parametrize("units", [32, 256, 304])
def test_every_launch_fits(rule, units):
    """A launch has less than 2^32 work items.  Rows and widths up to the 2^24 that the entry points take."""
    cases = [(kind, *size, units) for kind in KINDS for size in SIZES]
    for case, (small, workgroups, _) in zip(cases, rule(cases)):
        assert not small or (workgroups + 7) // 8 * 8 * 256 < 1 << 32, case
    # few rows of very many columns: in the larger tiles' reach
    wide = [(kind, M, K, E, units) for kind in KINDS for M, K, E in ((128, 1 << 24, 128), (256, 1 << 23, 256), (1, 1 << 24, 256))]
    assert not any(small for small, _, _ in rule(wide))


def test_the_tests_state_the_same_rule(rule):
    rng = random.Random(4)
    cases = [(kind, *size, 256) for kind in KINDS for size in SIZES]
    for _ in range(4000):
        E = rng.choice((0, 1, 2, 8, 32, 64, 100, 128, 200, 256, 257))
        M = rng.choice((rng.randint(1, 40000), 128 * rng.randint(1, 300), max(E, 1) * rng.choice((24, 32, 64, 256)) + rng.randint(-1, 1)))
        cases.append((rng.choice(KINDS), 32 * -(-M // 32) if E == 0 else max(M, 1), 128 * rng.randint(1, 130), E, rng.choice((64, 256))))
    own = 0
    for case, (small, _, segments) in zip(cases, rule(cases)):
        assert small == small_tiles(*case), case
        if case[0] != "mxfp4" and case[3] > 0:
            assert (not small and not segments) == own_rows(*case), case
            own += not small and not segments
    assert own > 10
