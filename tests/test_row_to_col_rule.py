"""The rule that sends one large matrix to the row->col kernel with whole segments, against the offsets that kernel stores at:
they have 32 bits, and the entry point takes up to 2^31 rows.  Host code, compiled here."""
import os
import shutil
import subprocess

import pytest

from paper_2603_02731_amd import build
from tests.rules import aligned_pieces

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "row_to_col_rule.hpp"
using namespace mxfp4;
using namespace mxfp4::row_to_col_seg;
int main(int argc, char **argv)
{
    for (int i = 1; i + 1 < argc; i += 2) {
        const int64_t M = atoll(argv[i]), K = atoll(argv[i + 1]);
        // every piece of a wave, as the kernel counts (32 bits) and as it has to be
        int wraps = 0;
        for (uint32_t lane = 0; lane < 64; ++lane)
            for (int step = 0; step < CPP; ++step)
                for (uint32_t past = 0; past < SEG; past += 16) {
                    const uint32_t from = (lane & 7u) * 16u + SEG - past;
                    const uint32_t off = store_row<uint32_t>(lane, 0) * (uint32_t)(M / 2) + (uint32_t)step * (uint32_t)(M / 2) + from;
                    wraps += off != store_row<uint64_t>(lane, step) * (uint64_t)(M / 2) + from;
                }
        printf("%d %d\n", (int)row_to_col_in_segments(M, K), wraps);
    }
    long long M, K, E, units;
    while (argc == 1 && scanf("%lld %lld %lld %lld", &M, &K, &E, &units) == 4)
        printf("%d\n", (int)row_to_col_in_aligned_pieces(M, K, (int)E, units));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """[(M, K)] -> [(in segments, pieces whose 32-bit offset is wrong)]."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    folder = tmp_path_factory.mktemp("rule")
    (folder / "rule.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", build.CSRC, str(folder / "rule.cpp"), "-o",
                    str(folder / "rule")], check=True)

    def ask(cases=None, experts=None):
        if experts is not None:
            text = "".join(" ".join(map(str, c)) + "\n" for c in experts)
            out = subprocess.run([str(folder / "rule")], input=text, check=True, capture_output=True, text=True).stdout.split()
            return [bool(int(v)) for v in out]
        out = subprocess.run([str(folder / "rule")] + [str(v) for c in cases for v in c], check=True, capture_output=True,
                             text=True).stdout.split()
        return [(bool(int(a)), int(b)) for a, b in zip(out[0::2], out[1::2])]

    return ask


def test_no_offset_wraps_where_the_kernel_is_taken(rule):
    last = 145592096  # 59 k-rows of M / 2 bytes and 192 more are 2^32
    edge = [last + 32 * d for d in range(-4, 5)]
    far = [150000032, 2 ** 28 + 32, 2 ** 29 + 96, 2 ** 30 + 32, 2 ** 31 - 32]
    near = [1441824, 10000032, 2 ** 27 + 32]
    for (M, K), (taken, wraps) in zip([(m, 128) for m in near + edge + far], rule([(m, 128) for m in near + edge + far])):
        assert not (taken and wraps), f"{wraps} pieces of [{M}, {K}] are stored 2^32 bytes too low"
        assert taken == (M % 128 != 0 and M <= last), (M, K)
    assert [w > 0 for _, w in rule([(150000032, 128), (2 ** 31 - 32, 128)])] == [True, True]


def test_size_from_which_it_is_taken(rule):
    assert [t for t, _ in rule([(45088, 4096), (45024, 4096), (45056, 4096), (180320, 1024), (32, 128), (2 ** 24 - 32, 2 ** 24)])] == \
        [True, False, False, True, False, True]


def test_the_tests_state_the_same_rule_for_aligned_pieces(rule):
    cases = [(M, K, E, units) for M in (1, 255, 257, 16384, 32000) for K in (128, 256, 384, 4096)
             for E in (1, 2, 64, 256, 257, 320, 383, 384, 1024) for units in (64, 256, 304)]
    assert rule(experts=cases) == [aligned_pieces(*c) for c in cases]
    assert any(aligned_pieces(*c) for c in cases)
