"""Which modules run level by level (csrc/inception_levels.h), compiled for the host: with the branches on streams a bf16 module whose layers share launches does,
unless two branches have layers that share nothing and of which neither is short beside the other."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_04728_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "inception_levels.h"
int main()
{
    int all, small, big, bf16, streams;
    long longest, second;
    while (scanf("%d %d %d %ld %ld %d %d", &all, &small, &big, &longest, &second, &bf16, &streams) == 7)
        printf("%d\n", dr::module_by_levels(dr::ModuleLayers{all, small, big, longest, second}, bf16, streams));
}
"""


@pytest.fixture(scope="module")
def by_levels(tmp_path_factory):
    d = tmp_path_factory.mktemp("levels")
    (d / "levels.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(d / "levels.cpp"), "-o", str(d / "levels")])
    return lambda *v: subprocess.run([str(d / "levels")], input="%d %d %d %d %d %d %d" % v, capture_output=True, text=True, check=True).stdout.strip() == "1"


@pytest.mark.parametrize("all_,small,big,longest,second,streams,expected", [
    (6, 0, 6, 0, 0, True, True),
    (6, 6, 0, 0, 0, True, True),
    (6, 3, 2, 0, 0, True, True),             # one that shares nothing but has a kernel of its own beside the others
    (6, 4, 1, 300, 0, True, True),           # a 5x5 on 12 channels
    (6, 2, 2, 828, 300, True, True),         # 3x3 on 92 and 5x5 on 12
    (6, 2, 2, 1000, 399, True, True),
    (6, 2, 2, 1000, 400, True, False),
    (6, 2, 2, 1692, 1100, True, False),      # 3x3 on 188 and 5x5 on 44
    (6, 2, 0, 484, 484, True, False),
    (6, 2, 2, 1692, 1100, False, True),      # branches in turn
    (6, 1, 1, 0, 0, True, True),
    (6, 1, 0, 0, 0, True, False),
    (6, 0, 1, 0, 0, False, False),
])
def test_bf16(by_levels, all_, small, big, longest, second, streams, expected):
    assert by_levels(all_, small, big, longest, second, True, streams) == expected


@pytest.mark.parametrize("all_,small,big,streams,expected", [
    (6, 4, 2, True, True),
    (6, 3, 3, True, False),
    (6, 4, 1, True, False),
    (6, 1, 1, False, True),
    (6, 1, 0, False, False),
])
def test_fp32(by_levels, all_, small, big, streams, expected):
    assert by_levels(all_, small, big, 0, 0, False, streams) == expected
