"""The bound on the offsets of the fp32 first-layer kernel's stores (csrc/conv_f32_taps.h), compiled for the host: where the rule takes a layer, every
scalar offset that a store may have -- of the filters that a block is rounded up to as well -- lies within 2 GiB, and so does every output."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_04728_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "conv_f32_taps.h"
int main()
{
    int K, y_ctot, P, Q;
    while (scanf("%d %d %d %d", &K, &y_ctot, &P, &Q) == 4) printf("%d %d\n", dr::taps_tm(K), dr::taps_store_fits(K, y_ctot, P, Q));
}
"""

CASES = [
    # K, channels of the output tensor, P, Q, taken
    (96, 96, 55, 55, True),
    (1, 1, 4200, 4200, False),                # 31 planes of 70.6 MB beside the one that exists: 2.19e9
    (8, 8, 4200, 4200, False),
    (1, 1, 4096, 4096, False),                # 32 planes: 2 GiB
    (1, 1, 4096, 4095, True),
    (40, 64, 2048, 2048, False),              # two images of 64 channels
    (33, 33, 2900, 2900, False),              # blocks of 64 filters: 2 x 33 planes in two images
    (33, 33, 2800, 2800, True),
    (33, 300, 900, 900, True),                # the output tensor's channels decide
    (33, 400, 900, 900, False),
    (3, 3, 1, 1, True),
]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("taps")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(d / "rule.cpp"), "-o", str(d / "rule")])

    def ask(cases):
        out = subprocess.run([str(d / "rule")], input="\n".join("%d %d %d %d" % c for c in cases), capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


def test_at_the_line(rule):
    assert [bool(fits) for _, fits in rule([c[:4] for c in CASES])] == [c[4] for c in CASES]


def test_offsets_of_the_layers_it_takes(rule):
    sides = [1, 3, 11, 55, 400, 1000, 2000, 2040, 2890, 3000, 4200, 8000]
    cases = [(K, K + more, side, max(1, side - 1)) for K in (1, 5, 15, 16, 31, 32, 33, 64, 65, 96, 97, 200) for more in (0, 7, 500) for side in sides]
    for (K, y_ctot, P, Q), (tm, fits) in zip(cases, rule(cases)):
        if fits:
            assert (32 * tm - 1) * P * Q * 4 < 2 ** 31 - 1           # the scalar part: filter 31 or 63 or 95 of a block
            images = -(-(128 + P * Q - 1) // (P * Q))                # that a tile of 128 pixels reaches into
            assert images * y_ctot * P * Q * 4 <= 2 ** 31
