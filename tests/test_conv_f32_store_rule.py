"""The bound on the offsets of the tiled fp32 convolution's store (csrc/conv_f32_store.h), compiled for the host: where the rule takes a layer, every scalar offset --
of the rows that a block of 32 filters is rounded up to as well -- lies within the 2 GiB that the buffer spans, and so does every output of a tile's images."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_04728_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "conv_f32_store.h"
int main()
{
    int ctot, P, Q, residual;
    while (scanf("%d %d %d %d", &ctot, &P, &Q, &residual) == 4) printf("%d\n", dr::store_tile_fits(ctot, P, Q, residual));
}
"""

CASES = [
    # channels, P, Q, residual, taken
    (256, 55, 55, False, True),
    (8, 4608, 4608, True, False),            # 27 planes of 85 MB beside the 8 that exist: 2.29e9
    (8, 4400, 4400, True, True),             # 2.09e9
    (8, 4608, 4608, False, True),            # no residual: 3 planes
    (1, 13400, 13400, False, False),         # 3 planes of 718 MB
    (1, 13300, 13300, False, True),
    (1, 4460, 4460, True, False),
    (1, 4459, 4459, True, True),             # 27 planes: 500 KB below 2 GiB
    (544, 1024, 1024, False, False),         # 2.3 GB of channels
    (4480, 1000, 60, False, False),          # 2.15 GB in two images
    (13, 4459, 4459, True, True),
    (14, 4459, 4459, True, False),           # two images of 14
    (4096, 1, 1, True, True),
]


@pytest.fixture(scope="module")
def fits(tmp_path_factory):
    d = tmp_path_factory.mktemp("store")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(d / "rule.cpp"), "-o", str(d / "rule")])

    def ask(cases):
        out = subprocess.run([str(d / "rule")], input="\n".join("%d %d %d %d" % c for c in cases), capture_output=True, text=True, check=True).stdout
        return [line == "1" for line in out.split()]
    return ask


def test_at_the_line(fits):
    assert fits([c[:4] for c in CASES]) == [c[4] for c in CASES]


def test_offsets_of_the_layers_it_takes(fits):
    sides = [1, 3, 11, 55, 400, 1000, 2000, 2900, 3300, 4459, 4460, 5000, 9000, 13300, 13400, 16000]
    cases = [(ctot, side, max(1, side - 1), res) for ctot in (1, 3, 8, 13, 32, 33, 200, 544, 4096) for side in sides for res in (False, True)]
    taken = 0
    for (ctot, P, Q, res), ok in zip(cases, fits(cases)):
        if ok:
            taken += 1
            assert (27 if res else 3) * P * Q * 4 < 2 ** 31 - 1       # the scalar part: row 24 + 3 of a block of 32; row 3 of an eight
            images = -(-(128 + P * Q - 1) // (P * Q))                 # that a tile of 128 pixels reaches into
            assert images * ctot * P * Q * 4 <= 2 ** 31
    assert taken > 60
