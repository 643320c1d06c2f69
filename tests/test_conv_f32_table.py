"""The one-word entries of the fp32 convolution's gather table (csrc/conv_f32_table.h), compiled for the host: wherever the predicate says
that a layer's offsets fit, every entry comes back whole -- also for filters taller than the map, whose last rows start
behind the last plane."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_04728_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "conv_f32_table.h"
int main()
{
    int C, H, W, R, S;
    while (scanf("%d %d %d %d %d", &C, &H, &W, &R, &S) == 5) {
        const bool fits = dr::tab1_fits(C, H, W, R, S);
        bool whole = true;
        // the entries of the first and the last plane (those between lie between)
        for (int c = 0; fits && c < C; c += C > 1 ? C - 1 : 1)
            for (int r = 0; r < R; ++r)
                for (int s = 0; s < S; ++s) {
                    const long off = (long)c * H * W + (long)r * W + s;
                    const int e = dr::tab1_entry((int)off, r * S + s);
                    whole = whole && e >= 0 && dr::tab1_offset(e) == off && dr::tab1_tap(e) == r * S + s;
                }
        printf("%d %d\n", fits, whole);
    }
}
"""

CASES = [
    # C, H, W, R, S, fits
    (64, 56, 56, 3, 3, True),
    (3, 224, 224, 5, 5, True),
    (1, 1, 45000000, 7, 1, False),            # a map of one row: the tensor has fewer than 2^26 elements, the filter's last row starts at 2.7e8
    (1, 1, 9000000, 31, 1, False),            # row 15 beyond 2^27
    (1, 1, (1 << 25) - 1, 3, 1, True),        # the largest offset is 2^26 - 2
    (1, 1, (1 << 25) - 1, 3, 2, True),        # 2^26 - 1
    (1, 1, (1 << 25) - 1, 3, 3, False),       # 2^26
    (2, 1, 1 << 24, 4, 1, False),             # 2^26, through the second plane
    (2, 1, (1 << 24) - 1, 4, 1, True),
    (1 << 20, 8, 8, 1, 1, True),              # 2^26 elements, the last plane at 2^26 - 64
    (46340, 46340, 2, 1, 1, False),           # a plane count whose product with the plane overflows 32 bits
    (2, 2, 2, 8, 4, False),                   # 32 taps
]


def test_entries_that_fit_come_back_whole(tmp_path):
    src, exe = tmp_path / "table.cpp", tmp_path / "table"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c[:5])) for c in CASES), capture_output=True, text=True, check=True).stdout
    got = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert len(got) == len(CASES)
    for case, (fits, whole) in zip(CASES, got):
        assert bool(fits) == case[5], case
        assert whole, case
