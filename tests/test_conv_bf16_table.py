"""Where the bf16 kernels' tables place the chunks of a contraction (csrc/conv_bf16_table.h), compiled for the host: for every output that is
asked for, the chunks read are exactly those inside the image and inside the contraction, at their true byte -- also where a filter row lies
2 GiB or more behind the first pixel of a window that begins before the tensor."""
import os
import random
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_04728_amd", "csrc")

# (the entries are numbered as in the kernels: 8 per slice, row_chunks of them from filter row to filter row)
PROGRAM = r"""
#include <cstdio>
#include "conv_bf16_table.h"
int main()
{
    int N, C, H, W, R, S, sh, sw, ph, pw, img, p, q;
    while (scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d", &N, &C, &H, &W, &R, &S, &sh, &sw, &ph, &pw, &img, &p, &q) == 13) {
        int row_chunks, read = 0, wrong = 0;
        const int slices = dr::chunk_slices(R, S, C, &row_chunks), c8 = C / 8, ih0 = p * sh - ph, iw0 = q * sw - pw;
        const unsigned base = dr::window_offset(img, ih0, iw0, H, W, C), outside = dr::window_mask(true, ih0, iw0, R, S, H, W);
        int filters = 0;
        for (int e = 0; e < slices * 8; ++e) {
            const int r = e / row_chunks, jl = e % row_chunks, s = jl / c8, c = jl % c8;
            const bool exists = r < R && s < S, inside = exists && ih0 + r >= 0 && ih0 + r < H && iw0 + s >= 0 && iw0 + s < W;
            const unsigned mask = dr::chunk_mask(exists, r, s), at = base + dr::chunk_offset(r, jl, W, C);
            const long long true_at = ((((long long)img * H + ih0 + r) * W + iw0 + s) * C + c * 8) * 2;
            filters += dr::chunk_exists(mask);
            read += (mask & outside) == 0;
            wrong += ((mask & outside) == 0) != inside || (inside && at != true_at) || !(mask & dr::WINDOW_NONE) || exists != dr::chunk_exists(mask);
        }
        printf("%d %d %d\n", wrong, read, filters == R * S * c8);
    }
}
"""


def run(tmp_path, lines):
    src, exe = tmp_path / "table.cpp", tmp_path / "table"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in lines), capture_output=True, text=True, check=True).stdout
    got = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert len(got) == len(lines)
    for line, (wrong, _, whole) in zip(lines, got):
        assert not wrong and whole, line
    return [read for _, read, _ in got]


# N, C, H, W, R, S, stride, padding, image, p, q of inputs below 2 GiB, and the chunks inside the image
FAR = [
    ((1, 512, 1, 139811, 16, 1, 16, 3, 15, 0, 0, 0, 46603), 64),             # a 143 MB row; the tap inside the map is 15 rows, 2^31 bytes, behind the window
    ((1, 512, 1, 139811, 16, 1, 16, 3, 15, 0, 0, 0, 0), 64),
    ((1, 8, 1, 9000000, 16, 1, 16, 1000, 15, 0, 0, 0, 8999), 1),
    ((1, 64, 3, 1200000, 16, 1, 4, 200, 13, 0, 0, 0, 5999), 24),             # rows 13, 14 and 15
    ((1, 64, 3, 1200000, 16, 1, 4, 200, 13, 0, 0, 3, 77), 24),               # rows 1, 2 and 3 of a window that begins one row before
    ((1, 8, 1, 130000000, 16, 9, 1, 100, 15, 4, 0, 15, 0), 5),               # 2.08 GB: rows that pass 2^32 several times
    ((1, 8, 1, 130000000, 16, 9, 1, 100, 15, 4, 0, 0, 1299999), 9),
    ((1, 8, 16, 8000000, 16, 3, 1, 100, 0, 1, 0, 0, 79999), 48),             # no padding above: offsets up to 2^31 all in range
    ((2, 16, 5, 11, 3, 3, 1, 1, 40, 40, 1, 20, 20), 0),                      # a window wholly in the padding
]


def test_rows_far_behind_the_window(tmp_path):
    assert run(tmp_path, [c for c, _ in FAR]) == [n for _, n in FAR]


def test_ordinary_layers(tmp_path):
    rng, lines = random.Random(6), []
    while len(lines) < 400:
        C, H, W, R, S = 8 * rng.randint(1, 40), rng.randint(1, 20), rng.randint(1, 20), rng.randint(1, 16), rng.randint(1, 9)
        sh, sw, ph, pw = rng.randint(1, 3), rng.randint(1, 3), rng.randint(0, R + 1), rng.randint(0, S + 1)
        P, Q = (H + 2 * ph - R) // sh + 1, (W + 2 * pw - S) // sw + 1
        if H + 2 * ph >= R and W + 2 * pw >= S:
            lines.append((4, C, H, W, R, S, sh, sw, ph, pw, rng.randint(0, 3), rng.randrange(P), rng.randrange(Q)))
    run(tmp_path, lines)
