"""Which layers the fp32 kernels on bf16 pieces take and how their workgroups share the tiles (csrc/conv_f32_pieces_plan.h, conv_f32_direct_plan.h), compiled for the host: where a tile fits,
no run of its outputs lies over more input pixels than LDS has places for; a plan gives every tile of every layer to exactly one workgroup."""
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_04728_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "conv_f32_direct_plan.h"
int main(int argc, char** argv)
{
    if (argc > 1 && !strcmp(argv[1], "plan")) {
        int n, cus;
        while (scanf("%d %d", &n, &cus) == 2) {
            long tiles[dr::PIECES_LAYERS];
            double cost[dr::PIECES_LAYERS];
            for (int i = 0; i < n; ++i)
                if (scanf("%ld %lf", &tiles[i], &cost[i]) != 2) return 1;
            dr::PiecesPlan p;
            const bool found = dr::pieces_plan(n, tiles, cost, cus, &p);
            printf("%d %d %.6f", found, p.workgroups, p.us);
            for (int i = 0; found && i < n; ++i) {
                printf(" %d", p.layer[i].n);
                for (int k = 0; k < p.layer[i].n; ++k) printf(" %d %d %d %d", p.layer[i].first[k], p.layer[i].first[k + 1], p.layer[i].per[k], p.layer[i].tile[k]);
            }
            printf("\n");
        }
        return 0;
    }
    if (argc > 1 && !strcmp(argv[1], "choose")) {
        int n;
        while (scanf("%d", &n) == 1) {
            dr::PiecesLayer l[dr::PIECES_LAYERS];
            for (int i = 0; i < n; ++i) {
                if (scanf("%d %d %d %d %d", &l[i].N, &l[i].C, &l[i].H, &l[i].K, &l[i].R) != 5) return 1;
                l[i].S = l[i].R; l[i].W = l[i].P = l[i].Q = l[i].H; l[i].sh = l[i].sw = 1;
                printf("%d ", dr::pieces_pays(l[i], 256));
            }
            int type[dr::PIECES_LAYERS];
            dr::PiecesPlan p;
            if (!dr::pieces_choose(n, l, 256, type, &p)) return 1;
            for (int i = 0; i < n; ++i) printf("%d ", type[i]);
            printf("\n");
        }
        return 0;
    }
    dr::PiecesLayer l;
    int ph, pw;
    while (scanf("%d %d %d %d %d %d %d %d %d %d %d", &l.N, &l.C, &l.H, &l.W, &l.K, &l.R, &l.S, &l.sh, &l.sw, &ph, &pw) == 11) {
        l.P = (l.H + 2 * ph - l.R) / l.sh + 1;
        l.Q = (l.W + 2 * pw - l.S) / l.sw + 1;
        double us = 0;
        printf("%d %d %d", dr::pieces_pays(l, 256), dr::direct_pays(l, 256), l.sh * l.sw > 1 ? dr::direct_best(l, 256, &us) : dr::pieces_best(l, 256, &us));
        for (const dr::PiecesTile& t : dr::pieces_tiles) printf(" %d", dr::pieces_fits(l, t) ? t.patch : 0);
        printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("pieces")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=undefined", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan")])

    def ask(lines, *args):
        out = subprocess.run([str(d / "plan"), *args], input="\n".join(lines), capture_output=True, text=True, check=True, timeout=60).stdout.splitlines()
        assert len(out) == len(lines)
        return [line.split() for line in out]
    return ask


def patch_pixels(P, Q, R, S, first, last):
    """Input pixels under the outputs first .. last of a stack of P x Q maps: per image the rows under its rows, Q + S - 1 wide."""
    rows = 0
    for img in range(first // (P * Q), last // (P * Q) + 1):
        a, b = max(first, img * P * Q) - img * P * Q, min(last, (img + 1) * P * Q - 1) - img * P * Q
        # the first image from its first row of the tile on, the others from their first row on
        rows += (b // Q if img == last // (P * Q) else P - 1) - (a // Q if img == first // (P * Q) else 0) + R
    return rows * (Q + S - 1)


def test_a_tile_that_fits_has_room_for_every_patch(program):
    rng = random.Random(4)
    layers = []
    while len(layers) < 400:
        R, S = rng.choice(((3, 3), (5, 5), (2, 4), (4, 2), (1, 9), (9, 1), (7, 7), (3, 5)))
        H, W = rng.choice((rng.randint(1, 12), rng.randint(5, 80))), rng.choice((rng.randint(1, 12), rng.randint(5, 80)))
        ph, pw = rng.randint(0, R), rng.randint(0, S)
        if H + 2 * ph >= R and W + 2 * pw >= S:
            layers.append((rng.randint(1, 40), 16, H, W, 64, R, S, 1, 1, ph, pw))
    fitting = 0
    for (N, _, H, W, _, R, S, _, _, ph, pw), (_, _, _, *caps) in zip(layers, program([" ".join(map(str, l)) for l in layers])):
        P, Q = H + 2 * ph - R + 1, W + 2 * pw - S + 1
        for pixels, cap in zip((128, 128, 128, 256), map(int, caps)):
            if not cap:
                continue
            fitting += 1
            most = max(patch_pixels(P, Q, R, S, n, min(n + pixels, N * P * Q) - 1) for n in range(0, N * P * Q, pixels))
            assert most <= cap and most <= R * S // 2 * 128, (N, H, W, R, S, ph, pw, pixels)
    assert fitting > 500


def test_the_kernel_and_tile_of_the_gpu_cases(program):
    from test_gpu_conv_f32_pieces import CASES, FAR, STRIDED
    got = program([" ".join(map(str, c[:7] + (1, 1) + c[7])) for c, _ in CASES] + [" ".join(map(str, c[:7] + c[7] + c[8])) for c, _ in STRIDED])
    assert [tuple(map(int, v[:3])) for v in got] == [(1, 0, t) for _, t in CASES] + [(0, 1, t) for _, t in STRIDED]
    assert [v[:2] for v in program([" ".join(map(str, FAR[s] + (s, s, 1, 1))) for s in (1, 2)])] == [["1", "0"], ["0", "1"]]
    # the layers with operands that pieces cannot hold
    assert [v[:2] for v in program(["28 32 30 30 96 3 3 1 1 1 1", "28 32 30 30 96 3 3 1 1 0 0", "40 32 41 33 200 3 3 2 2 1 1", "40 32 41 33 200 3 3 2 2 0 0"])] == [["1", "0"]] * 2 + [["0", "1"]] * 2


def test_the_tiles_of_layers_that_share_a_launch(program):
    """The modules of the GPU test: every layer is taken, and the launches have one tile for all and several."""
    from test_gpu_conv_f32_pieces import SHARED
    lines, expect = [], []
    for n, layers, tiles in SHARED:
        order = sorted(range(len(layers)), key=lambda i: -((layers[i][2] ** 2 * (layers[i][0] // 16) + 1) // 2))      # the longest contraction first
        lines.append("%d " % len(layers) + " ".join("%d %d 28 %d %d" % (n, layers[i][0], layers[i][1], layers[i][2]) for i in order))
        expect.append([1] * len(layers) + [tiles[i] for i in order])
    assert [list(map(int, v)) for v in program(lines, "choose")] == expect


def test_what_stays_with_the_other_kernels(program):
    taken = ((32, 96, 28, 28, 128, 3, 3, 1, 1, 1, 1), (52, 160, 28, 28, 288, 3, 3, 2, 2, 1, 1))
    beside = [(32, 96, 28, 28, 128, 1, 1, 1, 1, 0, 0),       # one tap
              (32, 96, 28, 28, 128, 3, 3, 2, 1, 1, 1),       # a stride in one direction
              (32, 24, 28, 28, 128, 3, 3, 1, 1, 1, 1),       # channels not in sixteens
              (32, 96, 28, 28, 128, 2, 4, 1, 1, 0, 3),       # eight taps
              (1, 96, 28, 28, 128, 3, 3, 1, 1, 1, 1),        # one image: few tiles
              (2, 16, 28, 300, 128, 3, 3, 1, 1, 1, 1),       # a row of 300 pixels
              (4, 16, 1200, 60, 64, 3, 3, 1, 1, 1, 1),       # 72000 pixels
              (64, 160, 7, 7, 320, 3, 3, 1, 1, 1, 1),        # tiles for half of the compute units
              (24, 16, 28, 28, 96, 3, 3, 1, 1, 1, 1),        # a block of 16 channels: short contractions
              (24, 16, 28, 28, 96, 5, 5, 1, 1, 2, 2),
              (128, 96, 28, 28, 256, 5, 5, 2, 2, 2, 2),      # strided, whole tiles of 64 filters
              (5, 64, 56, 56, 96, 3, 3, 2, 2, 1, 1),         # strided: not enough faster
              (97, 128, 35, 34, 40, 5, 5, 2, 2, 2, 2)]       # strided, 40 filters
    got = [v[:2] for v in program([" ".join(map(str, l)) for l in [*taken] + beside])]
    assert got == [["1", "0"], ["0", "1"]] + [["0", "0"]] * len(beside)


def test_every_tile_has_one_workgroup(program):
    rng = random.Random(5)
    cases = [(1, 256, [(1, 10.0)]), (1, 256, [(256, 10.0)]), (1, 256, [(257, 10.0)]), (2, 256, [(196, 27.0), (196, 12.5)]), (4, 256, [(1, 9.0), (1, 8.0), (1, 7.0), (1, 6.0)]),
             (1, 1, [(7, 3.0)]), (3, 256, [(100000, 50.0), (3, 1.0), (70000, 1.0)])]
    while len(cases) < 3000:
        n = rng.randint(1, 4)
        cases.append((n, rng.choice((1, 2, 8, 64, 256, 304)), sorted([(int(10 ** rng.uniform(0, 4)), rng.uniform(3, 100)) for _ in range(n)], key=lambda v: -v[1])))
    for (n, cus, layers), out in zip(cases, program(["%d %d " % (n, cus) + " ".join("%d %.6f" % v for v in layers) for n, cus, layers in cases], "plan")):
        assert out[0] == "1", (n, cus, layers)
        workgroups, us, v = int(out[1]), float(out[2]), [int(x) for x in out[3:]]
        assert 1 <= workgroups <= cus
        load = [0.0] * cus
        for tiles, cost in layers:
            ranges, v = v[0], v[1:]
            at, wg = 0, 0
            for _ in range(ranges):
                (first, end, per, tile), v = v[:4], v[4:]
                assert first == wg and end > first
                wg = end
                if per:
                    assert tile == at and end <= workgroups
                    at += per * (end - first)
                    for w in range(first, end):
                        load[w] += per * cost
            assert wg == cus and at == tiles, (n, cus, layers)
        assert max(load) == pytest.approx(us, rel=1e-6)
        # no longer than the work spread evenly and one more tile of each layer
        assert us <= sum(t * c for t, c in layers) / cus + sum(c for _, c in layers) + 1e-6


RULES = r"""
#include <cstdio>
#include "dr_internal.h"
using namespace dr;
int main()
{
    int stride, K, N, H, residual;
    while (scanf("%d %d %d %d %d", &stride, &K, &N, &H, &residual) == 5) {
        ConvGeom g{};
        g.N = N; g.C = 160; g.H = g.W = H; g.K = K; g.R = g.S = 3; g.sh = g.sw = stride; g.ph = g.pw = 1;
        g.P = g.Q = (H - 1) / stride + 1; g.Kg = g.C * 9; g.Ng = N * g.P * g.Q; g.y_ctot = K; g.w_krsc = 1;
        g.res_ctot = residual ? K : 0;
        ConvSmall job{};
        job.g = g;
        job.res = residual ? &g : nullptr;
        printf("%d %d %d %d", conv_f32_pieces_takes(g), conv_f32_direct_takes(g), conv_f32_small_takes(g, nullptr, false), conv_f32_scratch_bytes(g) != 0);
        // (refused before anything is launched)
        if (residual) printf(" %d", stride == 1 ? launch_conv_f32_pieces(&job, 1, nullptr) : launch_conv_f32_direct(job, nullptr));
        printf("\n");
    }
}
"""


def test_a_residual_stays_with_the_other_kernels(tmp_path):
    """A 3x3 layer with a residual is not counted as theirs, and keeps the kernel for small layers; the launchers refuse it."""
    rocm = "/opt/rocm"
    if not os.path.exists(os.path.join(rocm, "include", "hip", "hip_runtime.h")):
        pytest.skip("no HIP headers")
    from paper_1708_04728_amd import binding as B
    (tmp_path / "rules.cpp").write_text(RULES)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w", "-I", CSRC, "-I", os.path.join(rocm, "include"), str(tmp_path / "rules.cpp"), B.LIB_PATH,
                           "-Wl,--allow-shlib-undefined", "-Wl,-rpath," + os.path.dirname(B.LIB_PATH), "-o", str(tmp_path / "rules")])
    cases = ((1, 96, 16, 28), (1, 128, 14, 28), (2, 288, 52, 28))
    lines = ["%d %d %d %d %d" % (c + (r,)) for c in cases for r in (0, 1)]
    out = subprocess.run([str(tmp_path / "rules")], input="\n".join(lines), capture_output=True, text=True, check=True, timeout=60).stdout.splitlines()
    # pieces, direct, small layers, scratch; the launcher's answer
    refused = " %d" % B.DR_ERR_UNSUPPORTED
    assert out == ["1 0 0 0", "0 0 1 0" + refused, "1 0 0 0", "0 0 1 0" + refused, "0 1 0 0", "0 0 0 0" + refused]
