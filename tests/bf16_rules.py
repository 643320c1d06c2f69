"""The rules by which the library picks the kernel of a bf16 channels-last convolution with KRSC filters, restated: `route` names the kernel and
its tile, so that a test can say which one its cases are for.  A case is (N, C, H, W, K, R, S, stride, pad), a destination a channel offset
`off` in a tensor of K + off + extra channels; pointers are aligned, and the layer runs by itself (no launch shared, no other streams)."""
import oracle

CUS = 256
WIDE_TILES = [(5, 7), (4, 7), (7, 4), (6, 5), (3, 7), (6, 4), (4, 4), (2, 7), (2, 5), (4, 3)]


def ceil(a, b):
    return -(-a // b)


def out_size(case):
    N, C, H, W, K, R, S, stride, pad = case
    return oracle.conv_out_size(H, R, stride, pad), oracle.conv_out_size(W, S, stride, pad)


def slices(C, R, S, depth=64):
    """Slices of `depth` contraction elements: they run on from filter row to filter row where that saves some, else every row starts one."""
    run, per = S * (C // 8), depth // 8
    return min(ceil(R * run, per), R * ceil(run, per)) if run >= per else R * ceil(run, per)


def patch_rows(case):
    """conv_bf16_patch: output rows per tile, 0 = not for this kernel."""
    N, C, H, W, K, R, S, stride, pad = case
    P, Q = out_size(case)
    if C % 64 or K % 8 or stride != 1 or R * S < 2 or R > 7 or S > 7 or Q < 2 or Q > 256:
        return 0
    th = min(256 // Q, P)
    while th >= 1 and (C // 64) * (ceil((th + R - 1) * (W + 2 * pad), 32) * 32) > 352:
        th -= 1
    return th if th >= 1 and th * Q * 4 >= 256 * 3 else 0


def rows_rows(case):
    """conv_bf16_rows: stacked output rows per tile, 0 = not for this kernel."""
    N, C, H, W, K, R, S, stride, pad = case
    P, Q = out_size(case)
    if C % 16 or C > 64 or K % 8 or stride != 1 or R * S < 2 or R > 7 or S > 7 or P < 2 or Q < 2 or Q > 256:
        return 0
    tm = 3 if ceil(K, 96) * 96 <= ceil(K, 64) * 64 else 2
    budget = 80 * 1024 - (2 * tm * 32 * 128 + 512 + 1024)
    th = min(256 // Q, N * P)
    while th >= 1:
        segs = min(N, (th + P - 2) // P + 1)
        if ceil((th + (R - 1) * segs) * (W + 2 * pad) * (C // 8 + 1) * 16, 4096) * 4096 <= budget:
            break
        th -= 1
    if th < 1 or th * Q * 4 < 256 * 3:
        return 0
    return th if ceil(N * P, th) * ceil(K, tm * 32) * 4 >= CUS else 0


def wide_tile(K, ng, n):
    """conv_bf16_wide's model: (TM, TN, rounds) of a tile of 32 TM filters x 32 TN pixels."""
    best = None
    for tm, tn in WIDE_TILES:
        bm, bn = 32 * tm, 32 * tn
        gm, tiles = ceil(K, bm), ceil(ng, bn)
        gn = min(max(CUS // gm, 1), tiles)
        rounds = ceil(tiles, gn) * ceil(gn * gm, CUS)
        us = rounds * (n * max(0.644 * bm * bn / 32768, 12.85 * (bm + bn) / 8192) + 0.54 + 1.2 * bm * bn / 10000)
        if best is None or us < best[0] * (1 - 1e-6):
            best = (us, (tm, tn, rounds))
    return best[1]


def wide_takes(case, aligned=True):
    """(TM, TN, rounds), None = not conv_bf16_wide."""
    N, C, H, W, K, R, S, stride, pad = case
    P, Q = out_size(case)
    n = slices(C, R, S)
    if not aligned or K % 8 or K <= 32 or n < 3 or n > 128:
        return None
    t = wide_tile(K, N * P * Q, n)
    return None if t[2] > 1 and n <= (3 if R * S > 1 else 4) else t


def wide_fills(case):
    """Where it goes before the kernels with an input patch."""
    N, C, H, W, K, R, S, stride, pad = case
    P, Q = out_size(case)
    groups = ceil(K, 96) * ceil(N * P * Q, 252)
    return 2 * groups > CUS and 10 * groups <= 11 * CUS and wide_tile(K, N * P * Q, slices(C, R, S))[2] == 1


def stream_tile(K, ng, taps):
    """conv_bf16_dma's tile: filters x pixels."""
    if ceil(K, 64) * ceil(ng, 64) <= 2 * CUS:
        return "64 x 64"
    if K <= 32:
        return "32 x 128" if ceil(ng, 256) < CUS else "32 x 256"
    if taps > 1 and 96 < K <= 128 and CUS <= ceil(ng, 256) <= 2 * CUS:
        return "128 x 256"

    def rounds(bm):
        r = ceil(K, bm) * ceil(ng, 128) / (2 * CUS)
        return 1 if r <= 1 else (ceil(int(r * 2 * CUS), 2 * CUS) if r < 3 else r)
    c64, c96, r128 = rounds(64) * 2.44, rounds(96) * 3.44, rounds(128)
    if r128 <= 1 and r128 * 4.44 < min(c64, c96):
        return "128 x 128"
    return "96 x 128" if c96 < c64 else "64 x 128"


def route(case, off=0, extra=0):
    """(kernel, what else it is told apart by)."""
    N, C, H, W, K, R, S, stride, pad = case
    P, Q = out_size(case)
    ng, taps, aligned = N * P * Q, R * S, off % 8 == 0 and (K + off + extra) % 8 == 0

    def tiles(bm, bn):
        return ceil(K, bm) * ceil(ng, bn)
    if C % 8 or S > 9 or R > 16 or ng >= 1 << 24 or P * Q > 65536:
        return ("other",)
    if tiles(64, 64) <= (2 if taps > 1 else 1) * CUS:
        n = slices(C, R, S)
        way = "side by side" if taps == 1 and stride == 1 and pad == 0 else "table" if (n + 3) * 8 <= 2048 else "long"
        if tiles(32, 32) <= CUS:
            return "small", "32 x 32", way
        if tiles(64, 32) <= CUS:
            return "small", "64 x 32", way
        if tiles(64, 64) <= CUS:
            return "small", "64 x 64 by one" if n in (1, 3, 5) else "64 x 64", way
        t = wide_takes(case, aligned)
        return ("wide",) + t if t else ("small", "64 x 64 twice", way)
    if aligned and not (wide_fills(case) and wide_takes(case)):
        if patch_rows(case):
            return "patch", patch_rows(case)
        if rows_rows(case):
            return "rows", rows_rows(case)
    t = wide_takes(case, aligned)
    return ("wide",) + t if t else ("stream", stream_tile(K, ng, taps), "whole taps" if C % 64 == 0 else "along rows")
