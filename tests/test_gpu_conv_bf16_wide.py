"""GPU parity of the wide-tile bf16 convolution kernel (one persistent workgroup per compute unit, loading and multiplying waves
apart) against the fp64 oracle: every tile the library's rule picks (restated in `tile`), ragged filters and pixels, one round and
several, slices inside a tap, running on from filter row to filter row and starting one, strides, few slices; the store at channel
offsets, stacked first steps; and, beside each line of the rule, layers that stay with the streaming kernel."""
import numpy as np
import pytest

import oracle
import workloads
from paper_1708_04728_amd import binding as B
from util import case_seed, close, gpu, gpu_nhwc, host_nhwc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CUS = 256
TILES = [(5, 7), (4, 7), (7, 4), (6, 5), (3, 7), (6, 4), (4, 4), (2, 7), (2, 5), (4, 3)]


def slices(C, R, S):
    run = S * (C // 8)
    spr, flat = -(-run // 8), -(-R * run // 8)
    return flat if run >= 8 and flat < R * spr else R * spr


def tile(case):
    """The library's rule, restated: (TM, TN, rounds) of a tile of 32 TM filters x 32 TN pixels, None = not this kernel."""
    N, C, H, W, K, R, S, stride, pad = case
    ng = N * oracle.conv_out_size(H, R, stride, pad) * oracle.conv_out_size(W, S, stride, pad)
    t64, n = -(-ng // 64) * -(-K // 64), slices(C, R, S)
    if t64 <= CUS or K % 8 or K <= 32 or n < 3 or n > 128:
        return None
    best = None
    for tm, tn in TILES:
        bm, bn = 32 * tm, 32 * tn
        gm, gn_ = -(-K // bm), -(-ng // bn)
        gn = min(max(CUS // gm, 1), gn_)
        rounds = -(-gn_ // gn) * -(-gn * gm // CUS)
        us = rounds * (n * max(0.644 * bm * bn / 32768, 12.85 * (bm + bn) / 8192) + 0.54 + 1.2 * bm * bn / 10000)
        if best is None or us < best[0] * (1 - 1e-6):
            best = (us, (tm, tn, rounds))
    tm, tn, rounds = best[1]
    return None if rounds > 1 and n <= (3 if R * S > 1 else 4) else best[1]


def run(case, relu, off=0, extra=0, bias=True):
    N, C, H, W, K, R, S, stride, pad = case
    rng = np.random.default_rng(case_seed(case))
    x = workloads.round_to_bf16(rng.standard_normal((N, C, H, W)).astype(np.float32))
    w = workloads.round_to_bf16(rng.standard_normal((K, C, R, S)).astype(np.float32) * np.float32(np.sqrt(2.0 / (C * R * S))))
    b = (rng.standard_normal(K) * 0.1).astype(np.float32) if bias else None
    ref = oracle.conv2d(x, w, b, stride, pad, relu)
    y = B.NHWC(torch.full((N, ref.shape[2], ref.shape[3], K + off + extra), -7.0, dtype=torch.bfloat16, device="cuda"))
    B.conv2d_fwd(gpu_nhwc(x, "bf16"), B.conv_desc(K, C, R, S, stride, pad, relu, B.DR_KRSC), B.pack_filters(gpu(w, "bf16")), gpu(b) if bias else None, y,
                 y_c_offset=off)
    torch.cuda.synchronize()
    got = host_nhwc(y)
    assert (got[:, :off] == -7.0).all() and (got[:, off + K:] == -7.0).all()
    # one rounding of an fp32 sum: within one unit of the last place of the rounded exact result
    assert close(got[:, off:off + K], oracle.round_bf16(ref), 2.0 ** -7, "within one bf16 unit of the oracle")


@pytest.mark.parametrize("expected,case", [
    # (TM, TN, rounds), (N, C, H, W, K, R, S, stride, pad)
    ((2, 5, 1), (17, 8, 41, 15, 72, 3, 3, 1, 1)),                 # 3 slices
    ((2, 5, 2), (31, 24, 41, 47, 40, 3, 3, 1, 1)),                # 4 slices
    ((2, 7, 1), (22, 8, 36, 52, 40, 3, 3, 1, 1)),                 # 3 slices
    ((2, 7, 2), (55, 24, 58, 28, 40, 3, 3, 1, 1)),                # 4 slices
    ((3, 7, 1), (56, 8, 60, 39, 72, 3, 3, 2, 1)),                 # 3 slices
    ((3, 7, 2), (60, 24, 28, 30, 192, 5, 5, 1, 2)),               # 10 slices
    ((4, 3, 1), (25, 8, 26, 37, 72, 3, 3, 1, 1)),                 # 3 slices
    ((4, 3, 1), (40, 200, 15, 13, 328, 1, 1, 1, 0)),              # 4 slices
    ((4, 4, 1), (40, 8, 17, 48, 72, 3, 3, 1, 1)),                 # 3 slices
    ((4, 4, 2), (57, 264, 39, 27, 72, 1, 1, 1, 0)),               # 5 slices
    ((4, 7, 1), (46, 8, 41, 23, 104, 3, 3, 1, 1)),                # 3 slices
    ((4, 7, 2), (60, 24, 29, 30, 224, 3, 3, 1, 1)),               # 4 slices
    ((5, 7, 1), (47, 8, 37, 46, 288, 3, 3, 2, 1)),                # 3 slices
    ((6, 5, 2), (50, 24, 28, 29, 312, 3, 3, 1, 1)),               # 4 slices
    ((6, 4, 1), (42, 8, 44, 16, 136, 3, 3, 1, 1)),                # 3 slices
    ((6, 5, 1), (54, 8, 38, 16, 152, 3, 3, 1, 1)),                # 3 slices
    ((7, 4, 1), (45, 8, 33, 10, 392, 3, 3, 1, 1)),                # 3 slices
    ((2, 5, 1), (33, 136, 14, 14, 288, 3, 3, 1, 1)),              # 20 slices
    ((3, 7, 1), (60, 88, 21, 30, 96, 2, 3, 1, 1)),                # 9 slices
    ((3, 7, 1), (60, 24, 56, 29, 176, 4, 3, 2, 1)),               # 5 slices
])
def test_wide(expected, case):
    assert tile(case) == expected, tile(case)
    seed = case_seed(case)
    run(case, relu=seed % 2 == 0, off=8 * (seed % 3), extra=8 * (seed % 2), bias=seed % 4 != 0)


@pytest.mark.parametrize("case,off", [
    ((1, 16, 90, 190, 68, 3, 3, 1, 1), 0),         # filters no multiple of 8
    ((2, 24, 140, 120, 32, 3, 3, 1, 1), 0),        # 32 filters
    ((4, 24, 96, 84, 72, 3, 3, 1, 1), 4),          # channel offset no multiple of 8
    ((1, 128, 180, 190, 72, 1, 1, 1, 0), 0),       # two slices
    ((5, 256, 160, 170, 80, 1, 1, 1, 0), 0),       # 1x1, four slices, more than one round
    ((16, 8, 120, 130, 136, 3, 3, 2, 1), 0),       # three slices in more than one round
    ((35, 1032, 14, 14, 176, 3, 3, 1, 1), 0),      # 146 slices: beyond the table
])
def test_streaming_kernel_beside_the_lines(case, off):
    """Layers just beyond the lines of the rule keep to the streaming kernel."""
    assert off % 8 or tile(case) is None
    run(case, relu=True, off=off)


def test_stacked_first_steps():
    """First steps of a module as one layer: its filter ranges go to the concat output and to tensors of their own.  Bit for bit the
    banks one by one (smaller layers, other tiles)."""
    gen = torch.Generator(device="cuda").manual_seed(3)
    N, C, H, W = 40, 480, 14, 15
    ks = (192, 96, 16)
    x = torch.randn((N, H, W, C), device="cuda", generator=gen).abs().to(torch.bfloat16)
    inc = {"branches": [[("conv", dict(k=192, r=1, s=1, stride=1, pad=0)), ("relu", {})],
                        [("conv", dict(k=96, r=1, s=1, stride=1, pad=0)), ("relu", {}), ("conv", dict(k=40, r=1, s=1, stride=1, pad=0)), ("relu", {})],
                        [("conv", dict(k=16, r=1, s=1, stride=1, pad=0)), ("relu", {}), ("conv", dict(k=48, r=1, s=1, stride=1, pad=0)), ("relu", {})]]}
    from paper_1708_04728_amd import graph as G
    assert tile((N, C, H, W, sum(ks), 1, 1, 1, 0)) is not None
    layers = [("inception", inc)]
    params = []
    for k, c in ((192, C), (96, C), (40, 96), (16, C), (48, 16)):
        params += [B.pack_filters((torch.randn((k, c, 1, 1), device="cuda", generator=gen) * (2.0 / c) ** 0.5).to(torch.bfloat16)),
                   torch.randn(k, device="cuda", generator=gen) * 0.1]
    out = []
    for mode in (B.DR_FUSE_RELU | B.DR_FUSE_CONCAT | B.DR_FUSE_STACK, B.DR_FUSE_RELU | B.DR_FUSE_CONCAT):
        p = G.stack_first_steps(layers, params) if mode & B.DR_FUSE_STACK else params
        d = G.inception_desc(inc, C, mode, "bf16")
        y = torch.full((N, H, W, 192 + 40 + 48), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.empty(max(B.inception_workspace_bytes(B.NHWC(x), d), 256), dtype=torch.uint8, device="cuda")
        B.inception_fwd(B.NHWC(x), d, p[0::2], p[1::2], B.NHWC(y), ws)
        out.append(y)
    torch.cuda.synchronize()
    assert torch.isfinite(out[0].float()).all() and float(out[0].float().abs().max()) > 0
    assert torch.equal(out[0], out[1])
