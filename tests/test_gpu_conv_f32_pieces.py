"""GPU parity of the fp32 kernel on three bf16 pieces against the oracle: at the edges of its tiles (128 x 128, 96 x 128, 64 x 128 and 64 x 256 filters x pixels), its
slices and its patches, which cross rows and images; and operands that bf16 pieces cannot hold."""
import numpy as np
import pytest

import oracle
from paper_1708_04728_amd import binding as B
from util import TOL_F32, case_seed, close, gpu, host, note, rms_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def run(x, w, b, pad, relu, k_off=0):
    K, C, R, S = w.shape
    (N, _, H, W), (ph, pw) = x.shape, pad
    P, Q = H + 2 * ph - R + 1, W + 2 * pw - S + 1
    cd = B.conv_desc(K, C, R, S, 1, pad, relu, B.DR_KRSC)
    y = torch.full((N, K + 3, P, Q), float("nan"), device="cuda")
    B.conv2d_fwd(gpu(x), cd, B.pack_filters(gpu(w)), None if b is None else gpu(b), y, 2)
    torch.cuda.synchronize()
    assert bool(torch.isnan(y[:, :2]).all()) and bool(torch.isnan(y[:, K + 2:]).all())
    return host(y[:, 2:K + 2])


@pytest.mark.parametrize("case", [
    # N, C, H, W, K, R, S, pad: with 256 compute units the tile that the comment names
    (70, 16, 7, 43, 250, 3, 3, (0, 0)),     # 128 x 128, the last block of filters not whole; one block of channels
    (9, 32, 39, 46, 97, 3, 3, (2, 1)),      # ... more padding than the taps need
    (19, 32, 25, 41, 127, 4, 2, (0, 0)),    # ... eight taps: a block is four slices
    (150, 16, 46, 12, 128, 1, 9, (1, 0)),   # ... one row of taps
    (37, 32, 31, 17, 97, 9, 1, (2, 1)),     # ... one column
    (19, 48, 20, 55, 65, 3, 3, (0, 1)),     # 96 x 128, three blocks of channels: blocks start in the middle of a slice
    (5, 16, 86, 35, 129, 3, 3, (2, 2)),     # ... one filter in the last block
    (19, 16, 40, 27, 65, 5, 5, (1, 0)),     # ... 25 taps
    (9, 32, 43, 50, 64, 3, 3, (0, 0)),      # 64 x 128
    (300, 16, 7, 7, 65, 3, 3, (1, 1)),      # ... several images under a tile
    (700, 16, 5, 4, 72, 3, 3, (1, 1)),      # ... seven
    (37, 16, 39, 15, 33, 7, 7, (3, 3)),     # ... 49 taps
    (5, 16, 56, 56, 97, 3, 3, (1, 1)),      # ... the widest rows
    (37, 32, 55, 21, 33, 3, 3, (1, 1)),     # 64 x 256
    (9, 16, 86, 21, 250, 3, 3, (2, 0)),     # ...
    (37, 16, 43, 23, 33, 5, 5, (3, 2)),     # ... the largest patches
    (37, 32, 45, 10, 129, 9, 1, (5, 0)),    # ...
])
def test_pieces(case):
    N, C, H, W, K, R, S, pad = case
    rng = np.random.default_rng(case_seed(case))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((K, C, R, S)).astype(np.float32) * np.float32(np.sqrt(2.0 / (C * R * S)))
    b = rng.standard_normal(K).astype(np.float32)
    ref = oracle.conv2d(x, w, b, 1, pad, True)
    got = run(x, w, b, pad, True)
    assert close(got, ref, TOL_F32)
    # C R S / 16 sums of 16 products with 2^-24 of rounding each, and the pieces' small products at 2^-8 of that
    assert note("rms", rms_err(got, ref), 4 * 2.0 ** -24 * np.sqrt(C * R * S / 16) + 2.0 ** -24)
    assert close(run(x, w, None, pad, False), oracle.conv2d(x, w, np.zeros(K, np.float32), 1, pad, False), TOL_F32)


def test_operands_beyond_bf16_pieces():
    """Infinities, NaN, values that round to infinity in 8 bits, and operands whose lower pieces are too small for a bf16: as fp32 arithmetic has them."""
    N, C, H, W, K = 20, 32, 30, 30, 96
    rng = np.random.default_rng(7)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((K, C, 3, 3)).astype(np.float32) * np.float32(0.1)
    plain = run(x, w, None, (1, 1), False)
    big = x.copy()
    big[1, 3, 5, 7], big[2, 4, 0, 0], big[3, 31, 29, 29], big[4, 0, 9, 9] = np.inf, -np.inf, np.nan, 3.4e38
    got = run(big, w, None, (1, 1), False)
    with np.errstate(all="ignore"):
        ref = torch.nn.functional.conv2d(torch.from_numpy(big).double(), torch.from_numpy(w).double(), padding=1).numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    there = np.isfinite(ref)
    near = there & (np.abs(ref) > 1e30)
    assert near.sum() == 9 * K and np.max(np.abs(got[near] / ref[near] - 1)) < 1e-6
    assert close(got[there & ~near], ref[there & ~near], TOL_F32)
    wi = w.copy()
    wi[5, 2, 1, 1] = np.inf
    got, ref = run(x, wi, None, (0, 0), False), torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(wi).double()).numpy()
    assert np.isinf(got[:, 5]).all() and np.array_equal(np.sign(got[:, 5]), np.sign(ref[:, 5]))
    assert np.array_equal(np.delete(got, 5, 1), np.delete(run(x, w, None, (0, 0), False), 5, 1)) or close(np.delete(got, 5, 1), np.delete(ref, 5, 1), TOL_F32)
    # images and filters of their own magnitudes: 2^-118 .. 2^-90 beside 1
    for scale in (2.0 ** -118, 2.0 ** -103, 2.0 ** -90):
        small = x.copy()
        small[::2] *= np.float32(scale)
        got = run(small, w, None, (1, 1), False)
        ref = oracle.conv2d(small, w, np.zeros(K, np.float32), 1, 1, False)
        assert close(got[::2], ref[::2], TOL_F32, "2^%d" % np.log2(scale)) and close(got[1::2], ref[1::2], TOL_F32)
        ws = w.copy()
        ws[::3] *= np.float32(scale)
        got = run(x, ws, None, (1, 1), False)
        ref = oracle.conv2d(x, ws, np.zeros(K, np.float32), 1, 1, False)
        assert close(got[:, ::3], ref[:, ::3], TOL_F32, "2^%d" % np.log2(scale)) and close(np.delete(got, np.s_[::3], 1), np.delete(ref, np.s_[::3], 1), TOL_F32)
    assert np.array_equal(plain, run(x, w, None, (1, 1), False))


def test_layers_of_a_module_share_a_launch():
    """A 3x3 and a 5x5 layer side by side, with tiles of their own: the bits of each by itself."""
    N, side = 24, 28
    branches = [[("conv", {"k": 16, "r": 1, "s": 1, "stride": 1, "pad": 0}), ("relu", {}), ("conv", {"k": 96, "r": r, "s": r, "stride": 1, "pad": r // 2}), ("relu", {})] for r in (3, 5)]
    from paper_1708_04728_amd import graph as G
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((N, 64, side, side), device="cuda", generator=gen).abs()
    weights, biases = [], []
    for r in (3, 5):
        for k, c, s in ((16, 64, 1), (96, 16, r)):
            weights.append(B.pack_filters(torch.randn((k, c, s, s), device="cuda", generator=gen) * (2.0 / (c * s * s)) ** 0.5))
            biases.append(torch.randn(k, device="cuda", generator=gen) * 0.1)
    desc = G.inception_desc({"branches": branches}, 64, B.DR_FUSE_RELU | B.DR_FUSE_CONCAT, "f32")
    y = torch.empty((N, 192, side, side), device="cuda")
    ws = torch.empty(max(B.inception_workspace_bytes(x, desc), 256), dtype=torch.uint8, device="cuda")
    B.inception_fwd(x, desc, weights, biases, y, ws)
    alone = torch.empty_like(y)
    for i, r in enumerate((3, 5)):
        t = torch.empty((N, 16, side, side), device="cuda")
        B.conv2d_fwd(x, B.conv_desc(16, 64, 1, 1, 1, 0, True, B.DR_KRSC), weights[2 * i], biases[2 * i], t)
        B.conv2d_fwd(t, B.conv_desc(96, 16, r, r, 1, r // 2, True, B.DR_KRSC), weights[2 * i + 1], biases[2 * i + 1], alone, 96 * i)
    torch.cuda.synchronize()
    assert torch.equal(y, alone)
