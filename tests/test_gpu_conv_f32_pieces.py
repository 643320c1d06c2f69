"""GPU parity of the fp32 kernels on three bf16 pieces against the oracle: at the edges of their tiles (128 x 128, 96 x 128, 64 x 128 and 64 x 256 filters x pixels),
slices and patches, which cross rows and images, and at strides; and operands that bf16 pieces cannot hold."""
import numpy as np
import pytest

import oracle
from paper_1708_04728_amd import binding as B
from util import TOL_F32, case_seed, close, gpu, host, note, rms_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def run(x, w, b, pad, relu, stride=(1, 1)):
    K, C, R, S = w.shape
    N, _, H, W = x.shape
    P, Q = (oracle.conv_out_size(*v) for v in ((H, R, stride[0], pad[0]), (W, S, stride[1], pad[1])))
    cd = B.conv_desc(K, C, R, S, stride, pad, relu, B.DR_KRSC)
    y = torch.full((N, K + 3, P, Q), float("nan"), device="cuda")
    B.conv2d_fwd(gpu(x), cd, B.pack_filters(gpu(w)), None if b is None else gpu(b), y, 2)
    torch.cuda.synchronize()
    assert bool(torch.isnan(y[:, :2]).all()) and bool(torch.isnan(y[:, K + 2:]).all())
    return host(y[:, 2:K + 2])


# N, C, H, W, K, R, S, pad; the tile that the rule gives each (tests/test_conv_f32_pieces_plan.py)
CASES = [
    ((5, 32, 80, 67, 97, 3, 3, (2, 1)), 0),      # 128 x 128: 97 filters; more padding than the taps need
    ((100, 32, 31, 6, 97, 1, 9, (0, 5)), 0),      # one row of taps
    ((102, 32, 11, 20, 97, 9, 1, (4, 1)), 0),     # one column
    ((215, 16, 55, 4, 97, 5, 5, (3, 1)), 0),     # one block of channels, 25 taps
    ((9, 32, 54, 49, 65, 3, 3, (0, 0)), 1),      # 96 x 128
    ((37, 48, 31, 18, 65, 9, 1, (5, 1)), 1),     # three blocks of channels: blocks start in the middle of a slice
    ((150, 32, 8, 12, 129, 1, 9, (1, 3)), 1),    # one image and a bit under a tile
    ((12, 16, 61, 31, 65, 5, 5, (2, 2)), 1),
    ((300, 32, 7, 7, 65, 3, 3, (1, 1)), 2),      # 64 x 128: three images under a tile, one filter in the last block
    ((732, 32, 5, 4, 72, 3, 3, (1, 1)), 2),      # seven
    ((5, 32, 56, 56, 97, 3, 3, (1, 1)), 2),      # the widest rows
    ((51, 16, 51, 11, 33, 7, 7, (1, 2)), 2),     # 49 taps
    ((13, 48, 18, 47, 127, 3, 3, (2, 1)), 2),
    ((29, 32, 52, 35, 33, 3, 3, (0, 1)), 3),     # 64 x 256
    ((55, 16, 29, 33, 33, 5, 5, (3, 0)), 3),     # the largest patches
    ((85, 32, 51, 11, 33, 9, 1, (5, 0)), 3),
]
# N, C, H, W, K, R, S, stride, pad; the tile that the rule gives each
STRIDED = [
    ((37, 32, 39, 31, 200, 3, 3, (2, 2), (1, 2)), 0),
    ((19, 16, 78, 150, 200, 4, 4, (4, 4), (1, 0)), 0),
    ((3, 16, 123, 119, 200, 5, 5, (2, 2), (3, 0)), 0),      # an odd number of k-steps: half of the last slice is empty
    ((5, 32, 137, 74, 200, 1, 9, (2, 2), (1, 2)), 0),
    ((19, 32, 40, 135, 65, 3, 3, (2, 2), (1, 0)), 1),
    ((37, 16, 49, 91, 65, 4, 4, (3, 2), (2, 0)), 1),
    ((9, 48, 123, 36, 129, 3, 3, (2, 2), (1, 2)), 2),
    ((2, 16, 118, 101, 257, 5, 5, (2, 2), (2, 3)), 2),
]


@pytest.mark.parametrize("case", [c[:7] + ((1, 1), c[7]) for c, _ in CASES] + [c for c, _ in STRIDED])
def test_pieces(case):
    N, C, H, W, K, R, S, stride, pad = case
    rng = np.random.default_rng(case_seed(case))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((K, C, R, S)).astype(np.float32) * np.float32(np.sqrt(2.0 / (C * R * S)))
    b = rng.standard_normal(K).astype(np.float32)
    ref = oracle.conv2d(x, w, b, stride, pad, True)
    got = run(x, w, b, pad, True, stride)
    assert close(got, ref, TOL_F32)
    # C R S / 16 sums of 16 products with 2^-24 of rounding each, and the pieces' small products at 2^-8 of that
    assert note("rms", rms_err(got, ref), 4 * 2.0 ** -24 * np.sqrt(C * R * S / 16) + 2.0 ** -24)
    assert close(run(x, w, None, pad, False, stride), oracle.conv2d(x, w, np.zeros(K, np.float32), stride, pad, False), TOL_F32)


@pytest.mark.parametrize("stride", (1, 2))
def test_operands_beyond_bf16_pieces(stride):
    """Infinities, NaN, values that round to infinity in 8 bits, and images and filters of small operands: as fp32 arithmetic has them."""
    N, C, H, W, K = (28, 32, 30, 30, 96) if stride == 1 else (40, 32, 41, 33, 200)
    ss = (stride, stride)
    rng = np.random.default_rng(7)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((K, C, 3, 3)).astype(np.float32) * np.float32(0.1)
    plain = run(x, w, None, (1, 1), False, ss)
    big = x.copy()
    big[1, 3, 5, 7], big[2, 4, 0, 0], big[3, 31, 29, 29], big[4, 0, 9, 9] = np.inf, -np.inf, np.nan, 3.4e38
    got = run(big, w, None, (1, 1), False, ss)
    with np.errstate(all="ignore"):
        ref = torch.nn.functional.conv2d(torch.from_numpy(big).double(), torch.from_numpy(w).double(), padding=1, stride=stride).numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    there = np.isfinite(ref)
    near = there & (np.abs(ref) > 1e30)
    assert near.sum() == (9 if stride == 1 else 4) * K and np.max(np.abs(got[near] / ref[near] - 1)) < 1e-6
    assert close(got[there & ~near], ref[there & ~near], TOL_F32)
    wi = w.copy()
    wi[5, 2, 1, 1] = np.inf
    got, ref = run(x, wi, None, (0, 0), False, ss), torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(wi).double(), stride=stride).numpy()
    assert np.isinf(got[:, 5]).all() and np.array_equal(np.sign(got[:, 5]), np.sign(ref[:, 5]))
    assert np.array_equal(np.delete(got, 5, 1), np.delete(run(x, w, None, (0, 0), False, ss), 5, 1)) or close(np.delete(got, 5, 1), np.delete(ref, 5, 1), TOL_F32)
    # images and filters of their own magnitudes: 2^-118 .. 2^-90 beside 1
    for scale in (2.0 ** -118, 2.0 ** -103, 2.0 ** -90):
        small = x.copy()
        small[::2] *= np.float32(scale)
        got = run(small, w, None, (1, 1), False, ss)
        ref = oracle.conv2d(small, w, np.zeros(K, np.float32), stride, 1, False)
        assert close(got[::2], ref[::2], TOL_F32, "2^%d" % np.log2(scale)) and close(got[1::2], ref[1::2], TOL_F32)
        ws = w.copy()
        ws[::3] *= np.float32(scale)
        got = run(x, ws, None, (1, 1), False, ss)
        ref = oracle.conv2d(x, ws, np.zeros(K, np.float32), stride, 1, False)
        assert close(got[:, ::3], ref[:, ::3], TOL_F32, "2^%d" % np.log2(scale)) and close(np.delete(got, np.s_[::3], 1), np.delete(ref, np.s_[::3], 1), TOL_F32)
    assert np.array_equal(plain, run(x, w, None, (1, 1), False, ss))


@pytest.mark.parametrize("scale", (-105, -118, -140))
@pytest.mark.parametrize("stride", (1, 2))
def test_small_operands_beside_a_larger_one(stride, scale):
    """Of every eight channels one is about 1 where the other operand is 0, the rest about 2^scale (2^-140: subnormal): the sums consist of those alone."""
    N, C, H, W, K = (28, 32, 30, 30, 96) if stride == 1 else (40, 32, 41, 33, 200)
    rng = np.random.default_rng(-scale)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((K, C, 3, 3)).astype(np.float32)
    few, many = np.s_[:, ::8], np.arange(C) % 8 != 0
    for tiny, other in ((x, w), (w, x)):
        tiny, other = tiny.copy(), other * np.float32(2.0 ** 30)
        tiny[:, many] *= np.float32(2.0 ** scale)
        other[few] = 0
        a, b = (tiny, other) if tiny.shape == x.shape else (other, tiny)
        ref = torch.nn.functional.conv2d(torch.from_numpy(a).double(), torch.from_numpy(b).double(), padding=1, stride=stride).numpy()
        # as test_pieces
        assert note("rms", rms_err(run(a, b, None, (1, 1), False, (stride, stride)), ref), 4 * 2.0 ** -24 * np.sqrt(C * 9 / 16) + 2.0 ** -24)


@pytest.mark.parametrize("stride", (1, 2))
def test_sums_of_large_operands(stride):
    """Sums of about 2^80 to 2^122, image by image: on both sides of where pieces end."""
    N, C, H, W, K = (28, 32, 30, 30, 96) if stride == 1 else (40, 32, 41, 33, 200)
    rng = np.random.default_rng(stride)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((K, C, 3, 3)).astype(np.float32)
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), padding=1, stride=stride).numpy()
    scale = np.float32(2.0) ** (np.linspace(37, 78, N).round().astype(np.float32).reshape(N, 1, 1, 1))
    got = run(x * scale, w * np.float32(2.0 ** 40), None, (1, 1), False, (stride, stride)) / (scale.astype(np.float64) * 2.0 ** 40)
    # products of fp32 instructions: C R S / 2 sums
    assert close(got, ref, TOL_F32) and note("rms", rms_err(got, ref), 4 * 2.0 ** -24 * np.sqrt(C * 9 / 2) + 2.0 ** -24)


# the layer that test_channels_2_gib_apart runs at each stride, with 1 pixel of padding, into a tensor of FAR_CHANNELS
FAR, FAR_CHANNELS = {1: (1, 32, 1000, 60, 97, 3, 3), 2: (1, 32, 2000, 120, 200, 3, 3)}, 4480


@pytest.mark.parametrize("stride", (1, 2))
def test_channels_2_gib_apart(stride):
    """The last channels of a tensor of 1000 x 60 pixels and 1.07 GB an image: two images' worth of offsets do not fit the short form of the store."""
    N, C, H, W, K, R, S = FAR[stride]
    rng = np.random.default_rng(stride)
    x, w, b = (rng.standard_normal(s).astype(np.float32) for s in ((N, C, H, W), (K, C, R, S), K))
    x[0, 5, 700, 9] = np.inf                              # a block that is computed again
    y = torch.empty((N, FAR_CHANNELS, 1000, 60), device="cuda")
    y[:, FAR_CHANNELS - K - 2:] = 7.0
    B.conv2d_fwd(gpu(x), B.conv_desc(K, C, R, S, stride, 1, True, B.DR_KRSC), B.pack_filters(gpu(w)), gpu(b), y, FAR_CHANNELS - K - 1)
    torch.cuda.synchronize()
    got = host(y[:, FAR_CHANNELS - K - 1:FAR_CHANNELS - 1])
    assert bool((y[:, FAR_CHANNELS - K - 2] == 7.0).all()) and bool((y[:, FAR_CHANNELS - 1] == 7.0).all())
    ref = torch.nn.functional.conv2d(*(torch.from_numpy(t).double() for t in (x, w, b)), padding=1, stride=stride).clamp(min=0).numpy()
    there = np.isfinite(ref)
    assert (~there).sum() > 0 and np.array_equal(np.isposinf(got), np.isposinf(ref)) and close(got[there], ref[there], TOL_F32)


@pytest.mark.parametrize("case", (CASES[4][0][:7] + ((1, 1), CASES[4][0][7]), STRIDED[4][0]))
def test_filters_on_any_word(case):
    """Filters and biases that start 4 bytes behind a 16-byte boundary (slices of a parameter buffer): the same bits."""
    N, C, H, W, K, R, S, stride, pad = case
    gen = torch.Generator(device="cuda").manual_seed(K)
    x, w, b = (torch.randn(s, device="cuda", generator=gen) for s in ((N, C, H, W), (K, C, R, S), (K,)))
    cd = B.conv_desc(K, C, R, S, stride, pad, True, B.DR_KRSC)
    P, Q = (oracle.conv_out_size(*v) for v in ((H, R, stride[0], pad[0]), (W, S, stride[1], pad[1])))
    got = []
    for shift in (0, 1):
        y = torch.full((N, K, P, Q), float("nan"), device="cuda")
        params = []
        for t in (B.pack_filters(w), b):
            room = torch.full((t.numel() + 4,), float("nan"), device="cuda")
            params.append(room[shift:shift + t.numel()].view(t.shape))
            params[-1].copy_(t)
            assert params[-1].data_ptr() % 16 == 4 * shift
        B.conv2d_fwd(x, cd, *params, y)
        torch.cuda.synchronize()
        got.append(y)
    assert bool(torch.isfinite(got[0]).all()) and torch.equal(got[0], got[1])


def test_layers_of_a_module_share_a_launch():
    """A 3x3 and a 5x5 layer of 16 channels side by side, which stay with the other kernels: the bits of each by itself."""
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


# images of 28 x 28; channels, filters and side of each layer behind a 1x1; the tile that each has in the launch they share
SHARED = [
    (32, ((96, 128, 3), (16, 128, 5)), (0, 2)),
    (32, ((32, 96, 3), (32, 96, 5)), (2, 1)),
    (40, ((32, 96, 3), (32, 96, 5), (32, 96, 3)), (1, 1, 1)),                   # one tile for all
    (40, ((32, 96, 3), (32, 96, 5), (32, 128, 3), (32, 64, 5)), (1, 1, 3, 2)),
]


@pytest.mark.parametrize("case", SHARED)
def test_layers_on_pieces_share_a_launch(case):
    """Layers side by side, with tiles of their own: the bits of each by itself, every time.  Among the images some whose pixels are small all over, some with sums
    beyond pieces, whose blocks are computed again, and ordinary ones, which are not touched by what a workgroup computed before."""
    from paper_1708_04728_amd import graph as G
    n, layers, _ = case
    side, c0 = 28, 64
    branches = [[("conv", {"k": c, "r": 1, "s": 1, "stride": 1, "pad": 0}), ("relu", {}), ("conv", {"k": k, "r": r, "s": r, "stride": 1, "pad": r // 2}), ("relu", {})]
                for c, k, r in layers]
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((n, c0, side, side), device="cuda", generator=gen).abs()
    plain = x.clone()
    x[1::3] *= 2.0 ** -104
    x[2::6] *= 2.0 ** 90
    weights, biases = [], []
    for c, k, r in layers:
        for m, ch, s in ((c, c0, 1), (k, c, r)):
            weights.append(B.pack_filters(torch.randn((m, ch, s, s), device="cuda", generator=gen) * (2.0 / (ch * s * s)) ** 0.5))
            biases.append(torch.zeros(m, device="cuda"))
    desc = G.inception_desc({"branches": branches}, c0, B.DR_FUSE_RELU | B.DR_FUSE_CONCAT, "f32")
    ktot = sum(k for _, k, _ in layers)
    ws = torch.empty(max(B.inception_workspace_bytes(x, desc), 256), dtype=torch.uint8, device="cuda")
    reference = torch.empty((n, ktot, side, side), device="cuda")
    B.inception_fwd(plain, desc, weights, biases, reference, ws)
    y, alone = torch.empty_like(reference), torch.empty_like(reference)
    at = 0
    for i, (c, k, r) in enumerate(layers):
        t = torch.empty((n, c, side, side), device="cuda")
        B.conv2d_fwd(x, B.conv_desc(c, c0, 1, 1, 1, 0, True, B.DR_KRSC), weights[2 * i], biases[2 * i], t)
        B.conv2d_fwd(t, B.conv_desc(k, c, r, r, 1, r // 2, True, B.DR_KRSC), weights[2 * i + 1], biases[2 * i + 1], alone, at)
        at += k
    for _ in range(3):
        y.fill_(float("nan"))
        B.inception_fwd(x, desc, weights, biases, y, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, alone)
    assert torch.equal(y[0::6], reference[0::6])      # (784 pixels: an image of odd number shares a block of 32 with the one before it)
    assert close(host(y[1::3]) * 2.0 ** 104, host(reference[1::3]), TOL_F32) and close(host(y[2::6]) * 2.0 ** -90, host(reference[2::6]), TOL_F32)
