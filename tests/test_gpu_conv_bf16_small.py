"""GPU parity of the small-layer bf16 convolution kernel (loading and multiplying waves apart, several layers per launch) against
the fp64 oracle, where it can go wrong: contractions of one slice and of every remainder of the ring, both slice modes,
ragged filters / pixels / channel runs, every border, the scalar store, all three tile shapes, the largest layer it takes;
and modules whose branches share launches, with the pooling step in them."""
import numpy as np
import pytest

import oracle
import workloads
from bf16_rules import route
from paper_1708_04728_amd import binding as B
from util import TOL_BF16, case_seed, close, empty_nhwc, gpu, gpu_nhwc, host_nhwc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("case", [
    # N, C, H, W, K, R, S, stride, pad
    (1, 8, 5, 7, 8, 3, 3, 1, 1),          # 72 values: two slices, one channel chunk per tap
    (1, 24, 9, 11, 40, 3, 3, 1, 1),       # slices that run on from filter row to filter row, ragged filters
    (2, 40, 13, 10, 100, 5, 5, 2, 2),     # stride 2, filters no multiple of 8 (scalar store)
    (1, 64, 6, 6, 33, 3, 3, 1, 1),        # whole taps, 9 slices, a second filter block of one filter
    (3, 128, 7, 9, 64, 3, 3, 2, 1),       # two slices per tap
    (1, 16, 4, 4, 16, 3, 1, 1, 0),        # a filter row shorter than a slice: no run-on, three slices
    (1, 64, 3, 5, 24, 1, 1, 1, 0),        # one slice
    (1, 264, 3, 5, 24, 1, 1, 1, 0),       # 1x1, ragged run: 5 slices
    (1, 320, 9, 9, 56, 1, 1, 2, 0),       # strided 1x1
    (4, 96, 64, 64, 64, 1, 1, 1, 0),      # 256 tiles of 64 x 64: the largest layer with 1x1 filters
    (1, 48, 64, 61, 96, 3, 3, 1, 1),      # 64 x 32 tiles, half a filter block
    (2, 40, 43, 46, 200, 1, 1, 1, 0),     # 64 x 64 tiles in stages of one slice: one
    (1, 16, 41, 44, 344, 3, 3, 1, 1),     # three
    (5, 32, 36, 35, 72, 3, 3, 1, 1),      # five
    (10, 24, 29, 28, 72, 3, 3, 1, 1),     # 64 x 64 tiles in stages of two: four slices
    (12, 48, 22, 25, 96, 3, 3, 1, 1),     # seven
    (2, 24, 96, 84, 100, 3, 3, 1, 1),     # 504 tiles of 64 x 64, two to a compute unit, ragged; scalar store
    (3, 40, 96, 84, 32, 5, 5, 1, 2),      # two to a compute unit: 32 filters of 64, whole groups of 8
    (2, 24, 96, 84, 104, 3, 3, 1, 1),     # as many by itself: wide tiles
    (1, 1032, 2, 3, 8, 3, 3, 1, 1),       # long contraction, 146 slices
])
def test_small_layer(case):
    N, C, H, W, K, R, S, stride, pad = case
    assert route(case)[0] == ("wide" if case == (2, 24, 96, 84, 104, 3, 3, 1, 1) else "small"), route(case)
    rng = np.random.default_rng(case_seed(case))
    x = workloads.round_to_bf16(rng.standard_normal((N, C, H, W)).astype(np.float32))
    w = workloads.round_to_bf16(rng.standard_normal((K, C, R, S)).astype(np.float32) * np.float32(np.sqrt(2.0 / (C * R * S))))
    for bias, relu in ((True, True), (False, False)):
        b = (rng.standard_normal(K) * 0.1).astype(np.float32) if bias else None
        ref = oracle.conv2d(x, w, b, stride, pad, relu)
        y = empty_nhwc(ref.shape, "bf16")
        cd = B.conv_desc(K, C, R, S, stride, pad, relu, B.DR_KRSC)
        B.conv2d_fwd_ws(gpu_nhwc(x, "bf16"), cd, B.pack_filters(gpu(w, "bf16")), None if b is None else gpu(b), y, None)
        torch.cuda.synchronize()
        got = host_nhwc(y)
        # one rounding of an fp32 sum: within one unit of the last place of the rounded exact result, which is 2^-7 of a power of two and less
        # of any other value; close() asks for less than its bound, so that this lies above by the spacing of the doubles compared
        assert close(got, oracle.round_bf16(ref), 2.0 ** -7 * (1 + 2.0 ** -50), "within one bf16 unit of the oracle")


@pytest.mark.parametrize("case", [
    # N, C, H, W, K, R, S, stride, pad
    (1, 1792, 3, 4, 24, 3, 3, 1, 1),      # 252 slices: the longest contraction the chunk table holds
    (1, 1856, 3, 4, 24, 3, 3, 1, 1),      # 261: beyond it, worked out chunk by chunk; rows of whole slices
    (1, 648, 5, 7, 24, 5, 5, 1, 2),       # 254 slices that run on; the table would hold them, but not what is read ahead
    (2, 656, 6, 5, 40, 5, 5, 2, 2),       # 257 that run on, worked out: a row's last slice goes on into the next one
    (1, 1832, 2, 12, 24, 1, 9, 1, 4),     # one row of 2061 chunks, filter rows outside the image
    (1, 512, 7, 7, 200, 7, 7, 1, 0),      # a classifier's first layer: one pixel
    (1, 1856, 64, 65, 40, 3, 3, 1, 1),    # tiles of 64 x 32
    (1, 1856, 93, 90, 8, 3, 3, 1, 1),     # 64 x 64
    (1, 1856, 129, 130, 8, 3, 3, 1, 1),   # 64 x 64, two to a compute unit
    (1, 16448, 1, 3, 24, 1, 1, 1, 0),     # 1x1 filters at stride 1 need no table
    (1, 8, 19, 14, 16, 16, 9, 1, 4),      # the most filter rows and columns
    (2, 16, 9, 9, 40, 4, 3, 1, 1),        # filter rows shorter than a slice, an odd and an even number of slices left over
    (2, 88, 9, 9, 40, 2, 2, 1, 1),        # 22 chunks per filter row, two of them: six slices either way, every row starts one
    (1, 8, 5, 7, 1, 1, 1, 1, 0),          # one slice: the stage's second one begins 112 bytes behind the filter tensor
    (1, 8, 9, 7, 5, 1, 1, 2, 0),          # 48 bytes
    (2, 72, 6, 5, 1, 3, 3, 1, 1),         # 11 slices that run on: the twelfth begins 112 bytes behind it
])
def test_chunk_table(case):
    """Where a chunk of the contraction lies, over the forms of the table, against the fp64 oracle: one rounding of an fp32 sum."""
    N, C, H, W, K, R, S, stride, pad = case
    rng = np.random.default_rng(case_seed(case))
    x = workloads.round_to_bf16(rng.standard_normal((N, C, H, W)).astype(np.float32))
    w = workloads.round_to_bf16(rng.standard_normal((K, C, R, S)).astype(np.float32) * np.float32(np.sqrt(2.0 / (C * R * S))))
    b = (rng.standard_normal(K) * 0.1).astype(np.float32)
    ref = oracle.conv2d(x, w, b, stride, pad, False)
    y = empty_nhwc(ref.shape, "bf16")
    B.conv2d_fwd_ws(gpu_nhwc(x, "bf16"), B.conv_desc(K, C, R, S, stride, pad, False, B.DR_KRSC), B.pack_filters(gpu(w, "bf16")), gpu(b), y, None)
    torch.cuda.synchronize()
    assert close(host_nhwc(y), oracle.round_bf16(ref), 2.0 ** -7, "within one bf16 unit of the oracle")


@pytest.mark.parametrize("few,many,layer,tile,kernel", [
    # images with which the layer is a small one and with which it is not; C, H, W, K, R, S, stride, pad; the tile; the other kernel
    (2, 3, (24, 96, 84, 100, 3, 3, 1, 1), "64 x 64 twice", ("stream", "64 x 128")),       # slices that run on from filter row to filter row
    (1, 10, (24, 96, 84, 100, 3, 3, 1, 1), "64 x 64", ("stream", "128 x 256")),
    (10, 11, (128, 28, 28, 96, 1, 1, 1, 0), "64 x 64", ("stream", "64 x 64")),
    (1, 37, (200, 28, 28, 232, 1, 1, 1, 0), "32 x 32", ("stream", "128 x 128")),
    (6, 14, (64, 28, 28, 192, 3, 3, 1, 1), "64 x 64", ("patch",)),                        # whole taps
    (3, 46, (64, 28, 28, 192, 3, 3, 1, 1), "64 x 32", ("patch",)),
    (4, 15, (32, 64, 64, 64, 5, 5, 1, 2), "64 x 64", ("rows",)),
    (8, 34, (48, 14, 14, 304, 3, 3, 1, 1), "64 x 32", ("rows",)),
    (7, 8, (72, 96, 96, 64, 3, 3, 2, 1), "64 x 64", ("wide", 2, 5, 1)),                   # stride 2
    (5, 6, (200, 28, 28, 232, 1, 1, 1, 0), "64 x 64", ("wide", 2, 5, 1)),
    (16, 67, (160, 7, 7, 320, 3, 3, 1, 1), "32 x 32", ("wide", 2, 5, 1)),
])
def test_the_larger_kernels_bits(few, many, layer, tile, kernel):
    """The slices are multiplied in the order of the kernels for larger layers: the images of a batch within the rule have the bits
    that they have in one beyond it."""
    C, H, W, K, R, S, stride, pad = layer
    assert route((few,) + layer)[:2] == ("small", tile) and route((many,) + layer)[:len(kernel)] == kernel
    gen = torch.Generator(device="cuda").manual_seed(C)
    x = torch.randn((many, H, W, C), device="cuda", generator=gen).to(torch.bfloat16)
    w = B.pack_filters((torch.randn((K, C, R, S), device="cuda", generator=gen) * (2.0 / (C * R * S)) ** 0.5).to(torch.bfloat16))
    b = torch.randn(K, device="cuda", generator=gen) * 0.1
    cd = B.conv_desc(K, C, R, S, stride, pad, True, B.DR_KRSC)
    out = []
    for n in (few, many):
        y = torch.full((n, oracle.conv_out_size(H, R, stride, pad), oracle.conv_out_size(W, S, stride, pad), K), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.conv2d_fwd_ws(B.NHWC(x[:n]), cd, w, b, B.NHWC(y), None)
        out.append(y)
    torch.cuda.synchronize()
    assert torch.isfinite(out[1].float()).all() and float(out[1].float().abs().max()) > 0
    assert torch.equal(out[0], out[1][:few])


def test_small_layer_into_an_odd_channel_range():
    """A destination that 8-byte stores do not fit, other channels untouched."""
    rng = np.random.default_rng(3)
    x = workloads.round_to_bf16(rng.standard_normal((1, 16, 6, 6)).astype(np.float32))
    w = workloads.round_to_bf16(rng.standard_normal((20, 16, 3, 3)).astype(np.float32) * np.float32(0.1))
    ref = oracle.round_bf16(oracle.conv2d(x, w, None, 1, 1, False))
    wide = B.NHWC(torch.full((1, 6, 6, 33), -3.0, dtype=torch.bfloat16, device="cuda"))
    B.conv2d_fwd_ws(gpu_nhwc(x, "bf16"), B.conv_desc(20, 16, 3, 3, 1, 1, False, B.DR_KRSC), B.pack_filters(gpu(w, "bf16")), None, wide, None, y_c_offset=7)
    torch.cuda.synchronize()
    got = host_nhwc(wide)
    assert close(got[:, 7:27], ref, 2.0 ** -7)
    assert (got[:, :7] == -3.0).all() and (got[:, 27:] == -3.0).all()


@pytest.mark.parametrize("n,hw", [(1, (14, 14)), (2, (9, 13)), (5, (7, 7))])
@pytest.mark.parametrize("form", ["original", "slim"])
def test_module_whose_branches_share_launches(form, n, hw):
    """An inception module small enough for step-by-step execution, in every mode: against the oracle (the storage rule
    mirrored), stacked first steps with the bits of one convolution per branch."""
    from test_gpu_bf16_nets import run_net_bf16
    layer = (workloads.inception_original if form == "original" else workloads.inception_slim)("4b")
    rng = np.random.default_rng(17 + n)
    x = workloads.round_to_bf16(np.abs(rng.standard_normal((n, 512) + hw)).astype(np.float32))
    params = []
    workloads._walk(rng, [layer], 512, "bf16", params)
    ref = oracle.forward([layer], params, x, mirror_bf16=True)
    base = B.DR_FUSE_RELU | B.DR_FUSE_CONCAT
    plain = run_net_bf16([layer], params, x, inception_mode=base)
    for mode in (0, B.DR_CONCURRENT_BRANCHES, B.DR_FUSE_RELU, base, base | B.DR_CONCURRENT_BRANCHES):
        got = run_net_bf16([layer], params, x, inception_mode=mode)
        assert close(got, ref, TOL_BF16, "mode %d" % mode)
        assert np.array_equal(got, plain), mode
    from paper_1708_04728_amd import graph as G
    xg = G.to_device(x, "bf16", nhwc=True)
    net = B.Net(G.net_descs([layer], 512, inception_mode=base | B.DR_FUSE_STACK, pack="bf16"))
    y = G.empty_like_desc(net.output_desc(B.desc(xg)))
    ws = torch.empty(max(net.workspace_bytes(B.desc(xg)), 256), dtype=torch.uint8, device="cuda")
    net.fwd(xg, G.stack_first_steps([layer], G.flat_params(params, "bf16", pack=True)), y, ws)
    torch.cuda.synchronize()
    assert np.array_equal(G.to_host(y), plain)


@pytest.mark.parametrize("N,K,S,stride", [(2, 64, 128, 2), (1, 20, 93, 4), (2, 64, 130, 2)])
def test_first_layer_at_the_edge_of_the_rule(N, K, S, stride):
    """7x7 on three channels through the padded copy: the largest layer that runs here (128 x 128 outputs of two images = 512
    pixel tiles), a scalar store, and the first size that goes to the streaming kernel."""
    from test_gpu_bf16_nets import run_net_bf16
    rng = np.random.default_rng(S)
    H = S * stride
    x = workloads.round_to_bf16(rng.standard_normal((N, 3, H, H)).astype(np.float32))
    w = workloads.round_to_bf16(rng.standard_normal((K, 3, 7, 7)).astype(np.float32) * np.float32(0.1))
    b = (rng.standard_normal(K) * 0.1).astype(np.float32)
    layers = [workloads.conv(K, 7, stride, 3), workloads.relu()]
    got = run_net_bf16(layers, [{"w": w, "b": b}], x, fuse_relu=True)
    ref = oracle.forward(layers, [{"w": w, "b": b}], x)
    assert got.shape == (N, K, S, S)
    assert close(got, oracle.round_bf16(ref), 2.0 ** -7)


@pytest.mark.parametrize("N,I,O", [(1, 1024, 1000), (33, 72, 10), (70, 264, 200)])
def test_inner_product(N, I, O):
    """One-pixel images: a single row, ragged inputs, outputs that 8-byte stores do not fit."""
    rng = np.random.default_rng(I)
    x = workloads.round_to_bf16(rng.standard_normal((N, I)).astype(np.float32))
    w = workloads.round_to_bf16(rng.standard_normal((O, I)).astype(np.float32) * np.float32(I ** -0.5))
    b = rng.standard_normal(O).astype(np.float32)
    y = torch.empty((N, O), dtype=torch.bfloat16, device="cuda")
    B.fc_fwd(gpu(x, "bf16"), gpu(w, "bf16"), gpu(b), y)
    torch.cuda.synchronize()
    ref = x.astype(np.float64) @ w.astype(np.float64).T + b
    assert close(y.float().cpu().numpy(), oracle.round_bf16(ref.astype(np.float32)), 2.0 ** -7)
