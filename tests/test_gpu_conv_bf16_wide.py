"""GPU parity of the wide-tile bf16 convolution kernel (one persistent workgroup per compute unit, loading and multiplying waves
apart) against the fp64 oracle: every tile the library's rule picks (restated in bf16_rules.py), ragged filters and pixels, one round and
several, slices inside a tap, running on from filter row to filter row and starting one, strides, few slices; the store at channel
offsets, stacked first steps; and, beside each line of the rule, layers that stay with the streaming kernel."""
import numpy as np
import pytest

import oracle
import workloads
from bf16_rules import route, wide_fills
from paper_1708_04728_amd import binding as B
from util import case_seed, close, gpu, gpu_nhwc, host_nhwc, kernel_launches

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

def tile(case):
    """(TM, TN, rounds) where the layer by itself runs in wide tiles, or None."""
    r = route(case)
    return r[1:] if r[0] == "wide" else None


def run(case, relu, off=0, extra=0, bias=True, images=None):
    N, C, H, W, K, R, S, stride, pad = case
    rng = np.random.default_rng(case_seed(case))
    x = workloads.round_to_bf16(rng.standard_normal((N, C, H, W)).astype(np.float32))
    w = workloads.round_to_bf16(rng.standard_normal((K, C, R, S)).astype(np.float32) * np.float32(np.sqrt(2.0 / (C * R * S))))
    b = (rng.standard_normal(K) * 0.1).astype(np.float32) if bias else None
    pick = list(range(N)) if images is None else images
    ref = oracle.conv2d(x[pick], w, b, stride, pad, relu)
    y = B.NHWC(torch.full((N, ref.shape[2], ref.shape[3], K + off + extra), -7.0, dtype=torch.bfloat16, device="cuda"))
    B.conv2d_fwd(gpu_nhwc(x, "bf16"), B.conv_desc(K, C, R, S, stride, pad, relu, B.DR_KRSC), B.pack_filters(gpu(w, "bf16")), gpu(b) if bias else None, y,
                 y_c_offset=off)
    torch.cuda.synchronize()
    got = host_nhwc(y)
    assert (got[:, :off] == -7.0).all() and (got[:, off + K:] == -7.0).all()
    # one rounding of an fp32 sum: within one unit of the last place of the rounded exact result
    assert not np.isnan(got).any()
    assert close(got[pick, off:off + K], oracle.round_bf16(ref), 2.0 ** -7, "within one bf16 unit of the oracle")


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
    ((2, 5, 1), (1500, 64, 5, 5, 40, 3, 3, 1, 1)),                # maps of 25 pixels: a step of 32 leaves the image
    ((4, 7, 1), (4000, 40, 3, 4, 104, 3, 3, 1, 1)),               # 12: two images and 8 pixels on
    ((2, 5, 1), (22000, 24, 3, 3, 40, 3, 3, 1, 0)),               # one pixel: 32 images on
])
def test_wide(expected, case):
    assert tile(case) == expected, tile(case)
    seed = case_seed(case)
    run(case, relu=seed % 2 == 0, off=8 * (seed % 3), extra=8 * (seed % 2), bias=seed % 4 != 0)


@pytest.mark.parametrize("case,off,images", [
    ((1, 16, 90, 190, 68, 3, 3, 1, 1), 0, None),            # filters no multiple of 8
    ((2, 24, 140, 120, 32, 3, 3, 1, 1), 0, None),           # 32 filters
    ((4, 24, 96, 84, 72, 3, 3, 1, 1), 4, None),             # channel offset no multiple of 8
    ((1, 128, 180, 190, 72, 1, 1, 1, 0), 0, None),          # two slices
    ((5, 256, 160, 170, 80, 1, 1, 1, 0), 0, [0, 4]),        # 1x1, four slices, more than one round
    ((16, 8, 120, 130, 136, 3, 3, 2, 1), 0, None),          # three slices in more than one round
    ((56, 1032, 14, 14, 176, 3, 3, 1, 1), 0, [0, 31, 55]),  # 146 slices: beyond the table
])
def test_streaming_kernel_beside_the_lines(case, off, images):
    """Layers just beyond the lines of the rule keep to the streaming kernel."""
    assert route(case, off)[0] == "stream", route(case, off)
    run(case, relu=True, off=off, images=images)


def outputs(case, offs, batches):
    """The layer's outputs in a batch of each size, written at each channel offset."""
    N, C, H, W, K, R, S, stride, pad = case
    gen = torch.Generator(device="cuda").manual_seed(K)
    x = torch.randn((max(batches), H, W, C), device="cuda", generator=gen).to(torch.bfloat16)
    w = B.pack_filters((torch.randn((K, C, R, S), device="cuda", generator=gen) * (2.0 / (C * R * S)) ** 0.5).to(torch.bfloat16))
    b = torch.randn(K, device="cuda", generator=gen) * 0.1
    cd, out = B.conv_desc(K, C, R, S, stride, pad, True, B.DR_KRSC), []
    for off, n in zip(offs, batches):
        y = torch.full((n, oracle.conv_out_size(H, R, stride, pad), oracle.conv_out_size(W, S, stride, pad), K + off), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.conv2d_fwd(B.NHWC(x[:n]), cd, w, b, B.NHWC(y), y_c_offset=off)
        out.append(y[..., off:])
    torch.cuda.synchronize()
    assert torch.isfinite(out[0].float()).all() and float(out[0].float().abs().max()) > 0
    return out


@pytest.mark.parametrize("case", [
    (12, 64, 92, 90, 128, 3, 3, 2, 1),         # whole taps
    (8, 24, 100, 100, 104, 3, 3, 1, 1),        # slices that run on from filter row to filter row
    (6, 88, 56, 60, 200, 3, 3, 1, 1),          # every row starts one
    (7, 328, 55, 57, 96, 1, 1, 1, 0),
    (20, 40, 70, 66, 72, 5, 5, 2, 2),
])
def test_the_streaming_kernels_bits(case):
    """The same layer at a channel offset of 8 (wide tiles) and of 4 (streaming kernel): the order of the sums is the same."""
    assert route(case, 8)[0] == "wide" and route(case, 4)[0] == "stream", (route(case, 8), route(case, 4))
    a, b = outputs(case, (8, 4), (case[0], case[0]))
    assert torch.equal(a, b)


@pytest.mark.parametrize("layer,wide,patch,kernel", [
    # C, H, W, K, R, S, stride, pad; images with which it runs in wide tiles, and in a kernel with an input patch, on either side of a line
    ((64, 28, 28, 192, 3, 3, 1, 1), 21, 20, "patch"),      # half a workgroup of the other kernel per compute unit
    ((64, 28, 28, 192, 3, 3, 1, 1), 45, 46, "patch"),      # little more than one
    ((64, 28, 28, 64, 3, 3, 1, 1), 73, 74, "patch"),
    ((32, 28, 28, 128, 5, 5, 1, 2), 45, 46, "rows"),
    ((48, 14, 15, 304, 3, 3, 1, 1), 39, 38, "rows"),
    ((48, 14, 15, 304, 3, 3, 1, 1), 84, 85, "rows"),
])
def test_the_patch_kernels_bits(layer, wide, patch, kernel):
    """The images of a batch have the same bits in wide tiles and in a kernel with an input patch, one image more or fewer."""
    assert route((wide,) + layer)[0] == "wide" and wide_fills((wide,) + layer)
    assert route((patch,) + layer)[0] == kernel and not wide_fills((patch,) + layer)
    a, b = outputs((wide,) + layer, (0, 0), (wide, patch))
    n = min(wide, patch)
    assert torch.equal(a[:n], b[:n])


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


@pytest.mark.parametrize("n,c,h,w,widths", [
    # 1x1 | reduce, 3x3 | reduce, 5x5 | pool projection
    (40, 64, 14, 14, (64, 96, 208, 16, 48, 64)),            # small layers that crowd the device
    (3, 24, 61, 67, (8, 40, 232, 24, 32, 8)),               # eight filters, eight filters more than a block of 224, a pixel tile that is not whole
    (90, 32, 13, 15, (256, 160, 320, 32, 128, 128)),        # several rounds
    (25, 200, 15, 13, (72, 56, 104, 8, 16, 20)),            # a projection of 20 filters, which stays out
    (17, 40, 28, 28, (24, 360, 48, 344, 40, 48)),           # 5x5 on 344 channels: more chunks than the table holds
    (13, 64, 14, 15, (192, 92, 208, 44, 48, 64)),           # 3x3 on 92 channels, 5x5 on 44: on streams of their own where the caller wants that
    (128, 16, 7, 7, (384, 24, 384, 48, 128, 128)),
])
def test_layers_of_a_depth_share_a_launch(n, c, h, w, widths):
    """A module whose layers at one depth share a launch of wide tiles, in every mode: the bits of one launch per layer (which is what a
    kernel trace makes the library do), and the oracle's result on its first and last image."""
    from test_gpu_bf16_nets import run_net_bf16
    a, b3, k3, b5, k5, pp = widths
    conv, relu = workloads.conv, workloads.relu
    layer = ("inception", {"branches": [[conv(a, 1), relu()], [conv(b3, 1), relu(), conv(k3, 3, 1, 1), relu()], [conv(b5, 1), relu(), conv(k5, 5, 1, 2), relu()],
                                        [workloads.maxpool(3, 1, 1), conv(pp, 1), relu()]]})
    rng = np.random.default_rng(case_seed((n, c, h, w, widths)))
    x = workloads.round_to_bf16(np.abs(rng.standard_normal((n, c, h, w))).astype(np.float32))
    params = []
    workloads._walk(rng, [layer], c, "bf16", params)
    base = B.DR_FUSE_RELU | B.DR_FUSE_CONCAT
    B.trace_begin()
    plain = run_net_bf16([layer], params, x, inception_mode=base)
    B.trace_end()
    for mode in (0, B.DR_CONCURRENT_BRANCHES, B.DR_FUSE_RELU, base, base | B.DR_CONCURRENT_BRANCHES):
        assert np.array_equal(run_net_bf16([layer], params, x, inception_mode=mode), plain), mode
    pick = [0, n - 1]
    assert close(plain[pick], oracle.forward([layer], params, x[pick], mirror_bf16=True), 2e-2)


@pytest.mark.parametrize("n,c,h,w,pool", [
    (400, 8, 21, 1, (3, 1, 1)),              # one column, one channel group: an item per strip; a strip of one row at the end
    (448, 16, 3, 6, (3, 1, 1)),              # as many groups of items as may lie beside the layers on 256 compute units
    (449, 16, 3, 6, (3, 1, 1)),              # ... and one more: a launch of its own
    (60, 520, 13, 11, (3, 1, 1)),            # six groups an image, the last one not whole
    (8, 40, 1, 1000, (3, 1, 1)),             # rows of which a strip has one
    (5, 64, 40, 41, (3, 1, 1)),              # a share of few workgroups
])
def test_a_pooling_step_beside_the_layers(n, c, h, w, pool):
    """A module's pooling step in the launch of its first layers: the bits of a launch for each, also of negative values and where windows are cut off."""
    from test_gpu_bf16_nets import run_net_bf16
    conv, relu = workloads.conv, workloads.relu
    layer = ("inception", {"branches": [[conv(256, 1), relu()], [conv(128, 1), relu(), conv(64, 3, 1, 1), relu()], [workloads.maxpool(*pool), conv(64, 1), relu()]]})
    rng = np.random.default_rng(case_seed((n, c, h, w)))
    x = workloads.round_to_bf16(rng.standard_normal((n, c, h, w)).astype(np.float32) - 2)
    params = []
    workloads._walk(rng, [layer], c, "bf16", params)
    base = B.DR_FUSE_RELU | B.DR_FUSE_CONCAT
    B.trace_begin()
    plain = run_net_bf16([layer], params, x, inception_mode=base)
    B.trace_end()
    for mode in (0, base, base | B.DR_CONCURRENT_BRANCHES):
        assert np.array_equal(run_net_bf16([layer], params, x, inception_mode=mode), plain), mode
    pick = [0, n - 1]
    assert close(plain[pick], oracle.forward([layer], params, x[pick], mirror_bf16=True), 2e-2)


@pytest.mark.parametrize("branches,c,h,w", [
    ([[("conv", 30000)], [("conv", 30000)]], 8, 14, 14),             # more blocks of filters than compute units to run them side by side
    ([[("conv", 30000)], [("conv", 30000)]], 8, 7, 7),
    ([[("conv", 57400)], [("maxpool", 0), ("conv", 16)]], 264, 7, 7),       # a single one with the pooling step
    ([[("conv", 14400)], [("conv", 14400)], [("conv", 14400)], [("conv", 14400)]], 8, 7, 9),      # small layers that would crowd the device
])
def test_layers_too_wide_to_share_a_launch(branches, c, h, w):
    """A module whose layers have more filters than fit the compute units side by side runs them one by one."""
    from test_gpu_bf16_nets import run_net_bf16
    layer = ("inception", {"branches": [[s for kind, k in branch for s in ([workloads.conv(k, 1), workloads.relu()] if kind == "conv" else [workloads.maxpool(3, 1, 1)])]
                                        for branch in branches]})
    rng = np.random.default_rng(case_seed((branches, c, h, w)))
    x = workloads.round_to_bf16(rng.standard_normal((1, c, h, w)).astype(np.float32))
    params = []
    workloads._walk(rng, [layer], c, "bf16", params)
    base = B.DR_FUSE_RELU | B.DR_FUSE_CONCAT
    B.trace_begin()
    plain = run_net_bf16([layer], params, x, inception_mode=base)
    B.trace_end()
    for mode in (0, base, base | B.DR_FUSE_STACK, base | B.DR_CONCURRENT_BRANCHES):
        assert np.array_equal(run_net_bf16([layer], params, x, inception_mode=mode), plain), mode
    assert close(plain, oracle.forward([layer], params, x, mirror_bf16=True), 2e-2)


@pytest.mark.parametrize("n,c,h,w,branches,launches", [
    # branches: widths of a 1x1, of a 1x1 and what follows it, ("pool", width of the projection); kernels with ReLU and concat in the stores
    (448, 16, 3, 6, [(256,), (128, (3, 64)), ("pool", 64)], 2),            # as many groups of pooling items as may lie beside the layers of a depth
    (449, 16, 3, 6, [(256,), (128, (3, 64)), ("pool", 64)], 3),            # ... and one more: a launch of its own
    (40, 64, 14, 14, [(64,), (96, (3, 208)), (16, (5, 48)), ("pool", 64)], 2),      # small layers that crowd the device
    (4, 64, 14, 14, [(64,), (96, (3, 208)), (16, (5, 48)), ("pool", 64)], 2),       # ... and that do not: the kernel for small layers
    (25, 200, 15, 13, [(72,), (56, (3, 104)), (8, (5, 16)), ("pool", 20)], 3),      # a projection of 20 filters stays out
    (1, 8, 14, 14, [(30000,), (30000,)], 2),                                         # too wide to lie side by side
])
def test_launches_of_a_module(n, c, h, w, branches, launches):
    """How many kernels a module takes: which of its layers share a launch."""
    from paper_1708_04728_amd import graph as G
    conv, relu, layers, shapes = workloads.conv, workloads.relu, [], []
    for first, *rest in branches:
        steps, ci = ([workloads.maxpool(3, 1, 1)], c) if first == "pool" else ([conv(first, 1), relu()], first)
        if first != "pool":
            shapes.append((first, c, 1))
        for r in rest:
            r, k = r if isinstance(r, tuple) else (1, r)
            steps += [conv(k, r, 1, r // 2), relu()]
            shapes.append((k, ci, r))
            ci = k
        layers.append(steps)
    x = B.NHWC(torch.zeros((n, h, w, c), dtype=torch.bfloat16, device="cuda"))
    weights = [B.pack_filters(torch.zeros((k, ci, r, r), dtype=torch.bfloat16, device="cuda")) for k, ci, r in shapes]
    biases = [torch.zeros(k, device="cuda") for k, _, _ in shapes]
    d = G.inception_desc({"branches": layers}, c, B.DR_FUSE_RELU | B.DR_FUSE_CONCAT, "bf16")
    y = B.NHWC(torch.zeros((n, h, w, sum((b[-1][1] if isinstance(b[-1], tuple) else b[-1]) for b in branches)), dtype=torch.bfloat16, device="cuda"))
    ws = torch.empty(max(B.inception_workspace_bytes(x, d), 256), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    assert kernel_launches(lambda: B.inception_fwd(x, d, weights, biases, y, ws)) == launches
