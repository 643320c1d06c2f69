"""GPU parity of the tiled fp32 convolution's store against the oracle: whole and ragged blocks of 32 filters, stacked ranges that start at multiples of
8 (a descriptor for every eight filters) and elsewhere (element by element), residuals, no bias, offsets beyond 2 GiB."""
import numpy as np
import pytest

import oracle
import workloads
from paper_1708_04728_amd import binding as B, graph as G
from test_gpu_blocks import _run_stacked
from test_gpu_conv_bf16_chain import stage
from util import TOL_F32, case_seed, close, gpu, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def module_params(layer, c, rng):
    out = []
    for branch in layer[1]["branches"]:
        ci = c
        for kind, p in branch:
            if kind == "conv":
                w = rng.standard_normal((p["k"], ci, p["r"], p["r"])).astype(np.float32) * np.float32(np.sqrt(2.0 / (ci * p["r"] ** 2)))
                out.append({"w": w, "b": (rng.standard_normal(p["k"]) * 0.1).astype(np.float32)})
                ci = p["k"]
    return out


@pytest.mark.parametrize("widths,pack", [
    ((64, 32, 32), True),      # every block of 32 filters has one destination
    ((40, 24, 56), True),      # blocks of 32 with two destinations, eights with one
    ((20, 12, 13), True),      # eights with two; 45 filters in all
    ((20, 12, 13), False),
])
def test_stacked_ranges(widths, pack):
    """Three 1x1 branches on one input, one with a 3x3 behind it, on more pixels than the kernel for small layers takes; 2 and 7 images of 43 x 41."""
    c, h, w = 32, 43, 41
    a, b, k = widths
    conv, relu = workloads.conv, workloads.relu
    layer = ("inception", {"branches": [[conv(a, 1), relu()], [conv(b, 1), relu(), conv(k, 3, 1, 1), relu()], [conv(k, 1), relu()]]})
    rng = np.random.default_rng(case_seed((widths, pack)))
    params = module_params(layer, c, rng)
    for n in (3, 7):
        x = np.abs(rng.standard_normal((n, c, h, w))).astype(np.float32)
        ref = oracle.forward([layer], params, x)
        for mode in (B.DR_FUSE_RELU | B.DR_FUSE_STACK, B.DR_FUSE_RELU | B.DR_FUSE_CONCAT | B.DR_FUSE_STACK):
            assert close(_run_stacked(layer, params, x, mode, pack), ref, TOL_F32), (n, mode)


@pytest.mark.parametrize("mid,out", [(32, 96), (16, 77)])
def test_residual(mid, out):
    """Folded bottlenecks in fp32: the residual sum, on a filter count that fills its last block and on one that does not."""
    n, h, w = 5, 31, 33
    rng = np.random.default_rng(mid)
    layers, params = stage(rng, 32, ((mid, out), (mid, out)))
    x = np.abs(rng.standard_normal((n, 32, h, w))).astype(np.float32)
    ref = oracle.forward(layers, params, x, fold="given")
    net = B.Net(G.net_descs(layers, 32, folded=True))
    xg = gpu(x)
    y = torch.full(ref.shape, float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(max(net.workspace_bytes(B.desc(xg)), 256), dtype=torch.uint8, device="cuda")
    net.fwd(xg, G.flat_params(params, "f32"), y, ws)
    torch.cuda.synchronize()
    assert close(host(y), ref, TOL_F32)


@pytest.mark.parametrize("bias", [True, False])
def test_channels_2_gib_apart(bias):
    """24 filters into channels 520 .. 543 of a map of 1024 x 1024 with 544 channels: 2.3 GB of output, beyond the short form's offsets."""
    c, k, side, ctot = 16, 24, 1024, 544
    rng = np.random.default_rng(5)
    x = rng.standard_normal((1, c, side, side)).astype(np.float32)
    w = rng.standard_normal((k, c, 1, 1)).astype(np.float32) * np.float32(np.sqrt(2.0 / c))
    b = rng.standard_normal(k).astype(np.float32)
    y = torch.empty((1, ctot, side, side), dtype=torch.float32, device="cuda")
    y[:, ctot - k - 1:] = 7.0
    B.conv2d_fwd(gpu(x), B.conv_desc(k, c, 1, 1, 1, 0, True, B.DR_KCRS), gpu(w), gpu(b) if bias else None, y, ctot - k)
    torch.cuda.synchronize()
    got = host(y[:, ctot - k:])
    assert bool((y[:, ctot - k - 1] == 7.0).all())
    del y
    assert close(got, oracle.conv2d(x, w, b if bias else np.zeros(k, np.float32), 1, 0, True), TOL_F32)


def test_planes_of_a_gigabyte():
    """One filter on 13400 x 13400: three planes, the rows that an eight is rounded up to, are 2.15e9 bytes, beyond the short form's buffer."""
    side = 13400
    x = torch.rand((1, 1, side, side), device="cuda")
    w, b = torch.full((1, 1, 1, 1), 0.75, device="cuda"), torch.full((1,), -0.25, device="cuda")
    y = torch.full((1, 1, side, side), float("nan"), device="cuda")
    B.conv2d_fwd(x, B.conv_desc(1, 1, 1, 1, 1, 0, True, B.DR_KCRS), w, b, y)
    torch.cuda.synchronize()
    assert float((y - (x * 0.75 - 0.25).clamp(min=0)).abs().max()) <= 2.0 ** -22      # a product and a sum of values below 1, each rounded once


@pytest.mark.parametrize("side", [4400, 4608])
def test_residual_of_large_planes(side):
    """The residual sum on 8 filters of a map whose 27 planes, the rows that a block of 32 is rounded up to, end just below and beyond 2 GiB.  The 3x3 layer has
    its middle tap alone, so that the block is a sum per pixel."""
    rng = np.random.default_rng(side)
    c = 8
    params = [{"w": rng.standard_normal((1, c, 1, 1)).astype(np.float32) * np.float32(0.5), "b": np.full(1, 0.1, np.float32)},
              {"w": np.zeros((1, 1, 3, 3), np.float32), "b": np.full(1, 0.2, np.float32)},
              {"w": rng.standard_normal((c, 1, 1, 1)).astype(np.float32), "b": (rng.standard_normal(c) * 0.1).astype(np.float32)}]
    params[1]["w"][0, 0, 1, 1] = 0.75
    net = B.Net(G.net_descs([workloads.bottleneck(1, c, False)], c, folded=True))
    x = torch.rand((1, c, side, side), device="cuda")
    y = torch.full((1, c, side, side), float("nan"), device="cuda")
    ws = torch.empty(max(net.workspace_bytes(B.desc(x)), 256), dtype=torch.uint8, device="cuda")
    net.fwd(x, [gpu(p[k]) for p in params for k in ("w", "b")], y, ws)
    torch.cuda.synchronize()
    m = torch.zeros((side, side), device="cuda", dtype=torch.float64)
    for i in range(c):
        m += x[0, i].double() * float(params[0]["w"][0, i, 0, 0])
    m = ((m + float(params[0]["b"][0])).clamp(min=0) * 0.75 + float(params[1]["b"][0])).clamp(min=0)
    for i in range(c):
        ref = (m * float(params[2]["w"][i, 0, 0, 0]) + float(params[2]["b"][i]) + x[0, i].double()).clamp(min=0)
        assert float((y[0, i].double() - ref).abs().max()) < 2e-5       # some 15 roundings of values below 10
