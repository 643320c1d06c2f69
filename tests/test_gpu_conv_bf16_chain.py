"""GPU parity of the kernel that runs the end of a folded bottleneck (expansion, shortcut, the next block's first layer) in one pass:
the same bits as the layers run one after the other (which is what a kernel trace makes the library do), and the oracle's
result, at the edges of its 32-pixel blocks, its 16-channel steps and its widths."""
import numpy as np
import pytest

import oracle
import workloads
from paper_1708_04728_amd import binding as B, graph as G
from test_gpu_bf16_nets import folded_params
from util import TOL_BF16, case_seed, close

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def bn(k, rng):
    return {"gamma": rng.uniform(0.5, 1.5, k).astype(np.float32), "beta": (rng.standard_normal(k) * 0.1).astype(np.float32),
            "mean": (rng.standard_normal(k) * 0.1).astype(np.float32), "var": rng.uniform(0.5, 1.5, k).astype(np.float32)}


def stage(rng, c, blocks):
    """Bottlenecks (mid, out) on c channels and their folded parameters; the shortcut is projected where the widths differ or for the first."""
    layers, params = [], []
    for i, (mid, out) in enumerate(blocks):
        project = i == 0 or c != out
        layers.append(workloads.bottleneck(mid, out, project))
        for k, r, ci in ((mid, 1, c), (mid, 3, mid), (out, 1, mid)) + (((out, 1, c),) if project else ()):
            w = rng.standard_normal((k, ci, r, r)).astype(np.float32) * np.float32(np.sqrt(2.0 / (ci * r * r)))
            params += [{"w": w, "b": (rng.standard_normal(k) * 0.1).astype(np.float32)}, bn(k, rng)]
        c = out
    return layers, folded_params(params)


@pytest.mark.parametrize("case", [
    # N, C, H, W, ((mid, out), ...)
    (1, 8, 1, 1, ((8, 8),)),                                   # one pixel, one channel group
    (1, 64, 4, 8, ((64, 256), (64, 256))),                     # one whole block of pixels
    (1, 64, 3, 11, ((64, 256), (64, 256), (64, 256))),         # 33 pixels
    (2, 24, 5, 3, ((40, 72), (40, 72))),                       # ragged steps, 30 pixels
    (3, 56, 17, 19, ((48, 200), (32, 200), (32, 248))),        # a narrower block behind, then a projected one on too many channels
    (1, 64, 9, 9, ((32, 128), (64, 128), (64, 264))),          # a wider block behind (not joined), an output too wide for the kernel
    (9, 64, 61, 59, ((64, 256), (64, 256))),                   # 1013 blocks: the most that move as the lanes hold them
    (11, 64, 61, 59, ((64, 256), (64, 256), (64, 256))),       # 1238 blocks, the last one not whole: by lines, through LDS
    (10, 24, 55, 61, ((40, 72), (24, 72), (24, 200), (8, 200))),        # ... with ragged channel groups
    (23, 56, 61, 59, ((64, 248), (64, 248))),                  # ... several rounds of every wave
    (5, 64, 7, 63, ((64, 256), (64, 256), (64, 256))),         # the widest map whose 3x3 layers are joined too
    (2, 64, 33, 64, ((64, 256), (64, 256))),                   # ... and the first one on which they are not
    (1, 64, 300, 1, ((64, 200), (64, 200))),                   # rows of one pixel, ragged output groups
    (3, 64, 1, 57, ((64, 72), (64, 72), (32, 72), (32, 72))),  # images of one row; narrower blocks behind
    (19, 64, 30, 58, ((64, 256), (64, 256), (32, 256))),       # 259 tiles of 128 pixels: a second round for three workgroups
])
def test_chain(case):
    n, c, h, w, blocks = case
    rng = np.random.default_rng(case_seed(case))
    layers, params = stage(rng, c, blocks)
    x = workloads.round_to_bf16(np.abs(rng.standard_normal((n, c, h, w))).astype(np.float32))
    xg = G.to_device(x, "bf16", nhwc=True)
    net = B.Net(G.net_descs(layers, c, folded=True, pack="bf16"))
    flat = G.flat_params(params, "bf16", pack=True)
    ws = torch.empty(max(net.workspace_bytes(B.desc(xg)), 256), dtype=torch.uint8, device="cuda")
    out = []
    for traced in (False, True, False):
        y = G.empty_like_desc(net.output_desc(B.desc(xg)))
        y.t.fill_(float("nan"))
        ws.fill_(255)                                          # NaN where nothing has been written
        if traced:
            B.trace_begin()
        net.fwd(xg, flat, y, ws)
        torch.cuda.synchronize()
        if traced:
            B.trace_end()
        out.append(G.to_host(y))
    assert np.isfinite(out[0]).all()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    if n * h * w < 4000:
        ref = oracle.forward(layers, params, x, mirror_bf16=True, fold="given")
        # two implementations that round every stored tensor to bf16: 2e-2 per rounding in quadrature, 3 per block
        assert close(out[0], ref, TOL_BF16 * (3 * len(blocks)) ** 0.5, "oracle with bf16 storage")


@pytest.mark.parametrize("c,blocks,joined", [
    (64, ((64, 256),), True),
    (24, ((40, 72),), True),
    (64, ((64, 256), (64, 256)), True),          # with the next block's first layer
    (64, ((64, 256), (72, 256)), True),          # a next block that is too wide to be joined
    (64, ((64, 264),), False),                   # more outputs than the kernel holds
    (72, ((64, 256),), False),                   # a projected shortcut over more channels than it holds
    (64, ((72, 256),), False),                   # more inner channels
])
def test_the_projected_shortcut_is_stored_only_where_the_kernel_does_not_run(c, blocks, joined):
    """Which way a block went, by the scratch memory of its projected shortcut: the kernel keeps the shortcut in registers, the layers one by one
    (also: the kernel under a trace) store it."""
    n, h, w = 2, 7, 9
    rng = np.random.default_rng(c + len(blocks))
    layers, params = stage(rng, c, blocks)
    xg = G.to_device(workloads.round_to_bf16(np.abs(rng.standard_normal((n, c, h, w))).astype(np.float32)), "bf16", nhwc=True)
    net = B.Net(G.net_descs(layers, c, folded=True, pack="bf16"))
    flat = G.flat_params(params, "bf16", pack=True)
    y = G.empty_like_desc(net.output_desc(B.desc(xg)))
    need = net.workspace_bytes(B.desc(xg))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    # the scratch of a block: the outputs of its first and second layer and of its projection, each from a multiple of 256 bytes
    up = lambda v: (v + 255) // 256 * 256
    sizes = [(up(n * h * w * m * 2), n * h * w * k * 2 if i == 0 else 0) for i, (m, k) in enumerate(blocks)]
    base = need - max(2 * mid + up(proj) for mid, proj in sizes)
    lo, hi = base + 2 * sizes[0][0], base + 2 * sizes[0][0] + sizes[0][1]
    for traced in (False, True):
        ws.fill_(255)
        if traced:
            B.trace_begin()
        net.fwd(xg, flat, y, ws)
        torch.cuda.synchronize()
        if traced:
            B.trace_end()
        # (a wider block behind uses the start of the same memory for its own layers)
        part = ws[max(lo, base + 2 * max(mid for mid, _ in sizes)):hi]
        assert part.numel() > 0
        assert bool((part == 255).all()) == (joined and not traced), (traced, joined)


@pytest.mark.parametrize("mid,w,joined", [(64, 1, True), (64, 63, True), (64, 64, False), (56, 63, False)])
def test_the_middle_layer_is_stored_only_where_the_kernel_does_not_run_it(mid, w, joined):
    """Which way the 3x3 layer of a block without a projection went, by the scratch memory of its output."""
    n, h, c = 2, 5, 256
    rng = np.random.default_rng(mid + w)
    params = []
    for k, r, ci in ((mid, 1, c), (mid, 3, mid), (c, 1, mid)):
        wt = rng.standard_normal((k, ci, r, r)).astype(np.float32) * np.float32(np.sqrt(2.0 / (ci * r * r)))
        params += [{"w": wt, "b": (rng.standard_normal(k) * 0.1).astype(np.float32)}, bn(k, rng)]
    params = folded_params(params)
    layers = [workloads.bottleneck(mid, c, False)]
    x = workloads.round_to_bf16(np.abs(rng.standard_normal((n, c, h, w))).astype(np.float32))
    xg = G.to_device(x, "bf16", nhwc=True)
    net = B.Net(G.net_descs(layers, c, folded=True, pack="bf16"))
    flat = G.flat_params(params, "bf16", pack=True)
    y = G.empty_like_desc(net.output_desc(B.desc(xg)))
    # the scratch of a block: the outputs of its first and second layer, each from a multiple of 256 bytes
    size = n * h * w * mid * 2
    step = (size + 255) // 256 * 256
    ws = torch.full((net.workspace_bytes(B.desc(xg)),), 255, dtype=torch.uint8, device="cuda")
    net.fwd(xg, flat, y, ws)
    torch.cuda.synchronize()
    base = ws.numel() - 2 * step
    assert not bool((ws[base:base + size] == 255).all())
    assert bool((ws[base + step:base + step + size] == 255).all()) == joined
    ref = oracle.forward(layers, params, x, mirror_bf16=True, fold="given")
    assert close(G.to_host(y), ref, TOL_BF16 * 3 ** 0.5, "oracle with bf16 storage")      # as above, one block
