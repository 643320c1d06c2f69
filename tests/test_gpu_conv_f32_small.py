"""GPU parity of the small-layer fp32 convolution kernel (NCHW; the contraction of a 32 x 32 tile shared by the waves of a
workgroup) against the fp64 oracle where it can go wrong: fewer slices than waves, ragged filters and pixels, every border and
stride, both numbers of waves, the largest layer it takes and the first it does not; and a module whose branches share launches."""
import numpy as np
import pytest

import oracle
import workloads
from paper_1708_04728_amd import binding as B
from util import TOL_F32, case_seed, close, gpu, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("case", [
    # N, C, H, W, K, R, S, stride, pad, packed
    (1, 16, 3, 5, 8, 1, 1, 1, 0, False),         # one slice for eight waves
    (1, 16, 9, 7, 33, 3, 3, 1, 1, True),         # nine slices, a second filter block of one filter
    (2, 48, 13, 10, 100, 5, 5, 2, 2, True),      # stride 2, 75 slices, ragged pixels
    (3, 32, 8, 8, 64, 3, 1, 1, 0, True),         # unequal filter sides, no padding
    (1, 144, 6, 11, 40, 1, 1, 2, 0, False),      # strided 1x1 in KCRS order
    (4, 32, 32, 32, 40, 1, 1, 1, 0, True),       # 1x1 at the largest pixel count
    (2, 16, 64, 64, 64, 3, 3, 1, 1, True),       # 512 tiles: the most with eight waves
    (2, 16, 64, 66, 64, 3, 3, 1, 1, True),       # four waves
    (1, 16, 128, 176, 40, 3, 3, 1, 1, True),     # 1408 tiles, the largest layer
    (1, 16, 128, 177, 40, 3, 3, 1, 1, True),     # one more pixel tile column than that: the 64 x 64 tiles
    (1, 272, 4, 4, 24, 3, 3, 1, 1, True),        # few tiles, long contraction: cut over workgroups when scratch is given
])
def test_small_layer(case):
    N, C, H, W, K, R, S, stride, pad, packed = case
    rng = np.random.default_rng(case_seed(case))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32)
    xg, wg = gpu(x), gpu(w)
    if packed:
        wg = B.pack_filters(wg)
    for bias, relu in ((True, True), (False, False)):
        b = (rng.standard_normal(K) * 0.1).astype(np.float32) if bias else None
        ref = oracle.conv2d(x, w, b, stride, pad, relu)
        cd = B.conv_desc(K, C, R, S, stride, pad, relu, B.DR_KRSC if packed else B.DR_KCRS)
        y = torch.full(ref.shape, float("nan"), device="cuda")
        need = B.conv2d_workspace_bytes(xg, cd)
        for ws in (None, torch.empty(need, dtype=torch.uint8, device="cuda")) if need else (None,):
            if ws is None:
                B.conv2d_fwd(xg, cd, wg, None if b is None else gpu(b), y)
            else:
                B.conv2d_fwd_ws(xg, cd, wg, None if b is None else gpu(b), y, ws)
            torch.cuda.synchronize()
            assert close(host(y), ref, TOL_F32)


def test_filters_on_any_word():
    """Filters that start 4 bytes behind a 16-byte boundary (a slice of a parameter buffer): not the small-layer kernel's."""
    rng = np.random.default_rng(5)
    x = rng.standard_normal((1, 32, 14, 14)).astype(np.float32)
    w = (rng.standard_normal((40, 32, 3, 3)) * np.sqrt(2.0 / (32 * 9))).astype(np.float32)
    packed = B.pack_filters(gpu(w))
    room = torch.empty(packed.numel() + 1, device="cuda")
    shifted = room[1:].view(packed.shape)
    shifted.copy_(packed)
    assert shifted.data_ptr() % 16 == 4
    y = torch.full((1, 40, 14, 14), float("nan"), device="cuda")
    B.conv2d_fwd(gpu(x), B.conv_desc(40, 32, 3, 3, 1, 1, False, B.DR_KRSC), shifted, None, y)
    torch.cuda.synchronize()
    assert close(host(y), oracle.conv2d(x, w, None, 1, 1, False), TOL_F32)


def runs_small(n, c, hw, k, r, stride, scratch):
    """Whether the small-layer kernel takes the layer, by its bits: filters 4 bytes behind a 16-byte boundary are not its, so the same
    layer run with those gives the other kernel's sums."""
    rng = np.random.default_rng(k + hw)
    x = gpu(rng.standard_normal((n, c, hw, hw)).astype(np.float32))
    w = B.pack_filters(gpu((rng.standard_normal((k, c, r, r)) * np.sqrt(2.0 / (c * r * r))).astype(np.float32)))
    room = torch.empty(w.numel() + 1, device="cuda")
    shifted = room[1:].view(w.shape)
    shifted.copy_(w)
    cd = B.conv_desc(k, c, r, r, stride, r // 2, False, B.DR_KRSC)
    side = (hw + 2 * (r // 2) - r) // stride + 1
    out = []
    for f in (w, shifted):
        y = torch.full((n, k, side, side), float("nan"), device="cuda")
        need = B.conv2d_workspace_bytes(x, cd) if scratch else 0
        if need:
            B.conv2d_fwd_ws(x, cd, f, None, y, torch.empty(need, dtype=torch.uint8, device="cuda"))
        else:
            B.conv2d_fwd(x, cd, f, None, y)
        out.append(y)
    torch.cuda.synchronize()
    assert close(host(out[0]), host(out[1]), TOL_F32)
    return not torch.equal(out[0], out[1])


@pytest.mark.parametrize("n,c,hw,k,small", [
    (20, 192, 14, 352, True),        # 123 x 11 tiles
    (20, 192, 14, 384, False),       # 123 x 12: more than 5.5 per compute unit
    (83, 64, 7, 2048, False),        # 4067 pixels
    (84, 192, 7, 32, False),         # 4116 pixels
])
def test_1x1_layers_by_tiles(n, c, hw, k, small):
    assert runs_small(n, c, hw, k, 1, 1, False) == small


@pytest.mark.parametrize("n,c,hw,k,r,stride,small", [
    (1, 2048, 7, 64, 1, 1, False),       # 4 tiles, 128 slices: cut
    (1, 1024, 7, 64, 1, 1, True),        # 64 slices
    (3, 512, 14, 128, 3, 1, False),      # 76 tiles, 288 slices
    (3, 192, 14, 128, 3, 1, True),       # 108 slices
    (4, 352, 14, 256, 3, 1, True),       # 200 tiles: more than three quarters of a round
    (6, 352, 14, 256, 3, 1, False),      # 296 tiles: a second round, mostly idle
    (8, 352, 14, 320, 3, 1, True),       # 490
    (4, 192, 14, 160, 5, 1, True),       # 125 tiles, 300 slices
    (6, 352, 28, 192, 3, 2, False),      # 222 tiles, strided, 198 slices, 6.6 MB
    (6, 192, 28, 192, 3, 2, True),       # 108 slices
    (4, 192, 28, 256, 5, 2, True),       # 300 slices, 2.4 MB
])
def test_long_contractions_are_cut_where_there_is_scratch(n, c, hw, k, r, stride, small):
    assert runs_small(n, c, hw, k, r, stride, True) == small
    assert runs_small(n, c, hw, k, r, stride, False)


@pytest.mark.parametrize("c,k,images", [
    (64, 64, (90, 334, 335)),            # tiles of 64 x 64: 276, 1023 (32 channels deep), 1026 (16 deep)
    (288, 2048, (16, 21, 24)),           # 1568 (16 deep), 2080 (32), 2368 (16)
    (96, 96, (55, 56)),                  # 255 and 258 tiles of 32 x 128
])
def test_1x1_layers_at_any_slice_depth(c, k, images):
    """Both depths of a slice, on either side of the rule's lines: the images of a batch have the bits they have in the largest one."""
    rng = np.random.default_rng(c + k)
    n = max(images)
    x = rng.standard_normal((n, c, 14, 14)).astype(np.float32)
    w = (rng.standard_normal((k, c, 1, 1)) * np.sqrt(2.0 / c)).astype(np.float32)
    xg, wg = gpu(x), B.pack_filters(gpu(w))
    out = {}
    for m in images:
        out[m] = torch.full((m, k, 14, 14), float("nan"), device="cuda")
        B.conv2d_fwd(xg[:m], B.conv_desc(k, c, 1, 1, 1, 0, False, B.DR_KRSC), wg, None, out[m])
    torch.cuda.synchronize()
    assert close(host(out[n][-3:]), oracle.conv2d(x[-3:], w, None, 1, 0, False), TOL_F32)
    for m in images:
        assert torch.equal(out[m], out[n][:m])


@pytest.mark.parametrize("form", ["original", "slim"])
def test_module_whose_branches_share_launches(form):
    """A module on two ragged maps in every mode, packed filters, channel ranges of the output, stacked first steps."""
    from test_gpu_blocks import _run_stacked, run_inception
    layer = (workloads.inception_original if form == "original" else workloads.inception_slim)("4e")
    rng = np.random.default_rng(23)
    x = np.abs(rng.standard_normal((2, 528, 13, 15))).astype(np.float32)
    params = []
    workloads._walk(rng, [layer], 528, "f32", params)
    ref = oracle.forward([layer], params, x)
    base = B.DR_FUSE_RELU | B.DR_FUSE_CONCAT
    for mode in (0, B.DR_CONCURRENT_BRANCHES, B.DR_FUSE_RELU, base):
        assert close(run_inception(layer, params, x, mode, pack=True), ref, TOL_F32, "mode %d" % mode)
    for mode in (base | B.DR_FUSE_STACK, B.DR_FUSE_RELU | B.DR_FUSE_STACK):
        assert close(_run_stacked(layer, params, x, mode, True), ref, TOL_F32, "mode %d" % mode)
