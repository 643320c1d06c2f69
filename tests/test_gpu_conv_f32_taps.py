"""GPU parity of the fp32 kernel for first layers (filters 7, 8 or 10 to 12 taps wide, no padding, KCRS) against the fp64 oracle: every
overlap of the last group of taps, odd and even numbers of filter rows, one row, all filter block sizes (`filter_blocks` restates the
launcher's choice), ragged filters and pixels, windows that end on the tensor's last element, a channel range of a wider tensor, long contractions
on both sides of the rule."""
import numpy as np
import pytest

import oracle
from paper_1708_04728_amd import binding as B
from util import TOL_F32, case_seed, close, gpu

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def filter_blocks(case):
    """Blocks of 32 filters per workgroup, 0 = the tiled kernel."""
    N, C, H, W, K, R, S, stride = case
    tiles = -(-N * oracle.conv_out_size(H, R, stride, 0) * oracle.conv_out_size(W, S, stride, 0) // 128)
    if C * R > 64 and -(-K // 32) * tiles < 256:
        return 0
    tm = 1
    for t in (2, 3):
        if -(-K // (32 * t)) * t <= -(-K // (32 * tm)) * tm:
            tm = t
    return tm if -(-K // (32 * tm)) * tiles >= 128 else 1


@pytest.mark.parametrize("blocks,case", [
    # N, C, H, W, K, R, S, stride
    (1, (3, 3, 43, 47, 96, 11, 11, 4)),        # AlexNet's filter: 33 rows, the last without a partner
    (1, (140, 3, 35, 35, 96, 11, 11, 4)),      # 54 workgroups of 96 filters would be less than half a device
    (3, (340, 3, 35, 35, 96, 11, 11, 4)),      # 131
    (1, (30, 3, 67, 67, 100, 11, 11, 4)),      # ragged: blocks of 32, 28 filters over
    (2, (40, 3, 67, 67, 100, 11, 11, 4)),      # blocks of 64, 28 over
    (3, (75, 3, 67, 67, 70, 11, 11, 4)),       # blocks of 96, 26 over
    (2, (50, 3, 48, 50, 64, 7, 7, 2)),         # blocks of 64 with each width
    (2, (24, 2, 60, 59, 104, 5, 8, 2)),
    (2, (50, 1, 62, 63, 50, 4, 10, 2)),
    (2, (46, 2, 64, 61, 120, 3, 12, 3)),
    (3, (42, 3, 49, 48, 96, 7, 7, 2)),         # blocks of 96
    (3, (30, 2, 60, 59, 80, 5, 8, 2)),
    (3, (50, 1, 62, 63, 81, 4, 10, 2)),
    (3, (90, 2, 64, 61, 185, 3, 12, 3)),       # two, 89 filters in the second
    (1, (60, 2, 27, 39, 33, 8, 8, 2)),         # whole groups of taps; 16 rows; a block of one filter
    (1, (2, 1, 7, 7, 5, 7, 7, 1)),             # one pixel, which ends on the tensor's last element
    (1, (5, 3, 21, 30, 64, 7, 7, 2)),          # overlap of one
    (1, (4, 2, 15, 33, 40, 3, 10, 3)),         # overlap of two, window rows apart
    (1, (1, 1, 1, 300, 24, 1, 12, 1)),         # one filter row
    (1, (2, 4, 19, 25, 70, 5, 12, 1)),         # four channels
    (0, (1, 20, 15, 15, 48, 7, 7, 1)),         # 140 rows on 81 pixels: stays with the tiled kernel
    (1, (40, 20, 30, 30, 200, 7, 7, 1)),       # 140 rows, 180 x 7 workgroups
])
@pytest.mark.parametrize("relu", [False, True])
def test_conv_f32_taps(blocks, case, relu):
    assert filter_blocks(case) == blocks
    N, C, H, W, K, R, S, stride = case
    rng = np.random.default_rng(case_seed(case))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32)
    b = (rng.standard_normal(K) * 0.1).astype(np.float32) if relu else None
    ref = oracle.conv2d(x, w, b, stride, 0, relu)
    off, ctot = (3, K + 5) if case_seed(case) % 2 else (0, K)
    y = torch.full((N, ctot, ref.shape[2], ref.shape[3]), -7.0, device="cuda")
    B.conv2d_fwd(gpu(x), B.conv_desc(K, C, R, S, stride, 0, relu, B.DR_KCRS), gpu(w), None if b is None else gpu(b), y, y_c_offset=off)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    assert (got[:, :off] == -7.0).all() and (got[:, off + K:] == -7.0).all()
    assert close(got[:, off:off + K], ref, TOL_F32)


def cut_is_faster(case):
    """The library's rule for layers with scratch memory, restated."""
    N, C, H, W, K, R, S, stride = case
    ng = N * oracle.conv_out_size(H, R, stride, 0) * oracle.conv_out_size(W, S, stride, 0)
    rows32 = -(-K // 32) * 32 < -(-K // 64) * 64
    tiles = -(-K // 32) * -(-ng // 128) if rows32 else -(-K // 64) * -(-ng // 64)
    slices = -(-C * R * (-(-S // 4) * 4) // 16)
    if 2 * tiles > 256 or slices < 4:
        return False
    per = max(2, -(-slices // -(-512 // tiles)))
    splits = -(-slices // per)
    return splits > 1 and 6.4 + 0.84e-6 * splits * K * ng * 4 + 1.26 * (per - 2) + 0.071 * splits < 0.95 * (3 + 0.34 * -(-C * R // 2))


@pytest.mark.parametrize("case,cut", [
    ((2, 5, 12, 15, 1, 11, 11, 2), True),        # two outputs, 55 filter rows
    ((17, 5, 27, 25, 27, 12, 12, 4), True),
    ((7, 3, 40, 39, 6, 11, 11, 2), True),        # 33 rows: beside the line
    ((11, 5, 40, 41, 3, 7, 7, 4), True),         # 35
    ((2, 3, 66, 68, 240, 10, 10, 2), False),     # partial sums of 8 MB
    ((7, 5, 90, 92, 13, 8, 8, 4), True),
    ((7, 5, 170, 172, 13, 8, 8, 4), False),      # ... of 3 MB
    ((26, 1, 20, 23, 115, 8, 8, 4), False),      # 8 rows
    ((1, 3, 227, 227, 96, 11, 11, 4), False),    # AlexNet's first layer on one image
])
def test_cut_over_workgroups_where_that_is_faster(case, cut):
    """With scratch memory: the partial sums are written into it exactly where the rule says, and either way gives the layer."""
    assert cut_is_faster(case) == cut
    N, C, H, W, K, R, S, stride = case
    rng = np.random.default_rng(case_seed(case))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32)
    b = (rng.standard_normal(K) * 0.1).astype(np.float32)
    ref = oracle.conv2d(x, w, b, stride, 0, True)
    cd = B.conv_desc(K, C, R, S, stride, 0, True, B.DR_KCRS)
    need = B.conv2d_workspace_bytes(gpu(x), cd)
    assert need > 0
    ws = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
    y = torch.full(ref.shape, float("nan"), device="cuda")
    B.conv2d_fwd_ws(gpu(x), cd, gpu(w), gpu(b), y, ws)
    torch.cuda.synchronize()
    assert bool((ws != 0xA5).any()) == cut
    assert close(y.cpu().numpy(), ref, TOL_F32)


def test_values_beside_the_window():
    """Infinities right of a window, below it and in the other filters reach no other output."""
    x = torch.randn((2, 3, 40, 47), device="cuda")
    w = torch.randn((40, 3, 11, 11), device="cuda")
    cd = B.conv_desc(40, 3, 11, 11, 4, 0, False, B.DR_KCRS)
    y, z = torch.empty((2, 40, 8, 10), device="cuda"), torch.empty((2, 40, 8, 10), device="cuda")
    B.conv2d_fwd(x, cd, w, None, y)
    x[:, :, :, 11:15] = float("inf")              # columns 0 (0..10) has none of them, column 1 has
    w[17] = float("nan")
    B.conv2d_fwd(x, cd, w, None, z)
    torch.cuda.synchronize()
    keep = [m for m in range(40) if m != 17]
    assert torch.equal(y[:, keep, :, 0], z[:, keep, :, 0]) and torch.isnan(z[:, 17]).all() and not torch.isfinite(z[:, keep, :, 1]).any()
