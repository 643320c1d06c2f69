"""GPU parity of the bf16 channels-last convolution at the sizes where the streaming kernel hands over to the
other kernels: more than 2^24 output pixels in one call, and an input of 2 GiB or more (64-bit indexing).
The input is a seeded block repeated down the image (row h holds block row h % rows), so that the host never
holds the whole tensor; the oracle computes sampled output pixels one by one from their input windows."""
import numpy as np
import pytest

import oracle
import workloads
from paper_1708_04728_amd import binding as B
from util import TOL_BF16, gpu, close, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _window(block, H, W, p, q, R, S, pad):
    """Input window of output pixel (p, q) at stride 1 as a (1, C, R, S) array, zeros outside the image."""
    C, rows, _ = block.shape
    out = np.zeros((1, C, R, S), dtype=np.float32)
    for r in range(R):
        for s in range(S):
            ih, iw = p + r - pad, q + s - pad
            if 0 <= ih < H and 0 <= iw < W:
                out[0, :, r, s] = block[:, ih % rows, iw]
    return out


def _run(C, H, W, K, R, pad, rows, seed, marks):
    rng = np.random.default_rng(seed)
    block = workloads.round_to_bf16(rng.standard_normal((C, rows, W)).astype(np.float32))
    w = workloads.round_to_bf16(rng.standard_normal((K, C, R, R)).astype(np.float32) * np.float32(np.sqrt(2.0 / (C * R * R))))
    b = (rng.standard_normal((K,)) * 0.1).astype(np.float32)
    assert H % rows == 0
    xb = torch.from_numpy(np.ascontiguousarray(np.transpose(block, (1, 2, 0)))).to(torch.bfloat16).cuda()      # (rows, W, C)
    x = B.NHWC(xb.repeat(H // rows, 1, 1).reshape(1, H, W, C))
    del xb
    y = B.NHWC(torch.empty((1, H, W, K), dtype=torch.bfloat16, device="cuda"))
    wg = B.pack_filters(gpu(w, "bf16")) if B.can_pack(C, "bf16") else gpu(w, "bf16")
    cd = B.conv_desc(K, C, R, R, 1, pad, True, B.DR_KRSC if B.can_pack(C, "bf16") else B.DR_KCRS)
    B.conv2d_fwd(x, cd, wg, gpu(b), y)
    torch.cuda.synchronize()
    pix = {0, W - 1, (H - 1) * W, H * W - 1, H * W // 2}
    for m in marks:
        pix.update(n for n in (m - 1, m, m + 1) if 0 <= n < H * W)
    pix.update(int(v) for v in rng.integers(0, H * W, 300))
    pix = sorted(pix)
    idx = torch.tensor(pix, dtype=torch.long, device="cuda")
    got = y.t.reshape(H * W, K)[idx].float().cpu().numpy().astype(np.float64)
    ref = np.stack([oracle.conv2d(_window(block, H, W, n // W, n % W, R, R, pad), w, b, 1, 0, True)[0, :, 0, 0] for n in pix])
    assert close(got, ref, TOL_BF16)


def test_conv_bf16_more_than_2_to_24_output_pixels():
    # 4200 x 4200 = 17.6 M output pixels in one call (the streaming kernel indexes at most 2^24)
    _run(C=8, H=4200, W=4200, K=16, R=3, pad=1, rows=600, seed=21, marks=[1 << 24])


def test_conv_bf16_input_of_more_than_2_gib():
    # 11600 x 11600 x 8 bf16 = 2.15 GB: byte offsets beyond 32 bits, in the input and in the output
    H = W = 11600
    _run(C=8, H=H, W=W, K=8, R=3, pad=1, rows=400, seed=22, marks=[(1 << 31) // 16, (1 << 32) // 16 if (1 << 32) // 16 < H * W else H * W - 2])


@pytest.mark.parametrize("C,H,W,K,pad,stride", [
    (512, 1, 139811, 64, 15, (16, 3)),        # wide tiles: the one tap inside the map lies 2^31 bytes and more behind every window's first pixel
    (512, 1, 139811, 60, 15, (16, 3)),        # the streaming kernel
    (8, 1, 9_000_000, 32, 15, (16, 1000)),    # the kernel for small layers
    (64, 3, 1_200_000, 64, 13, (4, 200)),     # three rows: taps on both sides of 2^31
    (64, 3, 1_200_000, 32, 13, (4, 200)),
])
def test_filter_rows_2_gib_behind_the_window(C, H, W, K, pad, stride):
    """16 x 1 filters on a few very long rows: with the padding above the map a window begins before the tensor, and rows of the filter that are
    inside the map lie 2 GiB or more behind its first pixel."""
    gen = torch.Generator(device="cuda").manual_seed(K)
    x = torch.randn((1, H, W, C), device="cuda", generator=gen).to(torch.bfloat16)
    w = (torch.randn((K, C, 16, 1), device="cuda", generator=gen) * (1.0 / (C * H)) ** 0.5).to(torch.bfloat16)
    b = torch.randn(K, device="cuda", generator=gen) * 0.1
    P, Q = (H + 2 * pad - 16) // stride[0] + 1, (W - 1) // stride[1] + 1
    assert (pad + H - 1) * W * C * 2 >= 1 << 31
    y = torch.full((1, P, Q, K), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.conv2d_fwd(B.NHWC(x), B.conv_desc(K, C, 16, 1, stride, (pad, 0), False, B.DR_KRSC), B.pack_filters(w), b, B.NHWC(y))
    torch.cuda.synchronize()
    ref = b.double().expand(P, Q, K).clone()
    for p in range(P):
        for r in range(16):
            if 0 <= p * stride[0] - pad + r < H:
                ref[p] += x[0, p * stride[0] - pad + r, ::stride[1]].double() @ w[:, :, r, 0].double().t()
    # one rounding of an fp32 sum: within one unit of the last place of the rounded exact result
    assert close(y[0].double().cpu().numpy(), ref.to(torch.bfloat16).double().cpu().numpy(), 2.0 ** -7)


def test_filter_taller_than_a_wide_flat_map():
    """31 x 1 on one row of 9 million pixels, padded by 15: the one tap inside the map lies 15 rows, 1.35e8 elements, behind the window's first,
    which is more than a one-word entry of the fp32 gather table holds."""
    W = 9_000_001
    gen = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn((1, 1, 1, W), device="cuda", generator=gen)
    w = torch.randn((1, 1, 31, 1), device="cuda", generator=gen)
    b = torch.tensor([0.25], device="cuda")
    y = torch.full((1, 1, 1, W), float("nan"), device="cuda")
    B.conv2d_fwd(x, B.conv_desc(1, 1, 31, 1, 1, (15, 0)), w, b, y)
    torch.cuda.synchronize()
    # one product and one sum per output: exact up to the rounding of each
    ref = x.double() * w[0, 0, 15, 0].double() + 0.25
    assert float((y.double() - ref).abs().max()) <= 2.0 ** -22 * float(ref.abs().max())
