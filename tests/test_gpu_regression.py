"""GPU parity of the pieces that learn a slim layer (Sec. 3.1, Lemma 1) against the fp64 oracle: the loss and its
gradient, the gradient of a convolution's parameters, the descent step, and a short run of the whole loop."""
import numpy as np
import pytest

import oracle
import workloads
from paper_1708_04728_amd import binding as B
from util import TOL_F32, gpu, host, close, note, rel_err, rms_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _ws(nbytes):
    return torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")


def test_regression_loss_and_gradient():
    rng = np.random.default_rng(1)
    for shape in ((2, 5, 7, 9), (1, 3, 1, 1), (3, 192, 28, 28), (1, 1, 1, 300001)):
        f = np.maximum(rng.standard_normal(shape), 0).astype(np.float32)          # about half the entries are zero
        y = np.abs(rng.standard_normal(shape)).astype(np.float32)
        loss_ref, dz_ref = oracle.regression_loss_grad(f, y)
        fg, yg = gpu(f), gpu(y)
        dz = torch.empty_like(fg)
        loss = torch.zeros(1, device="cuda")
        B.regression_loss_grad(fg, yg, dz, loss, _ws(B.regression_loss_workspace_bytes()))
        torch.cuda.synchronize()
        assert float(loss.item()) == pytest.approx(loss_ref, rel=1e-5)
        # each entry is one subtraction and one doubling: exact in fp32 up to the subtraction's rounding
        np.testing.assert_allclose(host(dz), dz_ref, rtol=1e-6, atol=1e-6)
        assert ((host(dz) == 0) == (dz_ref == 0)).all()


# N, C, H, W, K, R, S, stride, pad
WGRAD_CASES = [
    (2, 3, 9, 8, 5, 3, 3, 1, 1),          # one tile, ragged everywhere
    (3, 64, 28, 28, 192, 3, 3, 2, 1),     # the slim layer of the conv2 block: 3 x 9 tiles, stride 2
    (2, 16, 14, 14, 70, 5, 5, 1, 2),      # 5x5, ragged filter block, 400 (c, r, s) columns
    (5, 8, 10, 6, 64, 1, 1, 1, 0),        # 1x1
    (1, 4, 31, 29, 9, 7, 7, 4, 3),        # one image (no partial sums), 7x7 stride 4
    (40, 2, 6, 6, 3, 3, 2, (2, 1), (1, 0)),  # many images: several per workgroup, non-square filter and stride
    (3, 8, 13, 9, 65, 3, 3, 1, 1),        # tiles of eight taps by 8 channels, one tap in the second
    (2, 9, 12, 11, 20, 4, 4, 1, 1),       # tiles of sixteen taps by 4 channels, one channel in the third
    (2, 3, 43, 39, 33, 11, 11, 4, 0),     # a layer on the image: eight tiles of sixteen taps, nine taps in the last
    (10, 8, 15, 18, 32, 3, 3, 4, 1),      # ten images of one slice each: a range per image
    (20, 3, 12, 8, 40, 3, 3, 4, 1),       # twenty: sixteen ranges, some of two slices
    (2, 72, 9, 11, 72, 3, 3, 1, 1),       # filters and channels in eights, one of them in the second tile
    (3, 24, 10, 13, 40, 3, 3, 2, 1),      # ... on tiles of two taps by 32 channels, a tap in the fifth that does not exist
    (2, 16, 7, 9, 8, 5, 5, 1, 2),         # ... four taps by 16
    (2, 24, 8, 8, 65, 3, 3, 1, 1),        # channels in eights, filters not
]


@pytest.mark.parametrize("case", WGRAD_CASES)
def test_conv_parameter_gradients(case):
    N, C, H, W, K, R, S, stride, pad = case
    rng = np.random.default_rng(7 + N * C)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    sh, sw = (stride, stride) if np.isscalar(stride) else stride
    ph, pw = (pad, pad) if np.isscalar(pad) else pad
    P, Q = oracle.conv_out_size(H, R, sh, ph), oracle.conv_out_size(W, S, sw, pw)
    dz = (rng.standard_normal((N, K, P, Q)) * (rng.random((N, K, P, Q)) < 0.6)).astype(np.float32)   # ReLU zeros
    dw_ref, db_ref = oracle.conv2d_bwd_params(x, dz, R, S, stride, pad)
    xg, dzg = gpu(x), gpu(dz)
    cd = B.conv_desc(K, C, R, S, stride, pad, True, B.DR_KCRS)
    dw = torch.full((K, C, R, S), float("nan"), device="cuda")
    db = torch.full((K,), float("nan"), device="cuda")
    for rep in range(2):       # the same workspace twice: nothing may depend on what it held
        ws = _ws(B.conv2d_bwd_params_workspace_bytes(xg, cd))
        ws.fill_(255)
        B.conv2d_bwd_params(xg, cd, dzg, dw, db, ws)
        torch.cuda.synchronize()
        assert close(host(dw), dw_ref, TOL_F32)
        assert close(host(db), db_ref, TOL_F32)
    first = host(dw).copy()
    B.conv2d_bwd_params(xg, cd, dzg, dw, db, ws)
    torch.cuda.synchronize()
    assert np.array_equal(host(dw), first)      # fixed summation order: bit-identical from run to run


def parameter_gradients(x, dz, K, R, S, stride, pad):
    cd = B.conv_desc(K, x.shape[1], R, S, stride, pad, True, B.DR_KCRS)
    dw, db = torch.full((K, x.shape[1], R, S), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
    B.conv2d_bwd_params(x, cd, dz, dw, db, _ws(B.conv2d_bwd_params_workspace_bytes(x, cd)))
    torch.cuda.synchronize()
    return host(dw), host(db)


# Tiles of one, two and three blocks of 64 filters; ranges long enough for products of bf16 pieces
LONG_CASES = [
    (40, 4, 44, 44, 8, 11, 11, 1, 0),         # one block of filters, ranges of 15 slices
    (40, 8, 41, 37, 64, 5, 5, 1, 2),          # ... 41 x 37 pixels: not in fours, nor in slices
    (12, 20, 33, 35, 100, 3, 3, 1, 1),        # two blocks, filters and channels that fill neither tile
    (20, 32, 53, 50, 128, 3, 3, 2, 1),        # ... channels in eights
    (10, 64, 54, 54, 192, 3, 3, 2, 1),        # three blocks, 27 x 27 pixels
    (24, 16, 30, 29, 385, 3, 3, (1, 2), 1),   # seven blocks, one at a time; one filter in the last
]


@pytest.mark.parametrize("case", LONG_CASES)
def test_conv_parameter_gradients_of_long_ranges(case):
    """Also with pixels that pieces cannot hold: infinite, near the largest and the smallest values that there are."""
    N, C, H, W, K, R, S, stride, pad = case
    rng = np.random.default_rng(11 + N * C)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    sh, sw = (stride, stride) if np.isscalar(stride) else stride
    P, Q = oracle.conv_out_size(H, R, sh, pad), oracle.conv_out_size(W, S, sw, pad)
    dz = (rng.standard_normal((N, K, P, Q)) * (rng.random((N, K, P, Q)) < 0.6)).astype(np.float32)
    dw_ref, db_ref = oracle.conv2d_bwd_params(x, dz, R, S, stride, pad)
    xg = gpu(x)
    plain, db = parameter_gradients(xg, gpu(dz), K, R, S, stride, pad)
    assert close(plain, dw_ref, TOL_F32) and close(db, db_ref, TOL_F32)
    # gradients of one filter, scaled: exact to the same relative error (a power of two)
    for scale in (2.0 ** -118, 2.0 ** 118):
        scaled = dz.copy()
        scaled[:, K // 2] *= np.float32(scale)
        got, _ = parameter_gradients(xg, gpu(scaled), K, R, S, stride, pad)
        assert close(got[K // 2] * np.float32(1 / scale), dw_ref[K // 2], TOL_F32, "2^%d" % np.log2(scale))
        assert close(np.delete(got, K // 2, 0), np.delete(dw_ref, K // 2, 0), TOL_F32)
    # one infinite gradient: weights of its filter, and of no other
    wild = dz.copy()
    wild[N // 2, K // 2, P // 2, Q // 2] = np.inf
    got, _ = parameter_gradients(xg, gpu(wild), K, R, S, stride, pad)
    assert not np.isfinite(got[K // 2]).all() and np.isfinite(np.delete(got, K // 2, 0)).all()
    assert close(np.delete(got, K // 2, 0), np.delete(dw_ref, K // 2, 0), TOL_F32)


@pytest.mark.parametrize("scale", (-105, -118, -140))
@pytest.mark.parametrize("r", (1, 3))
def test_conv_parameter_gradients_of_small_operands(r, scale):
    """Of every eight pixels one is about 1 where the other operand is 0, the rest about 2^scale (2^-140: subnormal): the sums consist of those alone."""
    N, C, P, K = (8, 512, 32, 384) if r == 1 else (16, 64, 32, 384)
    rng = np.random.default_rng(r)
    x = rng.standard_normal((N, C, P * r, P * r)).astype(np.float32)
    dz = rng.standard_normal((N, K, P, P)).astype(np.float32)
    few = np.zeros((P, P), bool)
    few[:, ::8] = True                                    # 32 pixels a row: one of every eight
    few_x = few.repeat(r, 0).repeat(r, 1)
    for small_x in (True, False):
        a, b = x.copy(), dz.copy()
        t, u, at, there = (a, b, few_x, few) if small_x else (b, a, few, few_x)
        t[..., ~at] *= np.float32(2.0 ** scale)
        u *= np.float32(2.0 ** 30)
        u[..., there] = 0
        # (taps do not overlap: a product of matrices)
        cols = a.astype(np.float64).reshape(N, C, P, r, P, r).transpose(0, 2, 4, 1, 3, 5).reshape(N * P * P, C * r * r)
        ref = (b.astype(np.float64).transpose(1, 0, 2, 3).reshape(K, N * P * P) @ cols).reshape(K, C, r, r)
        got, _ = parameter_gradients(gpu(a), gpu(b), K, r, r, r, 0)
        # N P P / 16 sums of 16 products with 2^-24 of rounding each
        assert note("rms", rms_err(got, ref), 4 * 2.0 ** -24 * np.sqrt(N * P * P / 16) + 2.0 ** -24)


def test_sgd_step_bit_exact():
    rng = np.random.default_rng(3)
    w = rng.standard_normal(100003).astype(np.float32)
    dw = rng.standard_normal(100003).astype(np.float32)
    lr = np.float32(0.0137)
    wg = gpu(w)
    B.sgd_step(wg, gpu(dw), float(lr))
    torch.cuda.synchronize()
    assert np.array_equal(host(wg).astype(np.float32), w - lr * dw)


def test_slim_layer_regression_follows_the_oracle():
    """Config 1's slim layer (3x3, stride 2, ReLU) learned from the output of the original block on a few seeded
    images: twelve descent steps on the GPU and in the oracle from the same start; the losses agree step by
    step and fall."""
    layers = workloads.CONFIGS[1]["original"]
    params = workloads.make_params(1, "original")
    x = workloads.make_input(1, 1)
    x = np.concatenate([x, x[:, ::-1].copy(), x[:, :, ::-1].copy()], axis=0)[:, :16, :20, :20].copy()    # 3 small images
    p16 = [{"w": params[0]["w"][:24, :16].copy(), "b": params[0]["b"][:24].copy()}]
    y = oracle.forward(layers, p16, x)                      # conv - ReLU - LRN - pool
    slim_w = workloads.make_params(1, "slim")[0]
    w0, b0 = slim_w["w"][:24, :16].astype(np.float32).copy(), slim_w["b"][:24].astype(np.float32).copy()
    lr = 5e-5
    w_ref, b_ref, ref_losses = w0.astype(np.float64), b0.astype(np.float64), []
    for _ in range(12):
        loss, w_ref, b_ref = oracle.regression_step(x, w_ref, b_ref, y, 2, 1, lr)
        ref_losses.append(loss)
    xg, yg, wg, bg = gpu(x), gpu(y), gpu(w0), gpu(b0)
    cd = B.conv_desc(24, 16, 3, 3, 1, 1, False, B.DR_KCRS)
    f = torch.empty(y.shape, device="cuda")
    dw, db, loss = torch.empty_like(wg), torch.empty_like(bg), torch.zeros(1, device="cuda")
    ws = _ws(max(B.conv2d_bwd_params_workspace_bytes(xg, B.conv_desc(24, 16, 3, 3, 2, 1, True, B.DR_KCRS)), B.regression_loss_workspace_bytes()))
    cd2 = B.conv_desc(24, 16, 3, 3, 2, 1, True, B.DR_KCRS)
    got = []
    for _ in range(12):
        B.slim_conv_fwd(xg, cd, 2, wg, bg, f)              # stride 1 x pool stride 2, ReLU forced on
        B.regression_loss_grad(f, yg, f, loss, ws)         # dz overwrites f
        got.append(float(loss.item()))
        B.conv2d_bwd_params(xg, cd2, f, dw, db, ws)
        B.sgd_step(wg, dw, lr)
        B.sgd_step(bg, db, lr)
    torch.cuda.synchronize()
    assert y.shape == (3, 24, 10, 10)
    np.testing.assert_allclose(got, ref_losses, rtol=2e-4)
    assert all(b_ < a_ for a_, b_ in zip(got, got[1:]))
    assert close(host(wg), w_ref, 10 * TOL_F32)


def test_degenerate_inputs():
    """No images / no pixels: the gradients are zero (and the kernels dereference nothing); an empty tensor has zero
    loss; unsupported layouts are refused before anything is launched."""
    cd = B.conv_desc(5, 3, 3, 3, 1, 1, True, B.DR_KCRS)
    x = torch.empty((0, 3, 8, 8), device="cuda")
    dz = torch.empty((0, 5, 8, 8), device="cuda")
    dw = torch.full((5, 3, 3, 3), float("nan"), device="cuda")
    db = torch.full((5,), float("nan"), device="cuda")
    B.conv2d_bwd_params(x, cd, dz, dw, db, _ws(B.conv2d_bwd_params_workspace_bytes(x, cd)))
    torch.cuda.synchronize()
    assert not host(dw).any() and not host(db).any()
    f = torch.empty((0, 4, 2, 2), device="cuda")
    loss = torch.full((1,), 7.0, device="cuda")
    B.regression_loss_grad(f, f, f, loss, _ws(B.regression_loss_workspace_bytes()))
    torch.cuda.synchronize()
    assert float(loss.item()) == 0.0
    xb = torch.zeros((1, 8, 4, 4), device="cuda", dtype=torch.bfloat16)
    with pytest.raises(B.DeepRebirthError):
        B.conv2d_bwd_params_workspace_bytes(xb, B.conv_desc(4, 8, 1, 1, 1, 0, True, B.DR_KCRS))
    x1 = torch.zeros((1, 16, 4, 4), device="cuda")
    with pytest.raises(B.DeepRebirthError):                      # KRSC filters
        B.conv2d_bwd_params_workspace_bytes(x1, B.conv_desc(4, 16, 1, 1, 1, 0, True, B.DR_KRSC))
    with pytest.raises(B.DeepRebirthError):                      # dz of the wrong shape
        B.conv2d_bwd_params(x1, B.conv_desc(4, 16, 1, 1, 1, 0, True, B.DR_KCRS), torch.zeros((1, 4, 3, 3), device="cuda"),
                            torch.zeros((4, 16, 1, 1), device="cuda"), None, _ws(256))
