"""GPU parity of the fp32 kernel for 3x3 filters that stay in KCRS order against the oracle, at the edges of its tiles (64 filters x 64 pixels, 32 x 128
where that pads the filter count less), its blocks of 8 channels and its borders; and the layers beside its rule."""
import numpy as np
import pytest

import oracle
from paper_1708_04728_amd import binding as B
from util import TOL_F32, case_seed, close, gpu, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("case", [
    # N, C, H, W, K, stride, pad
    (1, 16, 3, 3, 64, 1, 0),            # one output, two blocks of channels
    (1, 16, 1, 1, 1, 1, 1),             # one pixel, one filter: every tap but one is padding
    (2, 32, 13, 9, 64, 2, 1),           # a pixel tile that is not whole
    (1, 48, 8, 8, 130, 1, 1),           # 64 pixels, two filters in the last block
    (3, 64, 11, 17, 96, 2, 1),          # tiles of 32 x 128
    (1, 32, 16, 16, 33, 1, 2),          # ... one filter in the last block, wide padding
    (5, 16, 30, 30, 45, (2, 1), (0, 1)),
    (9, 64, 28, 28, 192, 2, 1),
    (1, 20, 9, 9, 64, 1, 1),            # 20 channels: beside the rule
])
def test_kcrs_3x3(case):
    N, C, H, W, K, stride, pad = case
    rng = np.random.default_rng(case_seed(case))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((K, C, 3, 3)).astype(np.float32) * np.float32(np.sqrt(2.0 / (9 * C)))
    b = rng.standard_normal(K).astype(np.float32)
    (sh, sw), (ph, pw) = ((v, v) if np.isscalar(v) else v for v in (stride, pad))
    P, Q = oracle.conv_out_size(H, 3, sh, ph), oracle.conv_out_size(W, 3, sw, pw)
    cd = B.conv_desc(K, C, 3, 3, stride, pad, True, B.DR_KCRS)
    buf = torch.zeros(w.size + 4, device="cuda")
    for shift in (0, 1):                # filters on a 16-byte boundary, and one word behind it (the general path)
        wg = buf[shift:shift + w.size].view(K, C, 3, 3)
        wg.copy_(gpu(w))
        for bias in (b, None):
            ref = oracle.conv2d(x, w, b if bias is not None else np.zeros(K, np.float32), stride, pad, True)
            y = torch.full((N, K + 3, P, Q), float("nan"), device="cuda")
            B.conv2d_fwd(gpu(x), cd, wg, None if bias is None else gpu(bias), y, 2)
            torch.cuda.synchronize()
            assert close(host(y[:, 2:K + 2]), ref, TOL_F32), (shift, bias is None)
            assert bool(torch.isnan(y[:, :2]).all()) and bool(torch.isnan(y[:, K + 2:]).all())
