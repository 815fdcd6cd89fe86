"""An infinite input belongs to the outputs whose sums contain it and to no other (the convolution's definition,
Section II, Fig. 2): kernels whose reduction is padded to whole instructions must not multiply it by a padding zero."""
import numpy as np
import pytest

import oracle
from helpers import rel_err
from paper_2006_09791_amd import workloads as wl
from test_gpu_parity import gpu  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
S = wl.ConvShape

CASES = [
    # N Cin H W Cout KH KW stride pad groups; kernel; bf16.  Reductions with a last k-step that is partly empty.
    (S(50, 36, 11, 13, 40, 3, 3, 1, 1, 1), "conv_split3<", True),      # 36 channels in chunks of sixteen: tap 9 does not exist
    (S(40, 44, 12, 14, 48, 3, 3, 2, 1, 1), "conv_split3<", True),      # the same, stride 2, even rows
    (S(3, 36, 9, 16, 48, 3, 3, 1, 1, 3), "conv_split3<", True),        # three groups of 12 channels
    (S(2, 48, 10, 10, 32, 3, 3, 1, 1, 2), "conv_mfma16b<", True),      # chunks of 8 channels: three of the last four units empty
    (S(3, 32, 9, 12, 64, 3, 3, 2, 1, 2), "conv_mfma16b<", True),       # chunks of 16: two empty
    (S(2, 48, 10, 12, 32, 3, 3, 1, 0, 2), "conv_mfma16b<", True),      # no padding
    (S(120, 36, 14, 14, 64, 1, 1, 1, 0, 1), "conv_mfma16s<", True),     # pointwise: four of the last 32 channels
    (S(300, 36, 15, 15, 128, 1, 1, 1, 0, 1), "conv_mfma16s<", False),
    (S(60, 68, 14, 14, 72, 3, 3, 1, 1, 1), "conv_split3<", False),
    (S(3, 70, 9, 6, 33, 3, 3, 1, 1, 1), "conv_mfma16u<", False),        # without staging: two of the last four channels
    (S(2, 50, 9, 7, 24, 1, 1, 2, 0, 1), "conv_mfma16u<", False),
    (S(207, 34, 17, 19, 32, 3, 3, 1, 1, 1), "conv_", False),
    (S(53, 64, 8, 8, 64, 3, 3, 1, 1, 1), "conv_mfma16w<", False),
    (S(300, 32, 16, 16, 32, 3, 3, 1, 1, 8), "conv_mfma4r<", False),     # four channels and filters per group
    (S(3, 37, 14, 14, 37, 3, 3, 1, 1, 37), "conv_d", False),            # depthwise
]


@pytest.mark.parametrize("s,kernel,bf16", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_infinity_stays_an_infinity(gpu, s, kernel, bf16):
    torch, b = gpu
    x, w = wl.make_input((s.N, s.Cin, s.H, s.W), 91), wl.make_weight(s.Cout, s.Cin // s.groups, s.KH, s.KW, 92)
    x[0, 0, 0, 0] = x[0, s.Cin - 1, s.H - 1, s.W - 1] = x[s.N - 1, 3, 4, 4] = np.inf
    x[0, 1, 3, 5] = x[1, 7, 2, 2] = -np.inf
    pw = b.gspc_pack_weights(torch.from_numpy(w).cuda(), s.groups, b.GSPC_BF16 if bf16 else b.GSPC_F32)
    xd = torch.from_numpy(x).cuda()
    if bf16:
        xd, x, w = b.gspc_pack_input_bf16(xd), wl.round_to_bf16(x)[1], wl.round_to_bf16(w)[1]
    y = b.gspc_conv2d_grouped(xd, pw, s.N, s.Cin, s.H, s.W, s.Cout, s.KH, s.KW, s.stride, s.pad, s.groups)
    torch.cuda.synchronize()
    assert b.gspc_last_kernel().startswith(kernel), b.gspc_last_kernel()
    y = y.cpu().numpy()
    ref = oracle.conv2d_grouped(x, w, s.stride, s.pad, s.groups, threads=8)
    assert np.isinf(ref).any() and np.array_equal(np.isnan(y), np.isnan(ref)), b.gspc_last_kernel()
    inf = np.isinf(ref)
    assert np.array_equal(np.isinf(y), inf) and np.array_equal(np.sign(y[inf]), np.sign(ref[inf]))
    ok = np.isfinite(ref)
    assert rel_err(y[ok], ref[ok]) < 1e-4
