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

BF16 = [
    # N Cin H W Cout KH KW stride pad groups; kernel.  Reductions with a last k-step that is partly empty.
    (S(50, 36, 11, 13, 40, 3, 3, 1, 1, 1), "conv_split3<"),      # 36 channels in chunks of sixteen: tap 9 does not exist
    (S(40, 44, 12, 14, 48, 3, 3, 2, 1, 1), "conv_split3<"),      # the same, stride 2, even rows
    (S(3, 36, 9, 16, 48, 3, 3, 1, 1, 3), "conv_split3<"),        # three groups of 12 channels
    (S(2, 48, 10, 10, 32, 3, 3, 1, 1, 2), "conv_mfma16b<"),      # chunks of 8 channels: three of the last four units empty
    (S(3, 32, 9, 12, 64, 3, 3, 2, 1, 2), "conv_mfma16b<"),       # chunks of 16: two empty
    (S(2, 48, 10, 12, 32, 3, 3, 1, 0, 2), "conv_mfma16b<"),      # no padding
]


@pytest.mark.parametrize("s,kernel", BF16, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_bf16_infinity_stays_an_infinity(gpu, s, kernel):
    torch, b = gpu
    x, w = wl.make_input((s.N, s.Cin, s.H, s.W), 91), wl.make_weight(s.Cout, s.Cin // s.groups, 3, 3, 92)
    x[0, 0, 0, 0] = x[0, s.Cin - 1, s.H - 1, s.W - 1] = x[s.N - 1, 3, 4, 5] = np.inf
    x[0, 1, 3, 5] = x[1, 7, 3, 2] = -np.inf
    _, xr = wl.round_to_bf16(x)
    _, wr = wl.round_to_bf16(w)
    pw = b.gspc_pack_weights(torch.from_numpy(w).cuda(), s.groups, b.GSPC_BF16)
    xd = b.gspc_pack_input_bf16(torch.from_numpy(x).cuda())
    y = b.gspc_conv2d_grouped(xd, pw, s.N, s.Cin, s.H, s.W, s.Cout, 3, 3, s.stride, s.pad, s.groups)
    torch.cuda.synchronize()
    assert b.gspc_last_kernel().startswith(kernel), b.gspc_last_kernel()
    y = y.cpu().numpy()
    ref = oracle.conv2d_grouped(xr, wr, s.stride, s.pad, s.groups, threads=8)
    assert np.isinf(ref).any() and np.array_equal(np.isnan(y), np.isnan(ref)), b.gspc_last_kernel()
    inf = np.isinf(ref)
    assert np.array_equal(np.isinf(y), inf) and np.array_equal(np.sign(y[inf]), np.sign(ref[inf]))
    ok = np.isfinite(ref)
    assert rel_err(y[ok], ref[ok]) < 1e-4
