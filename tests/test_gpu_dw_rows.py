"""Depthwise 3x3 layers on planes without an instance of their own (bands of rows, or several planes, per wavefront),
against the oracle's plain definition of the grouped convolution (Section II, Fig. 2)."""
import numpy as np
import pytest

import oracle
from helpers import err_metrics
from paper_2006_09791_amd import workloads as wl
from test_gpu_parity import gpu, run_conv  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def dw(N, C, H, W, stride):
    return wl.ConvShape(N, C, H, W, C, 3, 3, stride, 1, C)


SHAPES = [
    (dw(5, 13, 95, 95, 1), "1,false"),     # bands of one plane; planes that start at any alignment
    (dw(5, 13, 95, 95, 2), "2,false"),
    (dw(11, 13, 46, 85, 1), "1,false"),    # the last band shorter, its last strip ragged
    (dw(20, 13, 27, 79, 2), "2,false"),    # odd height at stride 2: the row below the plane
    (dw(3, 6, 90, 331, 1), "1,false"),     # long rows, four output rows per band
    (dw(3, 15, 90, 201, 2), "2,false"),
    (dw(3, 341, 1, 682, 1), "1,false"),    # one row: windows past the band; the last wavefronts of a block above 64 KB of LDS,
    (dw(4, 500, 2, 901, 2), "2,false"),    # 144 KB: the third and fourth load there as well
    (dw(3, 667, 2, 901, 2), "2,false"),    # ... of a last block with one wavefront
    (dw(1, 3, 5, 1, 1), "1,false"),        # one column
    (dw(1, 1, 1, 1, 2), "2,false"),        # one element
    (dw(400, 13, 9, 9, 1), "1,true"),      # several planes per wavefront, the last one with fewer
    (dw(401, 13, 9, 11, 2), "2,true"),
    (dw(700, 11, 2, 3, 1), "1,true"),      # planes of six elements
    (dw(700, 11, 1, 1, 1), "1,true"),      # of one
    (dw(300, 7, 8, 5, 2), "2,true"),
]


@pytest.mark.parametrize("s,kind", SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_rows(gpu, s, kind):
    y, x, w, name = run_conv(gpu, s, seed=81)
    assert name == f"conv_direct_rows<{kind}>", name
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    assert not np.isnan(y).any()
    # nine fused multiply-adds: each rounds the running sum by 2^-24 of sum |x w| at most
    assert err_metrics(y, ref, absum)["bound"] < 9 * 2.0 ** -24


@pytest.mark.parametrize("s,kernel", [
    (dw(3, 5, 89, 89, 1), "conv_direct_flat<"),       # 15 planes: a band per wavefront leaves most of the chip idle
    (dw(2, 5, 66, 66, 1), "conv_direct_flat<"),
    (dw(8, 1, 70, 70, 2), "conv_direct_flat<"),
    (dw(2, 21, 45, 45, 1), "conv_direct_flat<"),
    (dw(1, 208, 60, 60, 2), "conv_direct_rows<"),
    (dw(3, 72, 23, 93, 2), "conv_direct_rows<"),
    (dw(7, 37, 60, 61, 2), "conv_direct_rows<"),
    (dw(1, 92, 87, 87, 1), "conv_direct_rows<"),
    (dw(4, 115, 8, 8, 1), "conv_direct_rows<"),       # whole-quad rows: small planes in small launches
    (dw(2, 37, 4, 4, 1), "conv_direct_rows<"),
    (dw(130, 100, 8, 8, 1), "conv_direct_small<"),
    (dw(4, 115, 8, 8, 2), "conv_direct_small<"),
    (dw(12, 30, 32, 32, 1), "conv_direct_small<"),
    (dw(1, 3, 31, 31, 1), "conv_direct_rows<"),       # planes of up to about 40x40: at any launch size
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_launches_of_few_planes(gpu, s, kernel):
    y, x, w, name = run_conv(gpu, s, seed=82)
    assert name.startswith(kernel), name
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    assert err_metrics(y, ref, absum)["bound"] < 9 * 2.0 ** -24


@pytest.mark.parametrize("s,kernel", [
    (dw(115, 512, 8, 8, 1), "conv_direct_rows<1,true>"),         # whole-quad rows from 30 MB on
    (dw(114, 512, 8, 8, 1), "conv_direct_small<1,1,1,4,f32>"),
    (dw(395, 512, 8, 8, 1), "conv_direct_narrow<1,true>"),       # ... and from 100 MB with one output row per item
    (dw(380, 512, 8, 8, 1), "conv_direct_rows<1,true>"),         # 99.6 MB
    (dw(76, 512, 28, 32, 1), "conv_direct_rows<1,false>"),
    (dw(800, 512, 8, 8, 2), "conv_direct_narrow<2,true>"),
    (dw(250, 511, 9, 9, 2), "conv_direct_rows<2,true>"),         # regions of 3 KB
    (dw(90, 512, 87, 9, 1), "conv_direct_narrow<1,false>"),      # short rows: one output row per item, bands
    (dw(701, 511, 11, 9, 1), "conv_direct_narrow<1,true>"),      # several planes, the last wavefront with fewer
    (dw(100, 512, 90, 13, 2), "conv_direct_narrow<2,false>"),
    (dw(19, 512, 87, 9, 1), "conv_direct_narrow<1,false>"),      # bands from 60 MB on
    (dw(18, 512, 87, 9, 1), "conv_direct_rows<1,false>"),
    (dw(200, 512, 17, 17, 1), "conv_direct_narrow<1,true>"),     # 16 and 17 outputs on planes of more than 256 elements
    (dw(170, 512, 13, 17, 1), "conv_direct_rows<1,true>"),
    (dw(170, 512, 17, 18, 1), "conv_direct_rows<1,false>"),
    (dw(240, 272, 15, 15, 1), "conv_direct_narrow<1,true>"),     # never one small plane per wavefront
    (dw(530, 511, 25, 8, 2), "conv_direct_narrow<2,true>"),
    (dw(530, 511, 25, 9, 2), "conv_direct_narrow<2,true>"),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_launches_past_the_cache(gpu, s, kernel):
    y, x, w, name = run_conv(gpu, s, seed=83)
    assert name == kernel, name
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    assert not np.isnan(y).any()
    assert err_metrics(y, ref, absum)["bound"] < 9 * 2.0 ** -24


@pytest.mark.parametrize("N,C,H,W,kernel", [(9, 24, 61, 67, "rows"), (600, 6, 9, 9, "rows"), (90, 512, 87, 9, "narrow")])
def test_rows_residual_relu(gpu, N, C, H, W, kernel):
    torch, b = gpu
    dev = "cuda:0"
    ch = wl.Chain("dw", (N, C, H, W))
    ch.conv(0, 1, N, C, H, W, C, 3, 1, 1, C)
    ch.conv(1, 2, N, C, H, W, C, 3, 1, 1, C, relu=True, residual=0)
    x0, weights = wl.make_input(ch.input_shape, 6), ch.make_weights(7)
    b.gspc_set_chain_fusion(0)
    try:
        packed = [b.gspc_pack_weights(torch.from_numpy(v).to(dev), g) for v, g in zip(weights, ch.weight_groups)]
        bufs = [torch.empty(max(n, 1), device=dev) for n in ch.buf_elems]
        bufs[0].copy_(torch.from_numpy(x0).reshape(-1))
        b.gspc_run_layer_chain(b.LayerChain(ch.layers, packed, bufs))
        torch.cuda.synchronize()
        assert b.gspc_last_kernel().startswith(f"conv_direct_{kernel}<"), b.gspc_last_kernel()
    finally:
        b.gspc_set_chain_fusion(1)
    ref = oracle.run_chain(ch.layers, len(ch.buf_elems), x0, weights, threads=4)[ch.out_buf]
    got = bufs[ch.out_buf][:ref.size].cpu().numpy().reshape(ref.shape)
    rms = float(np.sqrt(np.mean(ref * ref)))
    # two layers of nine terms: 20 roundings of values up to a few times the result's rms
    assert float(np.max(np.abs(got - ref))) < 1e-5 * max(rms, 1.0)


def test_rows_infinity(gpu):
    """An infinity reaches the outputs whose windows hold it, and no other: neither across rows nor across planes."""
    torch, b = gpu
    for N, C, H, W in [(8, 26, 50, 49), (500, 5, 7, 9), (90, 512, 87, 9)]:
        x = np.ones((N, C, H, W), np.float32)
        x[0, 0, 3, W - 1] = np.inf
        x[0, 0, H - 1, 0] = -np.inf
        w = np.ones((C, 1, 3, 3), np.float32)
        pw = b.gspc_pack_weights(torch.from_numpy(w).to("cuda:0"), C)
        y = b.gspc_conv2d_grouped(torch.from_numpy(x).to("cuda:0"), pw, N, C, H, W, C, 3, 3, 1, 1, C).cpu().numpy()
        assert b.gspc_last_kernel().startswith("conv_direct_narrow<" if W * N * C * H > 3e7 else "conv_direct_rows<")
        bad = ~np.isfinite(y)
        want = np.zeros_like(bad)
        want[0, 0, 2:5, W - 2:] = True
        want[0, 0, H - 2:, :2] = True
        assert (bad == want).all()


def test_plane_kernels_can_be_switched_off(gpu):
    """GSPC_NO_DWPLANES leaves depthwise layers to the strip and flat kernels (read once per process, hence the child)."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = f"""
import sys
sys.path.insert(0, {root!r})
import torch
from paper_2006_09791_amd import binding as b
for N, C, H in ((20, 64, 15), (20, 64, 16), (128, 64, 14)):
    pw = b.gspc_pack_weights(torch.randn(C, 1, 3, 3, device="cuda"), C)
    b.gspc_conv2d_grouped(torch.randn(N, C, H, H, device="cuda"), pw, N, C, H, H, C, 3, 3, 1, 1, C)
    torch.cuda.synchronize()
    print(b.gspc_last_kernel())
"""
    out = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, GSPC_NO_DWPLANES="1"), check=True,
                         capture_output=True, text=True).stdout
    names = [l.split("<")[0] for l in out.splitlines() if l.startswith("conv_")]
    assert names == ["conv_direct_flat", "conv_direct_small", "conv_direct_flat"], out
