"""Small launches: the 16x16x4 kernel without staging, against the oracle's plain definition of the grouped
convolution (Section II, Fig. 2)."""
import numpy as np
import pytest

import oracle
from helpers import err_metrics, rel_err
from paper_2006_09791_amd import workloads as wl
from test_gpu_parity import gpu, run_conv  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
S = wl.ConvShape
SHAPES = [
    # N Cin H W Cout KH KW stride pad groups
    S(1, 64, 32, 32, 64, 3, 3, 1, 1, 4),
    S(1, 16, 1, 3, 16, 3, 3, 1, 1, 1),        # the narrowest row: every pixel at an edge
    S(2, 24, 3, 3, 24, 3, 3, 2, 1, 2),        # stride 2, odd width: the last window ends outside
    S(3, 40, 6, 4, 48, 3, 3, 2, 1, 1),        # stride 2, even width
    S(3, 70, 9, 5, 33, 3, 3, 1, 1, 1),        # padded channels and filters, 54 units in 16 waves
    S(5, 60, 29, 37, 84, 3, 3, 1, 1, 3),      # ragged last tile
    S(1, 512, 7, 7, 512, 3, 3, 1, 1, 2),      # 192 units: two rounds of loads per wave
    S(1, 256, 14, 14, 512, 1, 1, 2, 0, 1),    # 1x1, stride 2
    S(2, 50, 9, 7, 24, 1, 1, 2, 0, 1),        # 50 channels: a block of sixteen partly empty
    S(1, 960, 7, 7, 160, 1, 1, 1, 0, 1),
    S(3, 36, 5, 5, 20, 1, 1, 1, 0, 2),        # 18 channels and 10 filters per group
    S(17, 128, 4, 4, 64, 1, 1, 1, 0, 4),
    # waves that share a channel block, by threes and by pairs, and more waves than blocks
    S(1, 4, 9, 7, 16, 3, 3, 1, 1, 1),         # one block
    S(2, 16, 8, 8, 32, 3, 3, 1, 1, 1),        # four
    S(1, 23, 10, 9, 17, 3, 3, 2, 1, 1),       # six, the last one of three channels
    S(1, 36, 12, 11, 16, 3, 3, 1, 1, 1),      # nine blocks, sixteen waves
    # tiles that span images, and launches whose tiles are no multiple of the eight XCDs
    S(71, 8, 3, 3, 12, 3, 3, 1, 1, 1),        # planes of nine pixels
    S(31, 16, 3, 5, 16, 3, 3, 2, 1, 1),       # of six
    S(45, 48, 1, 3, 40, 1, 1, 1, 0, 1),       # of three
    S(1, 64, 5, 5, 48, 3, 3, 1, 1, 1),        # six tiles
]


@pytest.mark.parametrize("s", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_unit_kernel(gpu, s):
    y, x, w, name = run_conv(gpu, s, seed=61)
    assert name.startswith("conv_mfma16u<"), name
    assert not np.isnan(y).any(), name
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, s.pad, s.groups, return_abs=True, threads=8)
    m = err_metrics(y, ref, absum)
    # a product and a sum per term, each rounded once at most: K + 16 roundings of the running sum
    K = s.Cin // s.groups * s.KH * s.KW
    assert m["bound"] < (K + 17) * 2.0 ** -24, (name, m)
    assert m["floored"] < 1e-5, (name, m)


@pytest.mark.parametrize("s,waves", [
    (S(1, 64, 32, 32, 64, 3, 3, 1, 1, 4), 8),      # 256 tiles
    (S(21, 16, 12, 12, 32, 3, 3, 1, 1, 2), 4),     # 378 tiles of six units
    (S(6, 64, 16, 16, 128, 3, 3, 1, 1, 4), 2),     # 768 tiles of twelve
    (S(93, 96, 7, 7, 16, 1, 1, 1, 0, 2), 2),       # 570 tiles
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_unit_kernel_waves_start_together(gpu, s, waves):
    """Blocks get more waves than their units need only while the launch keeps to eight waves per compute unit."""
    name = run_conv(gpu, s, seed=62)[3]
    assert name.startswith(f"conv_mfma16u<{waves},"), name


@pytest.mark.parametrize("s,kernel", [
    (S(4, 144, 64, 64, 24, 1, 1, 1, 0, 1), "conv_mfma16<"),       # 2048 tiles of nine units on whole quads
    (S(4, 144, 62, 66, 24, 1, 1, 1, 0, 1), "conv_mfma16u<"),      # 2046
    (S(94, 64, 7, 7, 96, 1, 1, 1, 0, 1), "conv_mfma16<"),         # 1728 tiles, 47 pairs of images times 6
    (S(55, 64, 7, 7, 96, 1, 1, 1, 0, 1), "conv_mfma16u<"),        # 1014 tiles: all blocks run together
    (S(128, 64, 7, 7, 96, 1, 1, 1, 0, 1), "conv_mfma16u<"),       # 384 pairs: no longer a block per image
    (S(94, 66, 7, 7, 96, 1, 1, 1, 0, 1), "conv_mfma16u<"),        # channels that are no whole quads
    (S(115, 64, 6, 7, 96, 1, 1, 1, 0, 1), "conv_mfma16<"),        # 42 pixels
    (S(120, 64, 5, 7, 96, 1, 1, 1, 0, 1), "conv_mfma16u<"),       # 35
    (S(151, 256, 9, 9, 48, 1, 1, 1, 0, 4), "conv_mfma16u<"),      # 81 pixels, 12 filters per group, 3060 tiles
    (S(152, 256, 9, 9, 48, 1, 1, 1, 0, 4), "conv_mfma16<"),       # 3080
    (S(190, 128, 7, 7, 32, 1, 1, 1, 0, 2), "conv_mfma16<"),       # one filter tile per group, 95 pairs times 2
    (S(768, 128, 7, 7, 16, 1, 1, 1, 0, 1), "conv_mfma16s<"),      # 384 pairs
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_pointwise_layers_return_to_staging(gpu, s, kernel):
    """From the launch size on where the staged kernel is ahead; odd planes where one row fills its tiles."""
    y, x, w, name = run_conv(gpu, s, seed=64)
    assert name.startswith(kernel), name
    ref, absum = oracle.conv2d_grouped(x, w, 1, 0, s.groups, return_abs=True, threads=8)
    # (the split kernel: three dropped products, six roundings per 32 channels and the final sum, less than this)
    assert err_metrics(y, ref, absum)["bound"] < (s.Cin // s.groups + 17) * 2.0 ** -24, name


@pytest.mark.parametrize("s,kernel", [
    (S(49, 16, 16, 16, 64, 3, 3, 2, 1, 2), "conv_mfma16u<"),      # 784 tiles of six units
    (S(193, 32, 16, 16, 64, 3, 3, 2, 1, 4), "conv_mfma16u<"),     # 3088, 16 filters per group
    (S(97, 32, 16, 16, 80, 3, 3, 2, 1, 4), "conv_mfma16<"),       # 3104, 20 filters
    (S(96, 32, 16, 16, 80, 3, 3, 2, 1, 4), "conv_mfma16u<"),      # 3072
    (S(3, 40, 32, 32, 128, 3, 3, 1, 1, 2), "conv_mfma16w<"),      # 1536 tiles of 15 units, four waves each
    (S(3, 40, 32, 31, 128, 3, 3, 1, 1, 2), "conv_mfma16u<"),      # rows that it does not read four at a time
    (S(3, 32, 32, 32, 128, 3, 3, 1, 1, 2), "conv_mfma16u<"),      # 12 units
    (S(2, 40, 32, 32, 128, 3, 3, 1, 1, 2), "conv_mfma16u<"),      # 1024 tiles
    (S(20, 16, 16, 16, 64, 3, 3, 1, 1, 2), "conv_mfma16w<"),      # 1280 tiles of six units
    (S(19, 16, 16, 16, 64, 3, 3, 1, 1, 2), "conv_mfma16u<"),      # 1216
    (S(142, 16, 14, 8, 32, 3, 3, 1, 1, 2), "conv_mfma16u<"),      # 1988, planes of 112 pixels
    (S(22, 24, 12, 12, 128, 3, 3, 1, 1, 2), "conv_mfma16u<"),     # rows of 12
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_large_launches_return_to_staging(gpu, s, kernel):
    y, x, w, name = run_conv(gpu, s, seed=65)
    assert name.startswith(kernel), name
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    assert err_metrics(y, ref, absum)["bound"] < (9 * s.Cin // s.groups + 17) * 2.0 ** -24, name


@pytest.mark.parametrize("s,kernel", [
    # (the bound on the loads, tiles x units x loads of a unit, is 200k, for 1x1 on whole quads of pixels at stride 1 180k)
    (S(5, 256, 86, 86, 256, 3, 3, 2, 1, 16), "conv_mfma16u<"),    # generic, 222k
    (S(46, 126, 12, 93, 60, 3, 3, 2, 1, 3), "conv_mfma16u<"),     # padded channels and filters, 321k
    (S(190, 96, 27, 27, 40, 1, 1, 2, 0, 1), "conv_mfma16u<"),     # 1x1, stride 2, 210k
    (S(40, 500, 28, 30, 36, 1, 1, 2, 0, 1), "conv_mfma16u<"),     # 252k
    (S(10, 700, 14, 14, 112, 1, 1, 1, 0, 1), "conv_mfma16u<"),    # whole quads of pixels, 189k
    (S(28, 692, 21, 21, 24, 1, 1, 1, 0, 1), "conv_mfma16u<"),     # odd planes, 340k
    (S(1, 644, 25, 25, 477, 1, 1, 1, 0, 1), "conv_mfma16u<"),     # 258k
    # odd planes that are staged as single rows: twenty chunks of the reduction, ten
    (S(12, 640, 11, 11, 236, 1, 1, 1, 0, 1), "conv_mfma16u<"),
    (S(164, 320, 11, 11, 32, 1, 1, 1, 0, 1), "conv_mfma16<"),
    (S(12, 628, 6, 11, 544, 1, 1, 1, 0, 1), "conv_mfma16u<"),     # 157 chunks
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_beyond_the_bound(gpu, s, kernel):
    """Layers that the generic or the staged kernel would serve 4 bytes at a time."""
    y, x, w, name = run_conv(gpu, s, seed=66)
    assert name.startswith(kernel), name
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, s.pad, s.groups, return_abs=True, threads=8)
    assert err_metrics(y, ref, absum)["bound"] < (s.KH * s.KW * s.Cin // s.groups + 17) * 2.0 ** -24, name


@pytest.mark.parametrize("s", [S(2, 48, 9, 7, 40, 3, 3, 1, 1, 2), S(3, 40, 7, 7, 24, 1, 1, 2, 0, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_unit_kernel_epilogue_and_buffer_ends(gpu, s):
    """Residual and ReLU; inputs and outputs at the ends of larger buffers: nothing outside is written, and
    what lies outside (NaN) is not read into a result."""
    torch, b = gpu
    dev = torch.device("cuda:0")
    x, w = wl.make_input((s.N, s.Cin, s.H, s.W), 63), wl.make_weight(s.Cout, s.Cin // s.groups, s.KH, s.KW, 64)
    ho, wo = b.gspc_output_dims(s.H, s.W, s.KH, s.KW, s.stride, s.pad)
    res = wl.make_input((s.N, s.Cout, ho, wo), 65)
    guard = 1024
    big = [torch.full((a.size + 2 * guard,), float("nan"), device=dev) for a in (x, res, res)]
    xd, rd, yd = (t[guard:guard + a.size] for t, a in zip(big, (x, res, res)))
    xd.copy_(torch.from_numpy(x).reshape(-1))
    rd.copy_(torch.from_numpy(res).reshape(-1))
    pw = b.gspc_pack_weights(torch.from_numpy(w).to(dev), s.groups)
    layer = wl.Layer("conv", 0, 1, 2, s.N, s.Cin, s.H, s.W, s.Cout, s.KH, s.KW, s.stride, s.pad, s.groups, True, 0)
    b.gspc_run_layer_chain(b.LayerChain([layer], [pw], [xd, rd, yd]))
    torch.cuda.synchronize()
    assert b.gspc_last_kernel().startswith("conv_mfma16u<"), b.gspc_last_kernel()
    out = big[2].cpu().numpy()
    assert np.isnan(out[:guard]).all() and np.isnan(out[guard + res.size:]).all()
    ref = oracle.relu(oracle.add(oracle.conv2d_grouped(x, w, s.stride, s.pad, s.groups, threads=8), res))
    assert rel_err(out[guard:guard + res.size].reshape(res.shape), ref) < 1e-5
