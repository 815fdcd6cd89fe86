"""3x3 layers of few filters per group on the bf16 matrix instruction: blocks of 16 and 32 filters, filters that the
kernel splits itself, and the bf16 layers it takes from the 16x16x32 kernel; against the oracle's plain definition."""
import numpy as np
import pytest

import oracle
from helpers import err_metrics
from paper_2006_09791_amd import workloads as wl
from test_gpu_parity import gpu, run_conv  # noqa: F401  (fixture)
from test_gpu_split import split_bound

pytestmark = pytest.mark.gpu
S = wl.ConvShape
SHAPES = [
    # N Cin H W Cout KH KW stride pad groups
    (S(30, 56, 46, 46, 56, 3, 3, 1, 1, 2), "2,4,1,4,1,", "f32,true,true>"),          # 28 filters, padded channels
    (S(30, 138, 29, 29, 138, 3, 3, 1, 1, 2), "", "f32,false,false>"),     # 69: two tiles of 32 and five left
    (S(25, 160, 33, 33, 24, 3, 3, 1, 1, 2), "1,4,1,4,1,", "f32,false,false>"),      # 12 filters, 80 channels
    (S(120, 128, 23, 23, 128, 3, 3, 2, 1, 4), "", "f32,false,false>"),     # stride 2
    (S(4, 378, 38, 38, 36, 3, 3, 1, 1, 3), "1,2,1,4,1,", "f32,true,true>"),         # 126 channels
    (S(12, 64, 55, 55, 64, 3, 3, 1, 1, 4), "1,4,1,4,1,", "f32,false,false>/plain"),  # 16 and 16: split in the kernel
    (S(40, 64, 50, 46, 64, 3, 3, 1, 1, 4), "1,4,1,4,1,", "f32,true,true>/plain"),
    (S(200, 60, 31, 31, 36, 3, 3, 2, 1, 4), "1,2,1,4,1,", "f32,false,false>/plain"),  # stride 2, 15 and 9
    (S(30, 20, 70, 94, 16, 3, 3, 1, 1, 2), "1,4,1,4,1,", "f32,true,true>/plain"),    # 10 and 8
    (S(30, 60, 45, 47, 144, 3, 3, 1, 1, 6), "2,4,1,4,1,", "f32,false,false>"),      # 10 and 24: few weights, but split at packing
    (S(28, 60, 54, 54, 68, 3, 3, 2, 1, 4), "2,2,2,2,1,", "f32,true,false>"),         # 15 and 17 at stride 2, whose tiles fit no other block
    (S(24, 36, 76, 76, 72, 3, 3, 2, 1, 4), "2,2,2,2,1,", "f32,true,true>"),          # 9 and 18
    (S(40, 66, 60, 58, 6, 3, 3, 1, 1, 1), "1,4,1,4,1,", "f32,true,true>"),          # six filters
    (S(7, 120, 44, 44, 6, 3, 3, 1, 1, 3), "1,4,1,4,1,", "f32,true,true>/plain"),     # two filters
    (S(8, 100, 9, 9, 3, 3, 3, 1, 1, 1), "", "f32,false,false>"),                    # three
    (S(9, 30, 21, 22, 4, 3, 3, 1, 1, 2), "", "f32,true,false>/plain"),              # 15 channels, two filters
    (S(40, 300, 17, 17, 6, 3, 3, 1, 1, 3), "", "bf16,false,false>"),                # bf16, two filters
    (S(186, 7, 66, 66, 7, 3, 3, 2, 1, 1), "", "bf16,true,false>"),                  # seven and seven, stride 2
    (S(10, 72, 33, 34, 72, 3, 3, 1, 1, 4), "", "bf16,true,false>"),                 # groups of 18
    (S(6, 189, 18, 20, 189, 3, 3, 1, 1, 3), "", "bf16,true,true>"),                 # of 63
    (S(20, 104, 20, 39, 104, 3, 3, 1, 1, 1), "", "bf16,false,false>"),              # 104 channels
    (S(64, 256, 14, 14, 256, 3, 3, 1, 1, 2), "", "bf16,true,true>"),                # 128
    (S(10, 80, 41, 44, 57, 3, 3, 2, 1, 1), "", "bf16,true,false>"),                 # stride 2, 57 filters
    (S(3, 70, 40, 41, 49, 3, 3, 1, 1, 7), "", "bf16,false,false>"),                 # 10 and 7
]


@pytest.mark.parametrize("s,block,form", SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_blocks(gpu, s, block, form):
    torch, b = gpu
    bf16 = form.startswith("bf16")
    y, x, w, name = run_conv(gpu, s, seed=91, dtype=b.GSPC_BF16 if bf16 else b.GSPC_F32)
    assert name.startswith("conv_split3<" + block) and name.endswith(form), name
    if bf16:
        x, w = wl.round_to_bf16(x)[1], wl.round_to_bf16(w)[1]
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    assert not np.isnan(y).any(), name
    m = err_metrics(y, ref, absum)
    # (the bound of the pointwise form for nine times the terms, a quarter of a k-step lost per 16 channels)
    assert m["bound"] < split_bound(9 * s.Cin // s.groups + 16), (name, m)


@pytest.mark.parametrize("s,block", [
    (S(93, 228, 32, 16, 456, 3, 3, 2, 1, 3), "2,4,2,2,1,"),        # stride 2: near ties of 64 filters by 128 and by 64 pixels
    (S(72, 48, 52, 52, 100, 3, 3, 2, 1, 1), "2,4,2,2,1,"),
    (S(86, 336, 15, 8, 336, 3, 3, 2, 1, 1), "2,2,1,1,4,"),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_fp32_block_shapes(gpu, s, block):
    y, x, w, name = run_conv(gpu, s, seed=97)
    assert name.startswith("conv_split3<" + block), name
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    assert err_metrics(y, ref, absum)["bound"] < split_bound(9 * s.Cin // s.groups + 16) + 4 * 2.0 ** -24, name


@pytest.mark.parametrize("s,kernel", [
    (S(11, 15, 24, 24, 96, 3, 3, 1, 1, 3), "conv_mfma16<"),        # 5 channels, 32 filters, few blocks
    (S(5, 56, 23, 23, 192, 3, 3, 1, 1, 8), "conv_mfma16<"),        # 7 and 24, odd rows
    (S(18, 96, 31, 31, 512, 3, 3, 1, 1, 16), "conv_mfma16<"),      # 6 and 32 at a launch that fills the chip
    (S(11, 104, 58, 16, 208, 3, 3, 2, 1, 2), "conv_mfma16<"),      # stride 2, 52 and 104: no block of 64 filters twice per unit
    (S(127, 128, 12, 12, 128, 3, 3, 2, 1, 2), "conv_mfma16w<"),    # the kernel with resident filters
    (S(106, 6, 14, 23, 12, 3, 3, 2, 1, 2), "conv_direct_generic<"),  # 3 channels: 27 terms
    (S(72, 32, 35, 35, 32, 3, 3, 1, 1, 2), "conv_split3<"),        # 16 and 16
    (S(55, 14, 8, 42, 14, 3, 3, 1, 1, 2), "conv_split3<"),         # 7 and 7
    (S(20, 188, 14, 14, 188, 3, 3, 2, 1, 1), "conv_split3<"),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_fp32_layers_that_other_kernels_take_too(gpu, s, kernel):
    """The split kernel leaves layers of few products to the staged and the generic kernel where its estimate is behind."""
    y, x, w, name = run_conv(gpu, s, seed=96)
    assert name.startswith(kernel), name
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    # (the others: a product and a sum per term, each rounded once at most)
    k = 9 * s.Cin // s.groups
    bound = split_bound(k + 16) + 4 * 2.0 ** -24 if name.startswith("conv_split3<") else (k + 17) * 2.0 ** -24
    assert err_metrics(y, ref, absum)["bound"] < bound, name


@pytest.mark.parametrize("s,block", [
    (S(9, 348, 19, 19, 216, 3, 3, 1, 1, 3), "2,4,2,2,1,"),         # 116 channels, 72 filters in 200 tiles
    (S(3, 969, 17, 17, 96, 3, 3, 1, 1, 3), "2,2,2,2,1,"),          # 323 and 32
    (S(1, 292, 14, 23, 75, 3, 3, 1, 1, 1), "2,2,2,2,1,"),
    (S(18, 68, 56, 56, 68, 3, 3, 2, 1, 1), "2,2,2,2,1,"),          # stride 2: a block per compute unit, or two of half the size
    (S(39, 33, 29, 29, 66, 3, 3, 1, 1, 3), "2,4,1,4,1,"),          # 11 and 22, many tiles: the block of 32 filters x 256 pixels
    (S(102, 68, 10, 10, 68, 3, 3, 1, 1, 1), "1,4,1,4,1,"),         # 16 x 256
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_bf16_block_shapes(gpu, s, block):
    """Blocks of few filters stage a tile once per 16 or 32 filters: long reductions in few blocks keep the 64-filter ones."""
    torch, b = gpu
    y, x, w, name = run_conv(gpu, s, seed=94, dtype=b.GSPC_BF16)
    assert name.startswith("conv_split3<" + block), name
    x, w = wl.round_to_bf16(x)[1], wl.round_to_bf16(w)[1]
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    assert err_metrics(y, ref, absum)["bound"] < split_bound(9 * s.Cin // s.groups + 16), name


@pytest.mark.parametrize("s,kernel", [
    (S(24, 28, 11, 7, 28, 3, 3, 1, 1, 4), "conv_mfma16<"),         # groups of 7 on odd rows
    (S(3, 14, 7, 7, 15, 3, 3, 1, 1, 1), "conv_mfma16<"),
    (S(4, 10, 24, 22, 20, 3, 3, 1, 1, 2), "conv_mfma16<"),         # even rows, groups of 5
    (S(16, 7, 42, 31, 7, 3, 3, 1, 1, 1), "conv_mfma16<"),          # 92 instructions per compute unit
    (S(40, 7, 42, 31, 7, 3, 3, 1, 1, 1), "conv_split3<"),          # 230
    (S(26, 12, 10, 10, 12, 3, 3, 1, 1, 1), "conv_split3<"),        # even rows, 12 channels
    (S(24, 28, 11, 7, 28, 3, 3, 2, 1, 4), "conv_split3<"),         # stride 2
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_bf16_layers_of_few_products(gpu, s, kernel):
    """Channel counts without a 16x16x32 section: small launches keep the staged kernel."""
    torch, b = gpu
    y, x, w, name = run_conv(gpu, s, seed=95, dtype=b.GSPC_BF16)
    assert name.startswith(kernel), name
    x, w = wl.round_to_bf16(x)[1], wl.round_to_bf16(w)[1]
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    # (the staged kernel: every instruction of four terms rounds its sum once, for each of up to 16 channels and 9 taps)
    k = 9 * s.Cin // s.groups
    assert err_metrics(y, ref, absum)["bound"] < max(split_bound(k + 16), (k + 17) * 2.0 ** -24), name


@pytest.mark.parametrize("s,kernel", [
    (S(4, 48, 33, 33, 48, 3, 3, 2, 1, 4), "conv_mfma16b<"),        # merged in pairs, few blocks
    (S(15, 24, 9, 9, 112, 3, 3, 1, 1, 2), "conv_mfma16b<"),
    (S(6, 24, 25, 25, 24, 3, 3, 2, 1, 4), "conv_mfma16b<"),        # four groups of 6 channels in one
    (S(59, 24, 98, 98, 24, 3, 3, 2, 1, 4), "conv_mfma16b<"),       # at a launch that fills the chip
    (S(4, 96, 107, 107, 96, 3, 3, 1, 1, 16), "conv_mfma16b<"),
    (S(2, 544, 45, 13, 136, 3, 3, 1, 1, 2), "conv_mfma16b<"),      # 272 channels in chunks of 16, no merging
    (S(8, 208, 15, 15, 208, 3, 3, 1, 1, 1), "conv_mfma16b<"),
    (S(66, 160, 46, 16, 160, 3, 3, 2, 1, 32), "conv_split3<"),     # eight groups of 5 in one
    (S(40, 63, 8, 8, 63, 3, 3, 1, 1, 1), "conv_split3<"),
    (S(8, 192, 34, 34, 384, 3, 3, 1, 1, 32), "conv_split3<"),
    (S(16, 104, 20, 79, 104, 3, 3, 1, 1, 1), "conv_split3<"),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_bf16_layers_that_the_16x16x32_kernel_takes_too(gpu, s, kernel):
    """The one with the shorter estimate: the split kernel's form leaves the other's layers alone where it is behind."""
    torch, b = gpu
    y, x, w, name = run_conv(gpu, s, seed=93, dtype=b.GSPC_BF16)
    assert name.startswith(kernel), name
    x, w = wl.round_to_bf16(x)[1], wl.round_to_bf16(w)[1]
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    # (merged groups add zeros only: the bound of their own terms, each k-step of either kernel rounded once)
    assert err_metrics(y, ref, absum)["bound"] < split_bound(9 * s.Cin // s.groups + 16) + 4 * 2.0 ** -24, name


@pytest.mark.parametrize("s", [S(12, 64, 55, 55, 64, 3, 3, 1, 1, 4), S(30, 138, 29, 29, 138, 3, 3, 1, 1, 2)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("xs,ws", [(-110, 60), (60, -110), (70, 40)])
def test_scales(gpu, s, xs, ws):
    """Factors far from 1, and sums that overflow the scaled accumulators (recomputed as plain sums)."""
    torch, b = gpu
    x = wl.make_input((s.N, s.Cin, s.H, s.W), 92)
    w = wl.make_weight(s.Cout, s.Cin // s.groups, 3, 3, 92)
    xd = torch.from_numpy(np.ldexp(x, xs)).cuda()
    pw = b.gspc_pack_weights(torch.from_numpy(np.ldexp(w, ws)).cuda(), s.groups)
    y = b.gspc_conv2d_grouped(xd, pw, s.N, s.Cin, s.H, s.W, s.Cout, 3, 3, s.stride, s.pad, s.groups).cpu().numpy()
    assert b.gspc_last_kernel().startswith("conv_split3<"), b.gspc_last_kernel()
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    m = err_metrics(np.ldexp(y.astype(np.float64), -xs - ws), ref, absum)
    # (a plain sum rounds once per term: 9 * channels roundings of at most the sum of magnitudes)
    assert m["bound"] < 9 * s.Cin // s.groups * 2.0 ** -24, m
