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
    cpg = s.Cin // s.groups
    # from the second image on: one channel per group and every third pixel, which give sums of one term
    one = np.zeros((s.N, cpg, s.H, s.W), bool)
    for n in range(1, s.N):
        one[n, n % cpg, 1::3, 1::3] = True
    one[0] = True
    x = np.where(np.tile(one, (1, s.groups, 1, 1)), x, np.float32(0))
    x, w = (np.ldexp(np.ldexp(a, e), -e) for a, e in ((x, xs), (w, ws)))   # (what 2^-110 leaves of the smallest values)
    xd = torch.from_numpy(np.ldexp(x, xs)).cuda()
    pw = b.gspc_pack_weights(torch.from_numpy(np.ldexp(w, ws)).cuda(), s.groups)
    y = b.gspc_conv2d_grouped(xd, pw, s.N, s.Cin, s.H, s.W, s.Cout, 3, 3, s.stride, s.pad, s.groups).cpu().numpy()
    assert b.gspc_last_kernel().startswith("conv_split3<"), b.gspc_last_kernel()
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    err = np.abs(np.ldexp(y.astype(np.float64), -xs - ws) - ref) * 2.0 ** 24
    if xs + ws < 100:
        assert np.max(err[0] / absum[0]) < split_bound(9 * cpg + 16) * 2.0 ** 24
    else:   # (a plain sum rounds once per term: 9 * channels roundings of at most the sum of magnitudes)
        assert np.max(err[0] / absum[0]) < 9 * cpg
    # one term: three dropped products of half a unit and a rounding per product kept; without an operand's third part up to 128
    assert np.max(err[1:] - 7.5 * absum[1:]) <= 0.0, np.max(err[1:] / np.maximum(absum[1:], 1e-30))


FEW = [
    (S(30, 56, 46, 46, 56, 3, 3, 1, 1, 2), "2,4,1,4,1,", "f32"),       # 32 filters x 256 pixels
    (S(25, 160, 33, 33, 24, 3, 3, 1, 1, 2), "1,4,1,4,1,", "f32"),      # 16 x 256
    (S(12, 64, 55, 55, 64, 3, 3, 1, 1, 4), "1,4,1,4,1,", "plain"),     # filters split in the kernel
    (S(200, 60, 31, 31, 36, 3, 3, 2, 1, 4), "1,2,1,4,1,", "plain"),    # 16 x 128
    (S(39, 33, 29, 29, 66, 3, 3, 1, 1, 3), "2,4,1,4,1,", "bf16"),
    (S(102, 68, 10, 10, 68, 3, 3, 1, 1, 1), "1,4,1,4,1,", "bf16"),
]


@pytest.mark.parametrize("s,block,form", FEW, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_blocks_epilogue_and_buffer_ends(gpu, s, block, form):
    """Residual and ReLU; tensors inside larger buffers of NaN: nothing outside is written or read into a result."""
    torch, b = gpu
    x, w = wl.make_input((s.N, s.Cin, s.H, s.W), 98), wl.make_weight(s.Cout, s.Cin // s.groups, 3, 3, 99)
    bf16 = form == "bf16"
    if bf16:
        x, w = wl.round_to_bf16(x)[1], wl.round_to_bf16(w)[1]
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    res = wl.make_input(ref.shape, 100)
    guard = 4096
    big = [torch.full((a.size + 2 * guard,), float("nan"), device="cuda", dtype=torch.bfloat16 if bf16 and a is x else torch.float32)
           for a in (x, res, res)]
    xd, rd, yd = (t[guard:guard + a.size] for t, a in zip(big, (x, res, res)))
    xd.copy_(torch.from_numpy(x).reshape(-1))
    rd.copy_(torch.from_numpy(res).reshape(-1))
    pw = b.gspc_pack_weights(torch.from_numpy(w).cuda(), s.groups, b.GSPC_BF16 if bf16 else b.GSPC_F32)
    layer = wl.Layer("conv", 0, 1, 2, s.N, s.Cin, s.H, s.W, s.Cout, 3, 3, s.stride, 1, s.groups, True, 0)
    b.gspc_run_layer_chain(b.LayerChain([layer], [pw], [xd.view(torch.int16) if bf16 else xd, rd, yd]))
    torch.cuda.synchronize()
    name = b.gspc_last_kernel()
    assert name.startswith("conv_split3<" + block) and form in name, name
    out = big[2].cpu().numpy()
    assert np.isnan(out[:guard]).all() and np.isnan(out[guard + res.size:]).all()
    y = out[guard:guard + res.size].reshape(res.shape).astype(np.float64)
    # (and the rounding of the sum with the residual)
    bound = (split_bound(9 * s.Cin // s.groups + 16) + 2.0 ** -24) * (absum + np.abs(res))
    assert (np.abs(y - oracle.relu(oracle.add(ref, res))) < bound).all()


@pytest.mark.parametrize("value", [np.inf, np.nan, np.finfo(np.float32).max])
@pytest.mark.parametrize("s,block,form", FEW[:4], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_blocks_of_values_that_do_not_split(gpu, s, block, form, value):
    """An infinity, NaN or largest number among inputs or weights: the plain sum, and no other output changes."""
    torch, b = gpu
    cpg, kpg = s.Cin // s.groups, s.Cout // s.groups
    x, w = wl.make_input((s.N, s.Cin, s.H, s.W), 101), wl.make_weight(s.Cout, cpg, 3, 3, 102)
    w[:, 3] = np.float32(0.5)                                   # lower parts are zero
    x[:, -1] = np.where(np.abs(x[:, -1]) < 0.01, np.float32(0.01), x[:, -1])
    x[0, 3, 0, 0] = x[s.N - 1, cpg + 3, s.H - 1, s.W - 1] = x[7, 3, 5, 6] = value
    # (the centre tap never meets the padding; a sixteenth of the largest number, so that no plain sum overflows)
    w[s.Cout - 1, cpg - 1, 1, 1] = value if not np.isfinite(value) else value / np.float32(16)
    y = b.gspc_conv2d_grouped(torch.from_numpy(x).cuda(), b.gspc_pack_weights(torch.from_numpy(w).cuda(), s.groups),
                              s.N, s.Cin, s.H, s.W, s.Cout, 3, 3, s.stride, 1, s.groups).cpu().numpy().astype(np.float64)
    name = b.gspc_last_kernel()
    assert name.startswith("conv_split3<" + block) and form in name, name
    with np.errstate(invalid="ignore"):
        ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
        assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isinf(y), np.isinf(ref))
        assert np.array_equal(np.sign(y[np.isinf(y)]), np.sign(ref[np.isinf(ref)]))
        ok = np.isfinite(ref)
        # (sums that are recomputed as plain ones round once per term)
        assert np.max(np.abs(y[ok] - ref[ok]) / absum[ok]) < 9 * cpg * 2.0 ** -24
        # those of the filters and images without such a value keep the split's bound
        calm = np.s_[1:7, :s.Cout - 1]
        assert np.max(np.abs(y[calm] - ref[calm]) / absum[calm]) < split_bound(9 * cpg + 16)


@pytest.mark.parametrize("s,form", [
    (S(18, 8, 65, 65, 226, 3, 3, 2, 1, 2), "f32,false,false>"),            # 4 channels, 113 filters
    (S(36, 24, 35, 35, 840, 3, 3, 2, 1, 8), "f32,false,false>"),           # 3 and 105
    (S(31, 2, 89, 89, 113, 3, 3, 1, 1, 1), "bf16,false,false>"),           # 2 and 113
    (S(156, 4, 65, 65, 28, 3, 3, 2, 1, 1), "bf16,false,false>"),           # 4 and 28
    (S(47, 12, 83, 83, 33, 3, 3, 1, 1, 3), "bf16,false,false>"),           # three groups of 4 and 11
    (S(33, 48, 12, 18, 208, 3, 3, 2, 1, 16), "f32,true,false>/plain"),     # 3 and 13, split in the kernel
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_few_channels(gpu, s, form):
    """Groups of 2 to 4 channels: three quarters and more of a unit of the reduction are zeros."""
    torch, b = gpu
    bf16 = form.startswith("bf16")
    y, x, w, name = run_conv(gpu, s, seed=103, dtype=b.GSPC_BF16 if bf16 else b.GSPC_F32)
    assert name.startswith("conv_split3<") and name.endswith(form), name
    if bf16:
        x, w = wl.round_to_bf16(x)[1], wl.round_to_bf16(w)[1]
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    assert err_metrics(y, ref, absum)["bound"] < split_bound(9 * s.Cin // s.groups + 16), name
