"""3x3 layers on the bf16 matrix instruction (fp32 through the exact three-way split, bf16 with channel counts the
16x16x32 section does not take), against the oracle's plain definition of the grouped convolution (Section II, Fig. 2)."""
import numpy as np
import pytest

import oracle
from helpers import err_metrics, rel_err
from paper_2006_09791_amd import workloads as wl
from test_gpu_parity import gpu, run_conv  # noqa: F401  (fixture)
from test_gpu_split import SCALES, scaled, split_bound

pytestmark = pytest.mark.gpu
S = wl.ConvShape
SHAPES = [
    # N Cin H W Cout KH KW stride pad groups
    (S(40, 128, 14, 14, 128, 3, 3, 1, 1, 1), "f32,true,true"),     # tiles that start inside rows and span images
    (S(24, 64, 28, 28, 128, 3, 3, 1, 1, 1), "f32,true,true"),      # whole float4 rows, 2x2 tiles that fill no block
    (S(150, 96, 7, 7, 64, 3, 3, 1, 1, 1), "f32,false,false"),       # 49-pixel planes: three images per tile, 4-byte stores
    (S(30, 66, 13, 17, 66, 3, 3, 1, 1, 1), "f32,false,false"),      # odd rows, padded channels and filters
    (S(33, 100, 9, 22, 128, 3, 3, 1, 1, 2), "f32,true,false"),     # two groups of 50 channels, even width, odd plane
    (S(64, 128, 8, 8, 128, 3, 3, 1, 1, 1), "f32,true,true"),       # the chunks split over four waves
    (S(160, 64, 16, 16, 128, 3, 3, 2, 1, 1), "f32,true,true"),     # stride 2, even planes
    (S(300, 70, 15, 9, 64, 3, 3, 2, 1, 1), "f32,false,false"),     # stride 2, odd planes (40 outputs each)
    (S(9, 49, 60, 50, 48, 3, 3, 1, 1, 1), "f32,true,true"),        # more staging tasks than slots; a last chunk of one channel
    (S(900, 64, 3, 2, 64, 3, 3, 1, 1, 1), "f32,true,false"),       # planes of six pixels: twenty images per tile
    (S(50, 36, 11, 13, 40, 3, 3, 1, 1, 1), "bf16,false,false"),     # bf16, 36 channels
    (S(40, 42, 12, 14, 48, 3, 3, 2, 1, 2), "bf16,true,false"),     # bf16, stride 2, two groups of 21
]


@pytest.mark.parametrize("s,kind", SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_split3(gpu, s, kind):
    torch, b = gpu
    bf16 = kind.startswith("bf16")
    y, x, w, name = run_conv(gpu, s, seed=71, dtype=b.GSPC_BF16 if bf16 else b.GSPC_F32)
    assert name.startswith("conv_split3<") and name.endswith(kind + ">"), name
    if bf16:
        x, w = wl.round_to_bf16(x)[1], wl.round_to_bf16(w)[1]
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    assert not np.isnan(y).any(), name
    m = err_metrics(y, ref, absum)
    # (the bound of the pointwise form for nine times the terms, a quarter of a k-step lost per 16 channels, and
    # four partial sums)
    assert m["bound"] < split_bound(9 * s.Cin // s.groups + 16) + 4 * 2.0 ** -24, (name, m)
    assert m["floored"] < 1e-5, (name, m)


@pytest.mark.parametrize("s,kernel", [
    (S(40, 46, 24, 24, 32, 3, 3, 1, 1, 2), "conv_mfma16<"),       # 23 channels, 16 filters: rows read four at a time
    (S(260, 46, 25, 24, 32, 3, 3, 2, 1, 2), "conv_mfma16<"),       # at stride 2
    (S(40, 50, 24, 24, 32, 3, 3, 1, 1, 2), "conv_split3<"),       # 25 channels
    (S(100, 46, 24, 22, 32, 3, 3, 1, 1, 2), "conv_split3<"),       # rows read one at a time
    (S(40, 22, 24, 24, 56, 3, 3, 1, 1, 2), "conv_mfma16<"),       # 11 channels, 28 filters
    (S(40, 22, 24, 24, 64, 3, 3, 1, 1, 2), "conv_split3<"),       # 32 filters
    (S(40, 26, 24, 24, 56, 3, 3, 1, 1, 2), "conv_split3<"),       # 13 channels
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_layers_of_few_filters(gpu, s, kernel):
    """Few filters per group, which would leave most of a 64-filter tile empty: the staged kernel, where it reads whole quads."""
    y, x, w, name = run_conv(gpu, s, seed=72)
    assert name.startswith(kernel), name
    ref, absum = oracle.conv2d_grouped(x, w, s.stride, 1, s.groups, return_abs=True, threads=8)
    m = err_metrics(y, ref, absum)
    # (split: as above; else a product and a sum per term, each rounded once at most)
    k = 9 * s.Cin // s.groups
    bound = split_bound(k + 16) + 4 * 2.0 ** -24 if name.startswith("conv_split3<") else (k + 17) * 2.0 ** -24
    assert m["bound"] < bound, (name, m)


@pytest.mark.parametrize("s", [S(40, 64, 14, 14, 72, 3, 3, 1, 1, 1), S(64, 128, 8, 8, 128, 3, 3, 1, 1, 1),
                               S(150, 67, 7, 9, 80, 3, 3, 1, 1, 1)], ids=lambda s: "x".join(map(str, s)))
def test_split3_epilogue_and_buffer_ends(gpu, s):
    """Residual and ReLU; tensors inside larger buffers of NaN: nothing outside is written or read into a result."""
    torch, b = gpu
    dev = torch.device("cuda:0")
    x, w = wl.make_input((s.N, s.Cin, s.H, s.W), 73), wl.make_weight(s.Cout, s.Cin, 3, 3, 74)
    res = wl.make_input((s.N, s.Cout, s.H, s.W), 75)
    guard = 4096
    big = [torch.full((a.size + 2 * guard,), float("nan"), device=dev) for a in (x, res, res)]
    xd, rd, yd = (t[guard:guard + a.size] for t, a in zip(big, (x, res, res)))
    xd.copy_(torch.from_numpy(x).reshape(-1))
    rd.copy_(torch.from_numpy(res).reshape(-1))
    pw = b.gspc_pack_weights(torch.from_numpy(w).to(dev), 1)
    layer = wl.Layer("conv", 0, 1, 2, s.N, s.Cin, s.H, s.W, s.Cout, 3, 3, 1, 1, 1, True, 0)
    b.gspc_run_layer_chain(b.LayerChain([layer], [pw], [xd, rd, yd]))
    torch.cuda.synchronize()
    assert b.gspc_last_kernel().startswith("conv_split3<"), b.gspc_last_kernel()
    out = big[2].cpu().numpy()
    assert np.isnan(out[:guard]).all() and np.isnan(out[guard + res.size:]).all()
    ref = oracle.relu(oracle.add(oracle.conv2d_grouped(x, w, 1, 1, 1, threads=8), res))
    assert rel_err(out[guard:guard + res.size].reshape(res.shape), ref) < 1e-5


@pytest.mark.parametrize("ex,ew", SCALES)
def test_split3_keeps_its_precision_in_either_operand(gpu, ex, ew):
    """bf16 has no bits below 2^-133: no factor whose lower parts would need them may lose precision."""
    torch, b = gpu
    dev = torch.device("cuda:0")
    N, C, hw = 60, 64, 14
    x, w = scaled(wl.make_input((N, C, hw, hw), 95), wl.make_weight(64, C, 3, 3, 96), ex, ew)
    x[:, :, 4:8, :] = 0.0
    x[:, 1:, :, 5:8] = 0.0
    pw = b.gspc_pack_weights(torch.from_numpy(w).to(dev), 1)
    y = b.gspc_conv2d_grouped(torch.from_numpy(x).to(dev), pw, N, C, hw, hw, 64, 3, 3, 1, 1, 1)
    torch.cuda.synchronize()
    assert b.gspc_last_kernel().startswith("conv_split3<"), b.gspc_last_kernel()
    y = y.cpu().numpy().astype(np.float64)
    ref, absum = oracle.conv2d_grouped(x, w, 1, 1, 1, return_abs=True, threads=8)
    assert np.isfinite(y).all()
    K = 9 * C
    assert np.max(np.abs(y - ref) - (split_bound(K) + (4 + K) * 2.0 ** -24) * absum) <= (K + 1) * 2.0 ** -150


@pytest.mark.parametrize("value", [np.inf, np.nan, np.finfo(np.float32).max, 1e-36])
def test_split3_of_values_that_do_not_split(gpu, value):
    """Infinities, values next to the largest one and (whole images of) tiny ones give the plain sum."""
    torch, b = gpu
    dev = torch.device("cuda:0")
    N, C, hw = 60, 64, 14
    x, w = wl.make_input((N, C, hw, hw), 83), wl.make_weight(64, C, 3, 3, 84)
    w[:, 3] = np.float32(0.5)                      # lower parts are zero
    if value == 1e-36:
        x[:20] = np.float32(1e-36) * x[:20]
    else:
        x[0, 3, 0, 0] = x[N - 1, 3, hw - 1, hw - 1] = x[7, 3, 5, 6] = value
    pw = b.gspc_pack_weights(torch.from_numpy(w).to(dev), 1)
    y = b.gspc_conv2d_grouped(torch.from_numpy(x).to(dev), pw, N, C, hw, hw, 64, 3, 3, 1, 1, 1)
    torch.cuda.synchronize()
    assert b.gspc_last_kernel().startswith("conv_split3<"), b.gspc_last_kernel()
    y = y.cpu().numpy().astype(np.float64)
    xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
    with np.errstate(invalid="ignore"):
        ref = sum(np.einsum("kc,nchw->nkhw", w[:, :, i, j].astype(np.float64), xp[:, :, i:i + hw, j:j + hw])
                  for i in range(3) for j in range(3))
        assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isinf(y), np.isinf(ref))
        assert np.array_equal(np.sign(y[np.isinf(y)]), np.sign(ref[np.isinf(ref)]))
    ok = np.isfinite(ref)
    scale = np.maximum(np.abs(ref), 1e-36 if value == 1e-36 else 1.0)
    scale[20:] = np.maximum(scale[20:], 1.0)
    assert np.max(np.abs(y[ok] - ref[ok]) / scale[ok]) < 1e-5
