"""Pointwise layers on the bf16 matrix instruction: fp32 layers through the exact three-way split, bf16
layers as they are, against the oracle's plain definition of the grouped convolution (Section II, Fig. 2)."""
import numpy as np
import pytest

import oracle
from helpers import err_metrics, rel_err
from paper_2006_09791_amd import workloads as wl
from test_gpu_parity import gpu, run_conv  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
S = wl.ConvShape


def split_bound(cpg):
    """|g - r| / sum |x*w|: three dropped products of at most 2^-25 each (both factors rounded to the
    nearest bf16 twice over), one rounding of the accumulators per instruction (six per 32 channels, taken at
    their full weight) and the final sum."""
    return (3 * 0.5 + 6 * ((cpg + 31) // 32) + 2) * 2.0 ** -24


SHAPES = [
    # N Cin H W Cout KH KW stride pad groups
    (S(420, 40, 8, 8, 240, 1, 1, 1, 0, 1), "4,2,2,4"),     # the last filter tile of the second block empty; a quarter of a chunk
    (S(561, 33, 7, 7, 128, 1, 1, 1, 0, 1), "4,2,2,4"),     # 49-pixel planes: 4-byte loads and stores, ragged last tile
    (S(64, 64, 28, 28, 64, 1, 1, 1, 0, 1), "4,2,1,4"),     # 64-filter blocks, 16-byte stores
    (S(100, 31, 23, 31, 50, 1, 1, 1, 0, 1), "4,2,1,4"),    # odd plane, padded filters and channels
    (S(64, 96, 28, 28, 24, 1, 1, 1, 0, 1), "2,2,1,4"),     # fewer filters than a block
    (S(65, 48, 14, 14, 64, 1, 1, 1, 0, 2), "2,2,1,"),      # two groups of 24 channels and 32 filters
    (S(200, 144, 12, 12, 160, 1, 1, 1, 0, 1), "4,2,1,4"),  # filters split at packing time in 64-filter blocks
    (S(165, 160, 13, 13, 130, 1, 1, 1, 0, 1), "4,2,1,4"),  # the same on odd planes
    (S(8, 128, 14, 14, 512, 1, 1, 1, 0, 1), "2,2,1,2"),    # the smallest blocks
    (S(1, 250, 9, 11, 77, 1, 1, 1, 0, 1), "2,2,1,2"),      # bf16, no other matrix-core kernel takes it: any size
    (S(4000, 24, 1, 1, 200, 1, 1, 1, 0, 1), "2,2,1,"),     # planes of one pixel
]


@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("s,shape", SHAPES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_pointwise_split(gpu, s, shape, bf16):
    torch, b = gpu
    if s.N == 1 and not bf16:
        pytest.skip("a small fp32 launch: the kernel without staging (test_gpu_unit.py)")
    y, x, w, name = run_conv(gpu, s, seed=51, dtype=b.GSPC_BF16 if bf16 else b.GSPC_F32)
    # last template argument: the filters were split when they were packed
    form = ("bf16,", "true>") if bf16 else ("f32,", "true>" if s.Cin * s.Cout > 16384 else "false>")
    assert name.startswith("conv_mfma16s<" + shape) and form[0] in name and name.endswith(form[1]), name
    if bf16:
        x, w = wl.round_to_bf16(x)[1], wl.round_to_bf16(w)[1]
    ref, absum = oracle.conv2d_grouped(x, w, 1, 0, s.groups, return_abs=True, threads=8)
    assert not np.isnan(y).any(), name
    m = err_metrics(y, ref, absum)
    assert m["bound"] < split_bound(s.Cin // s.groups), (name, m)
    assert m["floored"] < 1e-5, (name, m)


@pytest.mark.parametrize("s,kernel", [
    (S(80, 32, 28, 28, 64, 1, 1, 1, 0, 4), "conv_mfma16<"),       # 8 channels, 16 filters per group, 250880 pixels times groups
    (S(80, 48, 28, 28, 64, 1, 1, 1, 0, 4), "conv_mfma16<"),       # 12 channels
    (S(79, 48, 28, 28, 64, 1, 1, 1, 0, 4), "conv_mfma16s<"),      # 247744
    (S(80, 52, 28, 28, 64, 1, 1, 1, 0, 4), "conv_mfma16s<"),      # 13 channels
    (S(80, 48, 28, 28, 68, 1, 1, 1, 0, 4), "conv_mfma16s<"),      # 17 filters
    (S(90, 48, 27, 27, 64, 1, 1, 1, 0, 4), "conv_mfma16s<"),      # planes that are no whole quads
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else v)
def test_layers_of_one_filter_tile(gpu, s, kernel):
    """One filter tile and few channels per group: the staged kernel, from the launch size on where it is ahead."""
    y, x, w, name = run_conv(gpu, s, seed=57)
    assert name.startswith(kernel), name
    ref, absum = oracle.conv2d_grouped(x, w, 1, 0, s.groups, return_abs=True, threads=8)
    cpg = s.Cin // s.groups
    bound = split_bound(cpg) if kernel == "conv_mfma16s<" else (cpg + 17) * 2.0 ** -24
    assert err_metrics(y, ref, absum)["bound"] < bound, name


@pytest.mark.parametrize("hw,cout", [(28, 64), (27, 40)])
def test_pointwise_split_epilogue_and_buffer_ends(gpu, hw, cout):
    """Residual and ReLU; nothing outside the output tensor is written (odd planes: 4-byte stores)."""
    torch, b = gpu
    dev = torch.device("cuda:0")
    N, cin = 70, 40
    x, w = wl.make_input((N, cin, hw, hw), 71), wl.make_weight(cout, cin, 1, 1, 72)
    res = wl.make_input((N, cout, hw, hw), 73)
    pw = b.gspc_pack_weights(torch.from_numpy(w).to(dev), 1)
    guard = 4096
    yd = torch.full((res.size + 2 * guard,), float("nan"), device=dev)
    layer = wl.Layer("conv", 0, 1, 2, N, cin, hw, hw, cout, 1, 1, 1, 0, 1, True, 0)
    b.gspc_run_layer_chain(b.LayerChain([layer], [pw], [torch.from_numpy(x).to(dev).reshape(-1),
                                                        torch.from_numpy(res).to(dev).reshape(-1),
                                                        yd[guard:guard + res.size]]))
    torch.cuda.synchronize()
    assert b.gspc_last_kernel().startswith("conv_mfma16s<"), b.gspc_last_kernel()
    out = yd.cpu().numpy()
    assert np.isnan(out[:guard]).all() and np.isnan(out[guard + res.size:]).all()
    ref = oracle.relu(oracle.add(oracle.conv2d_grouped(x, w, 1, 0, 1, threads=8), res))
    assert rel_err(out[guard:guard + res.size].reshape(res.shape), ref) < 1e-5


@pytest.mark.parametrize("exponent", [-126, -118, -105, 100])
def test_pointwise_split_keeps_its_precision_at_any_scale(gpu, exponent):
    """bf16 has no bits below 2^-133: inputs whose lower parts would need them must not lose precision."""
    torch, b = gpu
    dev = torch.device("cuda:0")
    x, w = wl.make_input((150, 32, 16, 16), 91), wl.make_weight(64, 32, 1, 1, 92)
    x = np.ldexp(np.where(np.abs(x) < 0.01, 0.01, x), exponent).astype(np.float32)
    pw = b.gspc_pack_weights(torch.from_numpy(w).to(dev), 1)
    y = b.gspc_conv2d_grouped(torch.from_numpy(x).to(dev), pw, 150, 32, 16, 16, 64, 1, 1, 1, 0, 1)
    torch.cuda.synchronize()
    assert b.gspc_last_kernel().startswith("conv_mfma16s<"), b.gspc_last_kernel()
    y = y.cpu().numpy().astype(np.float64)
    ref, absum = oracle.conv2d_grouped(x, w, 1, 0, 1, return_abs=True, threads=8)
    # (plus half a unit of the smallest denormal per product and for the result)
    assert np.max(np.abs(y - ref) - (split_bound(32) + 32 * 2.0 ** -24) * absum) <= 33 * 2.0 ** -150


# Exponents of inputs and weights: operands with fewer than 24 bits above bf16's 2^-133 against a second factor that
# makes the result an ordinary number; results below fp32's normal range; products near the largest number.
SCALES = [(-120, 45), (45, -120), (-126, 60), (-140, 99), (99, -140), (-60, -70), (-100, 100), (60, 60)]


def scaled(x, w, ex, ew):
    """The operands, none of them next to zero, at these exponents."""
    x = np.ldexp(np.where(np.abs(x) < 0.01, 0.01, x).astype(np.float64), ex)
    w = np.ldexp(np.where(np.abs(w) < 0.01, 0.01, w).astype(np.float64), ew)
    return x.astype(np.float32), w.astype(np.float32)


@pytest.mark.parametrize("ex,ew", SCALES)
@pytest.mark.parametrize("cin,cout", [(32, 64), (160, 128)], ids=["words", "parts"])
def test_pointwise_split_keeps_its_precision_in_either_operand(gpu, ex, ew, cin, cout):
    torch, b = gpu
    dev = torch.device("cuda:0")
    N, hw = 150, 16
    x, w = scaled(wl.make_input((N, cin, hw, hw), 93), wl.make_weight(cout, cin, 1, 1, 94), ex, ew)
    x[:, :, 3, :] = 0.0                       # sums of zeros stay zeros
    x[:, 1:, 5, 5] = 0.0                      # sums of one term
    pw = b.gspc_pack_weights(torch.from_numpy(w).to(dev), 1)
    y = b.gspc_conv2d_grouped(torch.from_numpy(x).to(dev), pw, N, cin, hw, hw, cout, 1, 1, 1, 0, 1)
    torch.cuda.synchronize()
    name = b.gspc_last_kernel()
    assert name.startswith("conv_mfma16s<") and name.endswith("true>" if cin * cout > 16384 else "false>"), name
    y = y.cpu().numpy().astype(np.float64)
    ref, absum = oracle.conv2d_grouped(x, w, 1, 0, 1, return_abs=True, threads=8)
    assert np.isfinite(y).all()
    # (plus half a unit of the smallest denormal per product and for the result)
    assert np.max(np.abs(y - ref) - (split_bound(cin) + cin * 2.0 ** -24) * absum) <= (cin + 1) * 2.0 ** -150


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, np.finfo(np.float32).max])
@pytest.mark.parametrize("hw,cout", [(16, 128), (15, 128), (16, 512)])
def test_pointwise_split_of_values_that_do_not_split(gpu, value, hw, cout):
    """An infinity times a zero part, or a part that overflows, must not show: results are those of the plain sum."""
    torch, b = gpu
    dev = torch.device("cuda:0")
    N, cin = 300, 36
    x, w = wl.make_input((N, cin, hw, hw), 81), wl.make_weight(cout, cin, 1, 1, 82)
    w[:, 3] = np.float32(0.5) + (np.arange(cout)[:, None, None] % 3) * np.float32(0.125)   # lower parts are zero
    x[0, 3, 0, 0] = x[N - 1, 3, hw - 1, hw - 1] = x[7, 3, 5, 6] = value
    pw = b.gspc_pack_weights(torch.from_numpy(w).to(dev), 1)
    y = b.gspc_conv2d_grouped(torch.from_numpy(x).to(dev), pw, N, cin, hw, hw, cout, 1, 1, 1, 0, 1)
    torch.cuda.synchronize()
    assert b.gspc_last_kernel().startswith("conv_mfma16s<"), b.gspc_last_kernel()
    y = y.cpu().numpy().astype(np.float64)
    ref = np.einsum("kc,nchw->nkhw", w[:, :, 0, 0].astype(np.float64), x.astype(np.float64))
    with np.errstate(invalid="ignore"):
        assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isinf(y), np.isinf(ref))
        assert np.array_equal(np.sign(y[np.isinf(y)]), np.sign(ref[np.isinf(ref)]))
    ok = np.isfinite(ref)
    assert np.max(np.abs(y[ok] - ref[ok]) / np.maximum(np.abs(ref[ok]), 1.0)) < 1e-5
