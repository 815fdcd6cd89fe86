"""Roofline figures of the benchmark line: kernels that execute another number of multiplications than Eq. 2
(Section IV-B) counts are held against the instruction that executes them."""
import pytest

import bench
from paper_2006_09791_amd import layer_timing


@pytest.mark.parametrize("kernel,executed,peak", [
    ("conv_mfma16<4,2,2,4,1,1,1,f32,true>", 1.0, 157.3),
    ("conv_mfma16u<8,3,1>", 1.0, 157.3),
    ("conv_mfma16w<1,2,2,2,false,8,f32>", 1.0, 157.3),
    ("conv_wino<1,1,1,1,2,true>", 16.0 / 36.0, 157.3),
    ("conv_mfma16s<4,2,2,4,f32,true,true>", 6.0, 2500.0),
    ("conv_split3<2,4,2,2,1,4,1,f32,true,true>", 6.0, 2500.0),
])
def test_roofline_of_executed_work(kernel, executed, peak):
    assert layer_timing.executed_work(kernel)[1:] == (executed, peak)
    flops, nbytes = 52.6e9, 310e6
    assert bench.compute_bound(kernel, flops, nbytes)
    k = {"time": 280e-6, "flops": flops, "bytes": nbytes, "launches": 1, "compute_bound": True}
    r = bench._roofline_object(kernel, k, {kernel: k})
    assert r["bound"] == "mfma" and r["peak"] == peak
    assert r["achieved"] == pytest.approx(flops / 280e-6 / 1e12 * executed, rel=1e-3)
    assert r["frac"] == pytest.approx(r["achieved"] / peak, abs=1e-4)
    assert ("eq2_effective_tflops" in r) == (executed != 1.0)


def test_bf16_layers_of_the_split_kernels_execute_what_eq2_counts():
    for kernel in ("conv_mfma16s<4,2,2,4,bf16,true,true>", "conv_split3<2,4,2,2,1,4,1,bf16,true,true>"):
        assert layer_timing.executed_work(kernel, "bf16") == (None, 1.0, 2500.0)


def test_ridge_of_the_split_kernels():
    assert bench.compute_bound("conv_mfma16<1,1,1,4,1,1,1,f32,true>", 40.0, 1.0)
    assert not bench.compute_bound("conv_mfma16s<2,2,1,4,f32,true,false>", 40.0, 1.0)
