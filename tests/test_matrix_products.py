"""What a pass multiplies with: the library's answer (host code) over the workloads' layers, and bench.py's use of it."""
import pytest

import bench
import paper_1412_6249_amd as pa
from synth.configs import CONV_LAYERS

FWD, BWD_DATA, BWD_WEIGHT, BWD_WEIGHT_BIAS = range(4)


def _products(layer, which):
    dt = pa.PURINE_F32 if layer.dtype == "f32" else pa.PURINE_BF16
    return pa.purine_conv_matrix_products(which, pa.conv_desc(layer.stride, layer.pad), layer.x_shape, layer.w_shape, dt)


@pytest.mark.parametrize("cfg, name, want", [
    (3, "b3_5x5", (1, 6)),             # backward-data has 16 rows: fp32 kernels; the weight gradient's operands are laid out in LDS as parts
    (3, "b2_3x3", (6, 6)),
    (4, "conv2", (6, 6)), (4, "conv4", (6, 6)),
    (4, "conv1", (1, 6)),              # three channels: likewise
    (2, "cccp1", (1, 1)), (5, "c3x3", (1, 1))])
def test_gradients_of_the_workloads(cfg, name, want):
    layer = next(l for l in CONV_LAYERS[cfg] if l.name == name)
    assert (_products(layer, BWD_DATA), _products(layer, BWD_WEIGHT)) == want
    assert _products(layer, BWD_WEIGHT_BIAS) == want[1]


def test_forward_passes_of_long_sums_depend_on_the_launch():
    """More than 2048 products per output: fp32 products, but not in a launch of few tiles."""
    d = pa.conv_desc(1, 1)
    f = lambda n, c: pa.purine_conv_matrix_products(FWD, d, (n, c, 13, 13), (384, c, 3, 3), pa.PURINE_F32)
    assert (f(128, 384), f(2, 384), f(128, 227), f(128, 228)) == (1, 6, 6, 1)


@pytest.mark.parametrize("n, c, hw, k, stride, want", [
    (8, 128, 28, 128, 1, (6, 6)), (64, 256, 27, 256, 1, (6, 6)), (64, 96, 54, 96, 1, (1, 1)),
    (18, 555, 27, 575, 1, (1, 1)),       # many row tiles, one workgroup per CU: slower on parts
    (13, 32, 46, 97, 1, (1, 6)),         # two groups of channels forward
    (30, 251, 60, 189, 2, (1, 1)),
    (5, 60, 17, 29, 2, (6, 6))])         # backward: a small launch
def test_1x1_layers(n, c, hw, k, stride, want):
    d = pa.conv_desc(stride, 0)
    assert tuple(pa.purine_conv_matrix_products(p, d, (n, c, hw, hw), (k, c, 1, 1), pa.PURINE_F32) for p in (FWD, BWD_DATA)) == want


@pytest.mark.parametrize("n, c, h, w, k, r, pad, want", [
    (2, 38, 8, 9, 42, 3, 1, [6, 6, 6, 6]),       # forward and backward-data in the kernel of small launches, the weight gradient's operands laid out in LDS
    (1, 272, 26, 26, 126, 1, 0, [6, 6, 6, 6]),
    (1, 64, 56, 56, 64, 3, 1, [6, 6, 1, 1])])    # the general weight gradient
def test_small_launches_multiply_parts_in_fp32_alone(n, c, h, w, k, r, pad, want):
    f = lambda dt: [pa.purine_conv_matrix_products(p, pa.conv_desc(1, pad), (n, c, h, w), (k, c, r, r), dt) for p in range(4)]
    assert f(pa.PURINE_F32) == want and f(pa.PURINE_BF16) == [1] * 4


def test_illegal_shapes_and_passes_give_zero():
    d = pa.conv_desc(1, 0)
    assert pa.purine_conv_matrix_products(FWD, d, (1, 3, 2, 2), (4, 3, 3, 3), pa.PURINE_F32) == 0
    assert pa.purine_conv_matrix_products(4, d, (1, 16, 8, 8), (16, 16, 3, 3), pa.PURINE_F32) == 0
    assert pa.purine_conv_matrix_products(FWD, d, (1, 16, 8, 8), (16, 16, 3, 3), pa.PURINE_I32) == 0


def test_bench_prices_a_pass_by_the_kernel_that_runs():
    for cfg, layers in CONV_LAYERS.items():
        for l in layers:
            for kind, which in ((0, FWD), (13, FWD), (2, BWD_DATA), (14, BWD_DATA), (3, BWD_WEIGHT), (15, BWD_WEIGHT)):
                n = _products(l, which)
                assert bench.products(l, kind) == n, (cfg, l.name, kind)
                assert bench.mfma_peak(l, kind) == (2500.0 / 6 if n == 6 else bench.PEAK_TFLOPS[l.dtype])
