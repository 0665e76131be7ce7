"""conv_rows_kernel (Forward of layers with few input channels, reductions along the rows of the filter): strides 1 to 4 and rows and
columns apart, odd and even paddings, filter rows of one to three quads, one to five row tiles, 32, 64 and 96 output
channels per tile and fewer, column blocks, tiles over several images, fp32 and bf16, values out of the split's range, equal
bits in every run, layers that it does not take.

Bounds: fp32 sums of split products are off by 1e-7 to 4e-7 of the result (11x11 filters), held to 1e-6; bf16 as in test_gpu_bf16.py."""
import numpy as np
import pytest

from paper_1804_04806_amd import ucd
from hip_helpers import check_specials, desc_of, inputs, not_finite_time_ratio, rect, rel_l2, run_hip, run_oracle, run_oracle_zeros
from test_gpu_bf16 import bf16_inputs, check_bf16_output, run_hip_bf16

pytestmark = pytest.mark.gpu

D, I = ucd.FWD, ucd.ALGO_IMPLICIT

# (n, c, h, w, k, r, s, strides, pads)
LAYERS = [rect(17, 3, 224, 227, 62, 7, 7, (2, 2), (3, 3)), rect(280, 3, 61, 59, 94, 7, 7, (2, 2), (0, 0)), rect(7, 1, 257, 131, 30, 11, 11, (1, 1), (5, 5)),
          rect(22, 2, 70, 140, 128, 5, 8, (1, 2), (2, 2)), rect(54, 3, 100, 121, 61, 7, 7, (3, 1), (2, 2)), rect(56, 4, 110, 200, 64, 6, 7, (2, 3), (5, 0)),
          rect(4200, 3, 7, 7, 63, 7, 7, (1, 1), (3, 3)), rect(2, 3, 150, 800, 60, 7, 7, (1, 1), (3, 3)), rect(66, 1, 227, 231, 64, 11, 11, (4, 4), (0, 2)),
          rect(12, 4, 61, 63, 320, 7, 7, (1, 1), (3, 3))]
LONG = [rect(45, 3, 224, 227, 62, 7, 7, (2, 2), (3, 3)), rect(17, 1, 257, 131, 30, 11, 11, (1, 1), (5, 5)), rect(140, 3, 100, 121, 61, 7, 7, (3, 1), (2, 2)),
        rect(11000, 3, 7, 7, 63, 7, 7, (1, 1), (3, 3))]


def described(s, dtype):
    return ucd.ucd_describe_micro(desc_of(s, dtype=dtype), D, I, s.N)[0]


@pytest.mark.parametrize("s", LAYERS, ids=str)
def test_few_channels(s):
    assert "conv_rows_kernel" in described(s, 0)
    x, w, _ = inputs(s, seed=91)
    ref = run_oracle(s, D, x=x, w=w)
    assert rel_l2(run_hip(s, D, [(I, s.N)], x=x, w=w), ref) <= 1e-6
    got = run_hip(s, D, [(I, s.N - 1), (I, 1)], x=x, w=w)
    assert rel_l2(got, ref) <= 1e-6 and np.abs(got - ref).max() <= 1e-4 * np.sqrt(np.mean(ref ** 2))


@pytest.mark.parametrize("s", LONG, ids=str)
def test_few_channels_bf16(s):
    assert "conv_rows_kernel" in described(s, 1)
    bits, (x, w, dy) = bf16_inputs(s, seed=92)
    ref = run_oracle(s, D, x=x, w=w, dy=dy)
    for parts in ([s.N], [1, s.N - 1]):
        check_bf16_output(run_hip_bf16(s, D, [(I, b) for b in parts], bits), ref, (s, parts))


def test_few_channels_equal_bits():
    s = LAYERS[0]
    x, w, _ = inputs(s, seed=93)
    first = run_hip(s, D, [(I, s.N)], x=x, w=w)
    assert all(np.array_equal(first, run_hip(s, D, [(I, s.N)], x=x, w=w)) for _ in range(3))


@pytest.mark.parametrize("s", [LAYERS[0], LAYERS[6]], ids=str)
@pytest.mark.parametrize("scale", [2.0 ** -110, 2.0 ** -60, 2.0 ** 60])
def test_few_channels_out_of_range(s, scale):
    """Filters below bf16's range and products near the ends of fp32's, which the fp32 instructions compute."""
    x, w, _ = inputs(s, seed=94)
    w = (w * np.float32(scale)).astype(np.float32)
    ref = run_oracle(s, D, x=x, w=w)
    assert rel_l2(run_hip(s, D, [(I, s.N)], x=x, w=w) / scale, ref / scale) <= 2e-6


@pytest.mark.parametrize("dtype, s", [(0, LAYERS[0]), (0, LAYERS[4]), (0, LAYERS[6]), (1, LONG[0]), (1, LONG[2])], ids=str)
def test_few_channels_not_finite(dtype, s):
    """Infinities and NaN come out where, and as, fp32 arithmetic gives them, and not at pixels whose taps end beside them; the others stay exact."""
    bits, (x, w, _) = bf16_inputs(s, seed=95)
    for at, v in (((0, -1, 1, 1), 0xFF80), ((-1, 0, -1, -1), 0x7FC0), ((3, 0, 5, 0), 0x7F80), ((2, 0, 6, -1), 0x7F80)):
        bits[0][at] = v
    x = (bits[0].astype(np.uint32) << 16).view(np.float32)
    got = (run_hip(s, D, [(I, s.N)], x=x, w=w) if dtype == 0 else run_hip_bf16(s, D, [(I, s.N)], bits)).astype(np.float64)
    ref = run_oracle(s, D, x=x, w=w)
    fine = np.isfinite(ref)
    assert fine.any() and not fine.all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert rel_l2(got[fine], ref[fine]) <= (5e-3 if dtype else 1e-6)


@pytest.mark.parametrize("dtype, s", [(0, LAYERS[0]), (0, LAYERS[2]), (0, LAYERS[3]), (0, LAYERS[9]), (1, LONG[0]), (1, LONG[1])], ids=str)
def test_few_channels_filter_not_finite(dtype, s):
    """The same of the filter, first and last taps beside the padding among them, together with infinities of x."""
    bits, (x, w, _) = bf16_inputs(s, seed=96)
    for at, v in (((0, 0, 0, 0), 0x7F80), ((-1, -1, -1, -1), 0x7FC0), ((4, 0, 2, 1), 0xFF80), ((4, -1, -1, 2), 0x7F80)):
        bits[1][at] = v
    bits[0][1, 0, 3, 4], bits[0][-1, -1, -2, 0] = 0x7F80, 0xFF80
    x, w = ((t.astype(np.uint32) << 16).view(np.float32) for t in bits[:2])
    got = (run_hip(s, D, [(I, s.N)], x=x, w=w) if dtype == 0 else run_hip_bf16(s, D, [(I, s.N)], bits)).astype(np.float64)
    check_specials(got, run_oracle_zeros(s, D, x=x, w=w), 5e-3 if dtype else 1e-6)


@pytest.mark.parametrize("dtype, s", [(0, LAYERS[0]), (0, LAYERS[2]), (0, LAYERS[4]), (1, LONG[0])], ids=str)
def test_few_channels_not_finite_time(dtype, s):
    """Every tile of such tensors is multiplied a second time, in fp32 on the fp32 instructions: 1.7 to 3.1 times the ordinary time, not the 50 to
    120 of sums taken tap by tap."""
    assert not_finite_time_ratio(s, D, dtype) < 6


@pytest.mark.parametrize("dtype, s", [(0, rect(9, 3, 145, 161, 64, 7, 7, (2, 2), (3, 3))), (0, rect(120, 3, 64, 64, 64, 3, 3, (1, 1), (1, 1))),
                                      (0, rect(64, 17, 112, 112, 64, 7, 7, (2, 2), (3, 3))), (0, rect(64, 3, 112, 112, 40, 7, 7, (2, 2), (3, 3))),
                                      (1, LAYERS[0]), (0, rect(256, 3, 227, 227, 96, 11, 11, (4, 4), (0, 0)))], ids=str)
def test_layers_that_it_does_not_take(dtype, s):
    assert "conv_rows_kernel" not in described(s, dtype)
