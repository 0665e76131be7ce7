"""conv_few_kernel (BackwardData of layers with few input channels, blocks of pixels as the rows of a tile): strides 1 to 4 and rows and
columns apart, blocks of one to eight strides, taps in one and in several steps and an odd number of them, output channels that are no
whole chunk of eight, column blocks, tiles over several images, pixels that no tap reaches, fp32 and bf16, values out of the split's
range, equal bits in every run, layers that it does not take.

Bounds: fp32 sums of split products are off by 1e-7 to 4e-7 of the result (11x11 filters), held to 1e-6; bf16 as in test_gpu_bf16.py."""
import numpy as np
import pytest

from paper_1804_04806_amd import ucd
from hip_helpers import check_specials, desc_of, inputs, not_finite_time_ratio, rect, rel_l2, run_hip, run_oracle, run_oracle_zeros
from test_gpu_bf16 import bf16_inputs, check_bf16_output, run_hip_bf16

pytestmark = pytest.mark.gpu

D, I = ucd.BWD_DATA, ucd.ALGO_IMPLICIT

# (n, c, h, w, k, r, s, strides, pads)
STRIDED = [rect(9, 3, 45, 61, 37, 7, 7, (2, 2), (3, 3)), rect(30, 3, 30, 29, 50, 7, 7, (2, 2), (0, 0)), rect(40, 1, 33, 34, 51, 11, 11, (4, 4), (0, 2)),
           rect(12, 2, 40, 130, 60, 5, 5, (2, 2), (2, 1)), rect(70, 4, 23, 21, 49, 3, 3, (2, 2), (1, 1)), rect(25, 8, 26, 27, 63, 7, 5, (2, 2), (0, 1)),
           rect(16, 3, 38, 40, 55, 7, 5, (3, 1), (2, 2)), rect(16, 5, 36, 41, 48, 4, 7, (1, 2), (1, 3)), rect(3, 1, 150, 200, 52, 6, 6, (2, 3), (5, 0)),
           rect(90, 2, 40, 39, 57, 13, 15, (4, 4), (3, 3)), rect(1400, 7, 9, 8, 65, 5, 5, (2, 2), (2, 2)), rect(60, 3, 113, 114, 17, 7, 7, (2, 2), (3, 3)),
           rect(60, 2, 110, 115, 53, 7, 7, (2, 2), (2, 3))]
PLAIN = [rect(24, 3, 112, 113, 21, 7, 7, (1, 1), (3, 3)), rect(140, 16, 25, 23, 33, 3, 3, (1, 1), (1, 1)), rect(60, 1, 60, 130, 18, 5, 4, (1, 1), (0, 3)),
         rect(100, 3, 44, 40, 19, 11, 11, (1, 1), (5, 5)), rect(500, 9, 13, 12, 40, 3, 5, (1, 1), (2, 2)), rect(33, 2, 64, 300, 17, 3, 3, (1, 1), (1, 0))]


def described(s, dtype):
    return ucd.ucd_describe_micro(desc_of(s, dtype=dtype), D, I, s.N)[0]


@pytest.mark.parametrize("s", STRIDED + PLAIN, ids=str)
def test_few_channels(s):
    assert "conv_few_kernel" in described(s, 0)
    _, w, dy = inputs(s, seed=81)
    ref = run_oracle(s, D, w=w, dy=dy)
    assert rel_l2(run_hip(s, D, [(I, s.N)], w=w, dy=dy), ref) <= 1e-6
    got = run_hip(s, D, [(I, s.N - 1), (I, 1)], w=w, dy=dy)
    assert rel_l2(got, ref) <= 1e-6 and np.abs(got - ref).max() <= 1e-4 * np.sqrt(np.mean(ref ** 2))


@pytest.mark.parametrize("s", STRIDED + PLAIN[:1] + PLAIN[2:4], ids=str)
def test_few_channels_bf16(s):
    assert "conv_few_kernel" in described(s, 1)
    bits, (x, w, dy) = bf16_inputs(s, seed=82)
    ref = run_oracle(s, D, x=x, w=w, dy=dy)
    for parts in ([s.N], [1, s.N - 1]):
        check_bf16_output(run_hip_bf16(s, D, [(I, b) for b in parts], bits), ref, (s, parts))


def test_few_channels_equal_bits():
    s = STRIDED[0]
    _, w, dy = inputs(s, seed=83)
    first = run_hip(s, D, [(I, s.N)], w=w, dy=dy)
    assert all(np.array_equal(first, run_hip(s, D, [(I, s.N)], w=w, dy=dy)) for _ in range(3))


@pytest.mark.parametrize("scale", [2.0 ** -110, 2.0 ** -60, 2.0 ** 60])
def test_few_channels_out_of_range(scale):
    """Filters below bf16's range and products near the ends of fp32's, which the fp32 instructions compute."""
    s = STRIDED[0]
    _, w, dy = inputs(s, seed=84)
    w = (w * np.float32(scale)).astype(np.float32)
    ref = run_oracle(s, D, w=w, dy=dy)
    assert rel_l2(run_hip(s, D, [(I, s.N)], w=w, dy=dy) / scale, ref / scale) <= 2e-6


@pytest.mark.parametrize("s", [STRIDED[0], STRIDED[-1], PLAIN[0], PLAIN[4]], ids=str)
@pytest.mark.parametrize("dtype", [0, 1])
def test_few_channels_not_finite(s, dtype):
    """Infinities and NaN come out where, and as, fp32 arithmetic gives them, and not at pixels of the same block; the others stay exact."""
    bits, (_, w, dy) = bf16_inputs(s, seed=85)
    for at, v in (((0, -1, 1, 1), 0xFF80), ((-1, 0, -1, -1), 0x7FC0), ((3, 2, 5, 0), 0x7F80)):
        bits[2][at] = v
    dy = (bits[2].astype(np.uint32) << 16).view(np.float32)
    got = (run_hip(s, D, [(I, s.N)], w=w, dy=dy) if dtype == 0 else run_hip_bf16(s, D, [(I, s.N)], bits)).astype(np.float64)
    ref = run_oracle(s, D, w=w, dy=dy)
    fine = np.isfinite(ref)
    assert fine.any() and not fine.all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert rel_l2(got[fine], ref[fine]) <= (5e-3 if dtype else 1e-6)


@pytest.mark.parametrize("s", [STRIDED[0], STRIDED[2], STRIDED[7], STRIDED[-1], PLAIN[0], PLAIN[4]], ids=str)
@pytest.mark.parametrize("dtype", [0, 1])
def test_few_channels_filter_not_finite(s, dtype):
    """The same of the filter, first and last taps among them, together with infinities of dy that meet each other and the filter's."""
    bits, (_, w, dy) = bf16_inputs(s, seed=86)
    for at, v in (((0, 0, 0, 0), 0x7F80), ((-1, -1, -1, -1), 0x7FC0), ((3, 0, 2, 1), 0xFF80)):
        bits[1][at] = v
    for at, v in (((1, 0, 1, 1), 0x7F80), ((1, 1, 1, 2), 0xFF80), ((2, 3, -1, -1), 0x7F80), ((2, 0, 4, 4), 0x7FC0)):
        bits[2][at] = v
    w, dy = ((t.astype(np.uint32) << 16).view(np.float32) for t in bits[1:])
    got = (run_hip(s, D, [(I, s.N)], w=w, dy=dy) if dtype == 0 else run_hip_bf16(s, D, [(I, s.N)], bits)).astype(np.float64)
    check_specials(got, run_oracle_zeros(s, D, w=w, dy=dy), 5e-3 if dtype else 1e-6)


@pytest.mark.parametrize("s, dtype", [(STRIDED[-1], 0), (STRIDED[-1], 1), (PLAIN[0], 0), (PLAIN[0], 1), (STRIDED[1], 0)], ids=str)
def test_few_channels_not_finite_time(s, dtype):
    """Every tile of such tensors is computed once more, with two passes that find its infinities: 4 to 7 times the ordinary time, not the 16 to
    80 of sums taken tap by tap."""
    assert not_finite_time_ratio(s, D, dtype) < 10


@pytest.mark.parametrize("s", [rect(9, 17, 45, 61, 37, 7, 7, (2, 2), (3, 3)), rect(9, 3, 45, 61, 37, 1, 7, (2, 2), (0, 3)),
                               rect(9, 3, 45, 61, 37, 1, 1, (1, 1), (0, 0)), rect(4, 3, 30, 31, 200, 7, 7, (1, 1), (3, 3)), rect(48, 5, 136, 248, 35, 2, 2, (2, 2), (1, 1)),
                               rect(90, 2, 17, 16, 57, 9, 8, (4, 4), (3, 3)), rect(12, 1, 214, 214, 1, 11, 11, (1, 1), (5, 5))], ids=str)
def test_layers_that_it_does_not_take(s):
    assert "conv_few_kernel" not in described(s, 0)
