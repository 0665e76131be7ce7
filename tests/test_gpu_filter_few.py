"""filter_few_kernel (BackwardFilter of layers with few input channels, all filter elements of a block of channels at once): strides 1 to 4 and
rows and columns apart, odd and even taps, rows of dy that end inside a group of eight pixels, channels in one and in several
blocks, 32 and 64 output channels per tile and fewer, blocks of columns, tiles over several images, accumulation, values out of the split's
range and values that are not finite, layers that it does not take.

Bounds: fp32 sums of split products over up to 1e6 pixels, added in any order, are off by 2e-7 to 8e-7 of the result, held to 3e-6."""
import numpy as np
import pytest

from paper_1804_04806_amd import ucd
from hip_helpers import check_specials, desc_of, inputs, rect, rel_l2, run_hip, run_oracle, run_oracle_zeros

pytestmark = pytest.mark.gpu

D, I = ucd.BWD_FILTER, ucd.ALGO_IMPLICIT

# (n, c, h, w, k, r, s, strides, pads)
NARROW = [rect(9, 1, 257, 131, 30, 11, 11, (1, 1), (5, 5)), rect(60, 2, 70, 140, 32, 5, 8, (1, 2), (2, 2)), rect(3, 3, 150, 800, 32, 7, 7, (1, 1), (3, 3)),
          rect(100, 8, 61, 63, 29, 5, 5, (1, 1), (1, 2))]
WIDE = [rect(70, 3, 224, 227, 62, 7, 7, (2, 2), (3, 3)), rect(1100, 3, 61, 59, 62, 7, 7, (2, 2), (0, 0)), rect(215, 3, 100, 121, 61, 7, 7, (3, 1), (2, 2)),
        rect(120, 3, 62, 330, 63, 7, 7, (1, 3), (5, 0)), rect(17200, 3, 7, 7, 60, 7, 7, (1, 1), (3, 3)), rect(155, 6, 80, 70, 64, 5, 5, (1, 1), (2, 2)),
        rect(48, 6, 100, 95, 64, 7, 7, (1, 1), (3, 3))]


def described(s, dtype):
    return ucd.ucd_describe_micro(desc_of(s, dtype=dtype), D, I, s.N)[0]


@pytest.mark.parametrize("s", NARROW + WIDE, ids=str)
def test_few_channels(s):
    assert "filter_few_kernel" in described(s, 0)
    x, _, dy = inputs(s, seed=101)
    ref = run_oracle(s, D, x=x, dy=dy)
    assert rel_l2(run_hip(s, D, [(I, s.N)], x=x, dy=dy), ref) <= 3e-6
    got = run_hip(s, D, [(I, s.N - 1), (I, 1)], x=x, dy=dy)
    assert rel_l2(got, ref) <= 3e-6 and np.abs(got - ref).max() <= 1e-4 * np.sqrt(np.mean(ref ** 2))


def test_few_channels_accumulate():
    s = NARROW[1]
    x, w, dy = inputs(s, seed=102)
    ref = run_oracle(s, D, x=x, dy=dy, beta=1.0, dw0=w)
    assert rel_l2(run_hip(s, D, [(I, s.N)], x=x, dy=dy, beta=1.0, dw0=w), ref) <= 3e-6


@pytest.mark.parametrize("s", [NARROW[1], WIDE[1]], ids=str)
@pytest.mark.parametrize("scale", [2.0 ** -110, 2.0 ** -60, 2.0 ** 60])
def test_few_channels_out_of_range(s, scale):
    """Gradients below bf16's range and products near the ends of fp32's, which the fp32 instructions compute."""
    x, _, dy = inputs(s, seed=103)
    dy = (dy * np.float32(scale)).astype(np.float32)
    ref = run_oracle(s, D, x=x, dy=dy)
    assert rel_l2(run_hip(s, D, [(I, s.N)], x=x, dy=dy) / scale, ref / scale) <= 5e-6


@pytest.mark.parametrize("s", [NARROW[2], WIDE[2], WIDE[4]], ids=str)
def test_few_channels_not_finite(s):
    """Infinities and NaN come out where, and as, fp32 arithmetic gives them: pixels of x that a tap does not reach, or reaches only beside
    dy's rows, leave it finite."""
    x, _, dy = inputs(s, seed=104)
    x[0, 0, -1, -1], x[1, 1, 0, 0], x[2, 2, 1, -1] = np.inf, -np.inf, np.nan
    ref = run_oracle(s, D, x=x, dy=dy)
    got = run_hip(s, D, [(I, s.N)], x=x, dy=dy).astype(np.float64)
    fine = np.isfinite(ref)
    assert fine.any() and not fine.all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert rel_l2(got[fine], ref[fine]) <= 5e-6


@pytest.mark.parametrize("s", [NARROW[0], NARROW[2], NARROW[3], WIDE[2], WIDE[3], WIDE[6]], ids=str)
def test_few_channels_dy_not_finite(s):
    """The same of dy: in the middle, beside the padding (a zero that an infinity meets there is a NaN, as in the GEMMs) and where a row ends inside
    a group of eight pixels; the other output channels stay exact.  Together with one of x."""
    x, _, dy = inputs(s, seed=105)
    dy[0, 2, s.P // 2, s.Q // 2], dy[1, -1, -1, -1], dy[2, 5, 0, 0], dy[-1, 7, s.P // 2, -1] = np.inf, -np.inf, np.nan, np.inf
    x[1, 0, 0, 0] = np.inf
    check_specials(run_hip(s, D, [(I, s.N)], x=x, dy=dy).astype(np.float64), run_oracle_zeros(s, D, x=x, dy=dy), 5e-6)


@pytest.mark.parametrize("dtype, s", [(0, rect(16, 3, 61, 59, 32, 7, 7, (2, 2), (0, 0))), (0, rect(256, 3, 227, 227, 96, 11, 11, (4, 4), (0, 0))),
                                      (0, rect(128, 17, 112, 112, 32, 7, 7, (2, 2), (3, 3))), (1, NARROW[0]), (0, rect(200, 3, 224, 224, 32, 7, 7, (2, 2), (3, 3))), (0, rect(256, 3, 112, 112, 64, 3, 3, (1, 1), (1, 1)))],
                         ids=str)
def test_layers_that_it_does_not_take(dtype, s):
    assert "filter_few_kernel" not in described(s, dtype)
