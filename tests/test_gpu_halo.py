"""conv_halo_kernel (BackwardData over a window in LDS): edges of its tiles of channels and positions, chunks of 16 channels
that the last one does not fill, column blocks, tiles over several images, paddings of either parity, strides and paddings of
rows and columns that differ, values out of range, equal bits in every run."""
import numpy as np
import pytest

from paper_1804_04806_amd import ucd
from paper_1804_04806_amd.synth import Shape
from hip_helpers import desc_of, inputs, recomputed_time_ratio, rect, rel_l2, run_hip, run_oracle

pytestmark = pytest.mark.gpu

I, D = ucd.ALGO_IMPLICIT, ucd.BWD_DATA

SHAPES = [
    # column stride 2: channels around the tile of 64, 17 to 65 output channels, positions over one and many images, rows
    # and columns odd and even, blocks of columns (the last one ragged), filters with fewer and more rows than columns
    Shape(20, 24, 14, 14, 400, 3, 3, 2, 1), Shape(31, 63, 13, 11, 65, 3, 3, 2, 0), Shape(5, 65, 29, 31, 33, 3, 3, 2, 2),
    Shape(2, 130, 26, 71, 50, 3, 3, 2, 1), Shape(40, 40, 7, 9, 400, 3, 3, 2, 1), Shape(1, 64, 61, 150, 47, 2, 3, 2, 1),
    Shape(6, 33, 40, 41, 17, 6, 3, 2, 1), Shape(60, 70, 8, 7, 130, 3, 3, 2, 1), Shape(9, 100, 20, 23, 64, 5, 5, 2, 2),
    Shape(9, 64, 21, 22, 49, 5, 5, 2, 1), Shape(4, 100, 31, 52, 150, 4, 5, 2, 3), Shape(30, 96, 12, 13, 130, 5, 5, 2, 0),
    # stride 1: tiles of 128 and of 64 channels
    Shape(101, 100, 20, 21, 20, 3, 3, 1, 1), Shape(85, 120, 23, 22, 37, 4, 3, 1, 0), Shape(61, 56, 28, 27, 17, 5, 5, 1, 2),
]


def _id(s):
    return f"n{s.N}c{s.C}h{s.H}w{s.W}k{s.K}r{s.R}s{s.S}st{s.stride}p{s.pad}"


def _run(s, w, dy, parts=None):
    assert parts or "conv_halo_kernel<" in ucd.ucd_describe_micro(desc_of(s), D, I, s.N)[0]
    return run_hip(s, D, [(I, b) for b in parts or [s.N]], w=w, dy=dy)


@pytest.mark.parametrize("s", SHAPES, ids=_id)
def test_halo_edges(s):
    _, w, dy = inputs(s, seed=51)
    ref = run_oracle(s, D, w=w, dy=dy)
    for parts in (None, [s.N - 1, 1] if s.N > 1 else None):
        assert rel_l2(_run(s, w, dy, parts), ref) <= 1e-6


# rows and columns of different strides and paddings: (1, 2), (2, 1), (3, 2), (3, 1), (4, 2); filters as wide as they are not high
RECT = [rect(60, 24, 14, 15, 100, 3, 3, (1, 2), (1, 0)), rect(101, 100, 20, 21, 20, 3, 3, (2, 1), (0, 1)),
        rect(6, 63, 29, 31, 65, 3, 3, (3, 2), (1, 2)), rect(70, 120, 28, 23, 40, 4, 3, (3, 1), (2, 0)),
        rect(9, 40, 25, 22, 49, 5, 5, (1, 2), (2, 1)), rect(12, 33, 31, 40, 150, 4, 5, (4, 2), (0, 2)),
        rect(7, 70, 33, 35, 20, 2, 3, (2, 2), (0, 1)), rect(37, 51, 45, 29, 77, 3, 5, (1, 1), (1, 2)),
        rect(85, 120, 23, 22, 36, 5, 3, (1, 1), (0, 2)), rect(61, 56, 29, 26, 17, 3, 5, (2, 1), (1, 0))]


@pytest.mark.parametrize("s", RECT, ids=str)
def test_halo_rows_and_columns_differ(s):
    _, w, dy = inputs(s, seed=54)
    ref = run_oracle(s, D, w=w, dy=dy)
    for parts in (None, [1, s.N - 1]):
        assert rel_l2(_run(s, w, dy, parts), ref) <= 1e-6


@pytest.mark.parametrize("det", (0, 1))
@pytest.mark.parametrize("s", [SHAPES[0], SHAPES[9], SHAPES[12], RECT[2]], ids=str)
def test_halo_gives_the_same_bits_in_every_run(s, det):
    """Also with a part of the tiles recomputed (one image holds a value below bf16's range)."""
    _, w, dy = inputs(s, seed=55)
    dy[0, 1, 1, 1] = 0xFFFFFF * 2.0 ** -143
    prev = ucd.ucd_set_deterministic(det)
    try:
        runs = [_run(s, w, dy) for _ in range(3)]
    finally:
        ucd.ucd_set_deterministic(prev)
    assert all(np.array_equal(runs[0], r) for r in runs[1:])


@pytest.mark.parametrize("s", [SHAPES[1], SHAPES[3], SHAPES[9], SHAPES[13]], ids=_id)
def test_halo_not_finite(s):
    """Infinities and NaN come out where, and as, fp32 arithmetic gives them; the other outputs stay exact."""
    _, w, dy = inputs(s, seed=52)
    dy[0, -1, 1, 1], dy[-1, 0, -1, -1], dy[0, 0, 0, 0] = -np.inf, np.nan, 3.3e38   # the last: infinite when rounded to bf16
    got = _run(s, w, dy).astype(np.float64)
    ref = run_oracle(s, D, w=w, dy=dy)
    ref = np.where(np.abs(ref) > np.finfo(np.float32).max, np.sign(ref) * np.inf, ref)
    fine = np.isfinite(ref)
    assert fine.any() and not fine.all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert rel_l2(got[fine], ref[fine]) <= 1e-6


@pytest.mark.parametrize("scale,partner", [(1e-37, 1.0), (1e30, 1.0), (2.0 ** -116, 2.0 ** 30), (2.0 ** -136, 2.0 ** 60)])
@pytest.mark.parametrize("s", [SHAPES[2], SHAPES[8]], ids=_id)
def test_halo_range(s, scale, partner):
    """Operands whose low parts leave bf16's range, and large ones, next to partners that bring the results back."""
    _, w, dy = inputs(s, seed=53)
    for a, b in ((scale, partner), (partner, scale)):
        ws, dys = w * np.float32(a), dy * np.float32(b)
        assert rel_l2(_run(s, ws, dys), run_oracle(s, D, w=ws, dy=dys)) <= 1e-6


def test_halo_recomputed_tiles_are_not_far_slower():
    """1.9 times the ordinary call (114 us against 217), 3 are the limit."""
    s = Shape(128, 64, 56, 56, 128, 3, 3, 2, 1)
    assert "conv_halo_kernel<" in ucd.ucd_describe_micro(ucd.layer(s), D, I, s.N)[0]
    assert recomputed_time_ratio(s, D) <= 3
