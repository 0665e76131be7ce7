"""gemm_kernel_small: edges of its 16 x 16 tiles and 16- and 32-row steps, refills of its row table, waves without a step of
their own, stride phases with and without taps, more than 31 taps, chunks that meet through atomics."""
import numpy as np
import pytest

from paper_1804_04806_amd import ucd
from paper_1804_04806_amd.synth import Shape
from hip_helpers import desc_of, inputs, rect, rel_l2, run_hip, run_oracle
from test_gpu_bf16 import bf16_inputs, check_bf16_output, run_hip_bf16

pytestmark = pytest.mark.gpu

I = ucd.ALGO_IMPLICIT
F, D, W = ucd.FWD, ucd.BWD_DATA, ucd.BWD_FILTER

# (shape, operations that run on the kernel: fp32, bf16)
SHAPES = [
    (Shape(1, 16, 4, 4, 16, 1, 1, 1, 0), (F, D, W), (F, D, W)), (Shape(1, 1, 3, 5, 17, 1, 1, 1, 0), (F, D, W), (D, W)),
    (Shape(1, 15, 1, 17, 15, 1, 1, 1, 0), (F, D, W), (D, W)), (Shape(3, 33, 5, 5, 31, 3, 3, 1, 1), (F, D, W), (D, W)),
    (Shape(2, 16, 9, 7, 32, 5, 3, 1, 1), (F, D, W), (F, D, W)), (Shape(1, 284, 6, 6, 32, 3, 3, 1, 1), (F, D, W), (F, D, W)),
    (Shape(1, 290, 6, 6, 32, 3, 3, 1, 1), (D, W), (F, D, W)), (Shape(1, 1020, 5, 5, 40, 3, 3, 1, 1), (D,), (F, D)),
    (Shape(1, 20, 6, 5, 640, 3, 3, 1, 1), (F, W), (F, D, W)), (Shape(2, 12, 13, 11, 34, 3, 3, 2, 1), (F, D, W), (F, D, W)),
    (Shape(2, 12, 13, 11, 34, 1, 1, 2, 0), (F, D, W), (F, D, W)), (Shape(1, 6, 17, 19, 20, 3, 3, 4, 0), (F, D, W), (F, D, W)),
    (Shape(1, 10, 17, 13, 36, 7, 7, 1, 3), (F, D, W), (F, D, W)), (Shape(1, 4, 23, 20, 24, 11, 11, 4, 0), (F, D, W), (F, D, W)),
    (Shape(1, 3, 31, 30, 40, 7, 7, 2, 3), (F, D, W), (D, W)), (Shape(4, 8, 17, 15, 32, 3, 3, 1, 1), (F, D, W), (F, D, W)),
    (Shape(8, 16, 16, 16, 32, 3, 3, 1, 1), (F, D, W), (F, D)), (Shape(60, 9, 13, 12, 32, 1, 1, 1, 0), (D, W), ()),
    (Shape(1, 256, 14, 14, 256, 3, 3, 1, 1), (F, D), (F, D)),
]


def _kernel(s, op, dtype=0):
    return ucd.ucd_describe_micro(desc_of(s, dtype), op, I, s.N)[0]


@pytest.mark.parametrize("s,f32,bf16", SHAPES, ids=lambda v: str(v) if isinstance(v, Shape) else "")
def test_small_layers(s, f32, bf16):
    """fp32: sums of at most 2560 products in runs of at most 640 per accumulator, as the other kernels' edge tests; bf16:
    products are exact, y and dx are held to the output rounding."""
    x, w, dy = inputs(s, seed=41)
    for op in (F, D, W):
        assert ("gemm_kernel_small" in _kernel(s, op)) == (op in f32), (op, _kernel(s, op))
        if op in f32:
            ref = run_oracle(s, op, x=x, w=w, dy=dy)
            assert rel_l2(run_hip(s, op, [(I, s.N)], x=x, w=w, dy=dy), ref) <= 1e-6, op
    if W in f32:
        dw0 = np.linspace(-1, 1, w.size, dtype=np.float32).reshape(w.shape)
        got = run_hip(s, W, [(I, s.N)], x=x, dy=dy, beta=1.0, dw0=dw0)
        assert rel_l2(got, run_oracle(s, W, x=x, dy=dy, beta=1.0, dw0=dw0)) <= 1e-6
    bits, (x, w, dy) = bf16_inputs(s, seed=42)
    for op in (F, D, W):
        assert ("gemm_kernel_small" in _kernel(s, op, 1)) == (op in bf16), (op, _kernel(s, op, 1))
        if op in bf16:
            got, ref = run_hip_bf16(s, op, [(I, s.N)], bits), run_oracle(s, op, x=x, w=w, dy=dy)
            if op == W:
                assert rel_l2(got, ref) <= 1e-6
            else:
                check_bf16_output(got, ref, ucd.OP_NAMES[op])


RECT = [rect(2, 12, 13, 11, 34, 3, 3, (1, 2), (1, 0)), rect(2, 10, 12, 15, 20, 3, 3, (2, 1), (0, 2)),
        rect(1, 8, 19, 17, 24, 5, 3, (3, 2), (2, 1)), rect(1, 6, 18, 21, 20, 3, 5, (1, 4), (0, 3)),
        rect(3, 5, 14, 13, 17, 2, 3, (4, 4), (1, 0)), rect(1, 4, 22, 19, 24, 7, 5, (2, 3), (3, 0)),
        rect(2, 9, 10, 11, 33, 1, 3, (1, 2), (0, 1)), rect(1, 10, 13, 16, 36, 7, 6, (1, 2), (1, 2))]


@pytest.mark.parametrize("s", RECT, ids=str)
def test_small_layers_rows_and_columns_differ(s):
    x, w, dy = inputs(s, seed=45)
    for op in (F, D, W):
        assert "gemm_kernel_small" in _kernel(s, op)
        assert rel_l2(run_hip(s, op, [(I, s.N)], x=x, w=w, dy=dy), run_oracle(s, op, x=x, w=w, dy=dy)) <= 1e-6, op
    bits, (x, w, dy) = bf16_inputs(s, seed=46)
    for op in (D, W):
        assert "gemm_kernel_small" in _kernel(s, op, 1)
        got, ref = run_hip_bf16(s, op, [(I, s.N)], bits), run_oracle(s, op, x=x, w=w, dy=dy)
        if op == W:
            assert rel_l2(got, ref) <= 1e-6
        else:
            check_bf16_output(got, ref, ucd.OP_NAMES[op])


def test_values_behind_a_filter_row_do_not_reach_it():
    """A lane reads four reduction rows at a time, at the end of a filter row also the next row's first ones."""
    s = Shape(1, 7, 5, 5, 20, 3, 3, 1, 1)
    x, w, _ = inputs(s, seed=43)
    w[3], w[5] = np.inf, np.nan
    got = run_hip(s, F, [(I, 1)], x=x, w=w)
    fine = [k for k in range(20) if k not in (3, 5)]
    assert "gemm_kernel_small" in _kernel(s, F)
    assert rel_l2(got[:, fine], run_oracle(s, F, x=x, w=w)[:, fine]) <= 1e-6
    assert not np.isfinite(got[:, [3, 5]]).any()


# sums of 1 to 64 products, BackwardFilter of more than 32 output channels up to 128
FEW = [(Shape(2, c, 7, 9, 20, r, r, 1, r // 2), F) for c, r in ((1, 1), (2, 1), (3, 1), (5, 1), (16, 1), (17, 1), (64, 1), (1, 3), (7, 3), (1, 7))] + \
      [(Shape(2, 20, 7, 9, k, r, r, st, r // 2), D) for k, r, st in ((1, 1, 1), (2, 1, 1), (15, 1, 1), (33, 1, 1), (63, 1, 1), (2, 3, 1), (7, 3, 1), (16, 3, 2), (4, 7, 2))] + \
      [(Shape(n, 10, h, w, k, r, r, st, p), W) for n, h, w, k, r, st, p in (
          (1, 1, 1, 20, 1, 1, 0), (1, 1, 2, 20, 1, 1, 0), (1, 3, 3, 20, 3, 1, 1), (1, 4, 4, 20, 1, 1, 0), (2, 5, 5, 20, 1, 1, 0),
          (1, 8, 8, 20, 3, 1, 1), (1, 9, 9, 20, 3, 2, 0), (1, 8, 8, 20, 7, 1, 3), (2, 7, 7, 40, 3, 1, 1), (2, 8, 8, 33, 1, 1, 0))]


@pytest.mark.parametrize("s,op", FEW, ids=str)
def test_sums_of_few_products_are_rounded_once(s, op):
    """Products of 48 bits are summed in 64-bit arithmetic: the result is off by half a unit of its last place and, where terms
    cancel, by a rounding at 2^-53 of the largest partial sum for each of them."""
    x, w, dy = inputs(s, seed=44)
    assert "gemm_kernel_small" in _kernel(s, op)
    a, b, rows = {F: (x, w, s.C * s.R * s.S), D: (dy, w, s.K * s.R * s.S), W: (x, dy, s.N * s.P * s.Q)}[op]
    got, ref = run_hip(s, op, [(I, s.N)], x=x, w=w, dy=dy).astype(np.float64), run_oracle(s, op, x=x, w=w, dy=dy)
    half = 0.5 * np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64)
    cancelled = rows * 2.0 ** -53 * rows * np.abs(a).max() * np.abs(b).max()
    assert (np.abs(got - ref) <= half * (1 + 1e-6) + cancelled).all()
