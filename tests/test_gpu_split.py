"""fp32 GEMMs on the bf16 matrix pipe (three-way split operands): edges of its tiles, loaders and range handling.

Bounds.  A product of two split operands leaves out terms below 2^-24 of it and accumulates in fp32; over n
rows the worst relative L2 error that fp32 accumulation in chunks allows is a few 2^-24 * sqrt(n), and the
kernel is built to stay below what the fp32 matrix instructions give (3e-7 to 1e-6 on these shapes): 1e-6."""
import re

import numpy as np
import pytest

from paper_1804_04806_amd import ucd
from paper_1804_04806_amd.synth import Shape
from hip_helpers import inputs, rel_l2, run_hip, run_oracle

pytestmark = pytest.mark.gpu

I, MIRROR = ucd.ALGO_IMPLICIT, ucd.ALGO_IMPLICIT_MIRROR

SHAPES = [
    # Forward / mirrored BackwardData: output channels around each tile height (64, 96, 128), reductions that end
    # inside a 16-row step, inside a 4-row load and inside a 64-row window
    Shape(2, 37, 9, 11, 34, 3, 3, 1, 1), Shape(2, 33, 8, 8, 33, 1, 1, 1, 0), Shape(1, 21, 12, 12, 65, 3, 3, 1, 1),
    Shape(3, 5, 31, 30, 96, 11, 11, 4, 0), Shape(2, 9, 20, 20, 97, 7, 7, 2, 3), Shape(2, 3, 14, 14, 129, 5, 5, 1, 2),
    Shape(2, 128, 9, 7, 64, 1, 1, 1, 0), Shape(3, 80, 11, 6, 127, 1, 1, 1, 0), Shape(2, 79, 8, 8, 65, 1, 1, 1, 0),
    Shape(24, 64, 33, 33, 128, 3, 3, 1, 1), Shape(33, 67, 40, 40, 250, 2, 2, 1, 0),
    # BackwardFilter: images whose pixel count is 1, 2 or 3 above a multiple of 4, one row or column of pixels,
    # strides 1 to 3, outputs narrower and wider than the input, more than 31 taps, more rows than the pixel table
    Shape(5, 17, 13, 13, 40, 3, 3, 1, 1), Shape(7, 9, 7, 7, 50, 3, 3, 1, 2), Shape(9, 6, 1, 25, 33, 1, 3, 1, 0),
    Shape(3, 8, 25, 1, 70, 3, 1, 1, 0), Shape(4, 19, 18, 15, 130, 3, 3, 2, 1), Shape(2, 11, 23, 22, 64, 7, 7, 2, 3),
    Shape(3, 10, 17, 19, 96, 7, 7, 1, 3), Shape(2, 12, 20, 21, 61, 3, 3, 3, 0), Shape(1, 1, 6, 5, 33, 2, 2, 1, 1),
    Shape(2, 260, 9, 9, 256, 1, 1, 1, 0),
    # the same heights with reductions long enough for the split kernel in launches of one round of workgroups
    Shape(1, 23, 12, 12, 65, 3, 3, 1, 1), Shape(2, 9, 14, 14, 129, 5, 5, 1, 2), Shape(2, 387, 9, 7, 64, 1, 1, 1, 0),
    Shape(3, 401, 11, 6, 127, 1, 1, 1, 0), Shape(2, 390, 8, 8, 65, 1, 1, 1, 0),
    # BackwardFilter layers whose runs break or that need two masks per pixel, large enough for the split kernel
    Shape(300, 19, 18, 14, 130, 3, 3, 2, 1), Shape(210, 19, 23, 22, 64, 7, 7, 2, 3), Shape(14, 10, 17, 19, 96, 7, 7, 1, 3),
    # 128 x 256 tiles on eight waves: output channels just under 256, pixels just over a multiple of 256, filters of
    # nearly 512 columns; border masks, none, and more than 31 taps; column strides 1 and 2
    Shape(61, 56, 20, 21, 250, 3, 3, 1, 1), Shape(61, 56, 22, 23, 250, 3, 3, 1, 0), Shape(61, 10, 20, 21, 250, 7, 7, 1, 3),
    Shape(61, 56, 40, 41, 250, 3, 3, 2, 1), Shape(61, 56, 41, 43, 250, 3, 3, 2, 0), Shape(61, 10, 40, 41, 250, 7, 7, 2, 3),
]


def _id(s):
    return f"n{s.N}c{s.C}h{s.H}w{s.W}k{s.K}r{s.R}s{s.S}st{s.stride}p{s.pad}"


def _runs(s):
    """Operations whose GEMM has more than 32 rows: those run on the split kernel."""
    runs = [(ucd.FWD, I), (ucd.BWD_FILTER, I)] if s.K > 32 else []
    if s.C > 32 and s.stride == 1 and s.pad <= min(s.R, s.S) - 1:
        runs.append((ucd.BWD_DATA, MIRROR))
    return runs


def _kernels(s, op, algo):
    return ucd.ucd_describe_micro(ucd.layer(s), op, algo, s.N)[0]


def _tile_runs(s):
    """(operation, algorithm, layer): the operations above with so many images that they leave gemm_kernel_small."""
    for op, algo in _runs(s):
        t = s
        while "gemm_kernel_small" in _kernels(t, op, algo):
            t = t.with_batch(t.N + 1)
        yield op, algo, t


def _check_edges(s, op, algo):
    x, w, dy = inputs(s, seed=7)
    got = run_hip(s, op, [(algo, s.N)], x=x, w=w, dy=dy)
    ref = run_oracle(s, op, x=x, w=w, dy=dy)
    assert rel_l2(got, ref) <= 1e-6, (ucd.OP_NAMES[op], s.N, rel_l2(got, ref))


@pytest.mark.parametrize("s", SHAPES, ids=_id)
def test_split_gemm_edges(s):
    for op, algo, t in _tile_runs(s):
        rows = (t.C if op == ucd.FWD else t.K) * t.R * t.S
        text = _kernels(t, op, algo)
        split = "gemm_kernel_split<" in text
        assert split or "gemm_kernel<" in text, text
        if op == ucd.BWD_FILTER:  # strided layers and padded ones of many taps: from a number of multiplications on
            assert split or (t.K * t.C * t.R * t.S * t.N * t.P * t.Q < 1.6e9 and (t.stride > 1 or t.R * t.S > 31))
        else:
            assert split or rows < 384   # short reductions stay on the fp32 kernel
        _check_edges(t, op, algo)
        if t.N > s.N:
            _check_edges(s, op, algo)


def test_shapes_reach_every_tile_and_loader():
    """Which kernels the shapes above run is the launch rules' choice: every tile of the split kernel with every
    operand loader that it takes for such tiles has to be among them."""
    seen = set()
    for s in SHAPES:
        for op, algo in _runs(s):
            text = ucd.ucd_describe_micro(ucd.layer(s), op, algo, s.N)[0]
            if "gemm_kernel_split" in text:
                tile = re.search(r"Tile<(\w+)>", text).group(1)
                taps = "free" if s.pad == 0 and s.R * s.S > 1 else "big" if s.R * s.S > 31 else "few"
                seen.add((tile, "pixels" if op != ucd.BWD_FILTER else f"filter stride {min(s.stride, 3)}", taps))
    for tile in ("64x64", "64x128", "96x128", "128x64", "128x128", "128x256"):
        assert any(t == tile for t, _, _ in seen), (tile, sorted(seen))
    for taps in ("few", "free", "big"):
        assert ("128x256", "pixels", taps) in seen and ("128x256", "filter stride 1", taps) in seen, sorted(seen)
        assert ("128x256", "filter stride 2", taps) in seen, sorted(seen)


@pytest.mark.parametrize("s", [SHAPES[i] for i in (6, 9, 10, 13, 14, 0, 24, 26)], ids=_id)
def test_split_gemm_not_finite(s):
    """Infinities and NaN come out where, and as, fp32 arithmetic gives them; the other outputs stay exact."""
    for op, algo, s in _tile_runs(s):
        x, w, dy = inputs(s, seed=8)
        finite_dy = dy.copy()
        x[0, 0, 0, 0], x[-1, -1, -1, -1], dy[0, -1, 0, 0], dy[-1, 0, -1, -1] = np.inf, np.nan, -np.inf, np.nan
        x[0, 1, 0, 0] = 3.3e38  # finite, but infinite when rounded to bf16
        # BackwardFilter's kernels multiply dy with the padding's zeros, the oracle skips them
        g = finite_dy if op == ucd.BWD_FILTER and s.pad else dy
        got = run_hip(s, op, [(algo, s.N)], x=x, w=w, dy=g).astype(np.float64)
        ref = run_oracle(s, op, x=x, w=w, dy=g)
        ref = np.where(np.abs(ref) > np.finfo(np.float32).max, np.sign(ref) * np.inf, ref)
        fine = np.isfinite(ref)
        assert not fine.all() and fine.any()
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
        assert np.array_equal(np.isneginf(got), np.isneginf(ref))
        assert rel_l2(got[fine], ref[fine]) <= 1e-6


# Operands whose low parts leave bf16's range (below 2^-102) or that vanish in it (below 2^-134: denormals), the other
# operand near 1 or so large that the results are ordinary numbers, and large ones.  fp32 operands of any size are
# exact inputs; the partner keeps results above 2^-110, where fp32 sums of a few 2^-149 steps still meet the bound.
RANGES = [(1e-37, 1.0), (1e-30, 1.0), (1e30, 1.0), (2.0 ** -116, 2.0 ** 30), (2.0 ** -124, 2.0 ** 40), (2.0 ** -136, 2.0 ** 60)]


@pytest.mark.parametrize("scale,partner", RANGES)
@pytest.mark.parametrize("s", [SHAPES[0], SHAPES[11]], ids=_id)
def test_split_gemm_range(s, scale, partner):
    for op, algo, s in _tile_runs(s):
        x, w, dy = inputs(s, seed=9)
        for first in (True, False):   # which operand is the small one
            a, b = np.float32(scale if first else partner), np.float32(partner if first else scale)
            xs, ws, dys = (x * a, w * b, dy) if op == ucd.FWD else (x, w * b, dy * a) if op == ucd.BWD_DATA else (x * b, w, dy * a)
            got = run_hip(s, op, [(algo, s.N)], x=xs, w=ws, dy=dys)
            ref = run_oracle(s, op, x=xs, w=ws, dy=dys)
            assert rel_l2(got, ref) <= 1e-6, (ucd.OP_NAMES[op], first, rel_l2(got, ref))


@pytest.mark.parametrize("s", [SHAPES[i] for i in (0, 9, 11, 13, 26)], ids=_id)
def test_split_gemm_small_parts(s):
    """One image, one output channel or one input channel far below bf16's range among ordinary ones, whose results
    are compared by themselves."""
    tiny, up = np.float32(2.0 ** -130), np.float32(2.0 ** 40)
    for op, algo, s in _tile_runs(s):
        x, w, dy = inputs(s, seed=10)
        x[0] *= tiny
        w[1] *= tiny
        dy[:, 2] *= tiny
        xs, ws, dys = (x, w * up, dy) if op == ucd.FWD else (x, w * up, dy) if op == ucd.BWD_DATA else (x * up, w, dy)
        got = run_hip(s, op, [(algo, s.N)], x=xs, w=ws, dy=dys)
        ref = run_oracle(s, op, x=xs, w=ws, dy=dys)
        parts = {ucd.FWD: [(0, 0), (0, 3), (1, 3)], ucd.BWD_DATA: [(0,), (1,)], ucd.BWD_FILTER: [(2,), (3,)]}[op]
        for at in parts:
            assert rel_l2(got[at], ref[at]) <= 1e-6, (ucd.OP_NAMES[op], at, rel_l2(got[at], ref[at]))


# ---- fused Winograd F(2x2,3x3) ----------------------------------------------------------
WF = ucd.ALGO_WINOGRAD_FUSED
WINO_SHAPES = [
    # input channels around the 16-channel step and the 8-channel blocks of the transformed filter, output channels
    # around the 64-channel block, tiles around the 64-tile block, odd and even widths, paddings 0 to 2
    Shape(1, 32, 6, 6, 64, 3, 3, 1, 1), Shape(3, 49, 13, 13, 65, 3, 3, 1, 1), Shape(2, 40, 9, 16, 31, 3, 3, 1, 0),
    Shape(2, 47, 10, 7, 130, 3, 3, 1, 2), Shape(5, 56, 8, 11, 3, 3, 3, 1, 1), Shape(1, 100, 17, 16, 96, 3, 3, 1, 1),
    Shape(3, 64, 5, 4, 37, 3, 3, 1, 2), Shape(2, 36, 3, 3, 40, 3, 3, 1, 1),
    Shape(3, 33, 13, 13, 63, 3, 3, 1, 1), Shape(2, 41, 7, 7, 66, 3, 3, 1, 1),
]
PHASE_SHAPES = [Shape(2, 3, 31, 35, 48, 11, 11, 4, 0), Shape(1, 9, 22, 17, 33, 5, 5, 2, 2), Shape(2, 4, 23, 23, 40, 7, 7, 3, 1)]


def _wino_runs(s):
    """Operations on the split kernel: 32 input channels, 41 with more than 64 output channels."""
    return ([(ucd.FWD, s)] if s.C >= (32 if s.K <= 64 else 41) and s.stride == 1 else []) + \
           ([(ucd.BWD_DATA, s)] if s.K >= (32 if s.C <= 64 or s.stride > 1 else 41) else [])


@pytest.mark.parametrize("s", WINO_SHAPES + PHASE_SHAPES, ids=_id)
def test_split_winograd_edges(s):
    """Bound: Winograd's transforms amplify the operands' rounding by less than 4 (their matrices have entries 0, 1
    and 1/2 and at most three terms a row), so 4 times the direct kernels' bound; measured 2e-7 to 6e-7."""
    x, w, dy = inputs(s, seed=17)
    for op, _ in _wino_runs(s):
        assert "wino_fused_split_kernel" in ucd.ucd_describe_micro(ucd.layer(s), op, WF, s.N)[0]
        for parts in ([s.N], [1] * s.N):
            got = run_hip(s, op, [(WF, b) for b in parts], x=x, w=w, dy=dy)
            ref = run_oracle(s, op, x=x, w=w, dy=dy)
            assert rel_l2(got, ref) <= 4e-6, (ucd.OP_NAMES[op], parts, rel_l2(got, ref))


@pytest.mark.parametrize("s", [WINO_SHAPES[1], WINO_SHAPES[2], WINO_SHAPES[3], WINO_SHAPES[5], PHASE_SHAPES[1]], ids=_id)
def test_split_winograd_not_finite(s):
    """What arithmetic makes not finite is not finite, and blocks that hold such values are otherwise as exact as the
    rest: only outputs within a tile's reach of the pixel may differ from the oracle's."""
    x, w, dy = inputs(s, seed=18)
    t = dy if s.stride > 1 else x
    t[0, 1, 2, 2], t[-1, -1, 0, 0] = np.inf, np.nan
    op = ucd.BWD_DATA if s.stride > 1 else ucd.FWD
    got = run_hip(s, op, [(WF, s.N)], x=x, w=w, dy=dy).astype(np.float64)
    ref = run_oracle(s, op, x=x, w=w, dy=dy)
    assert not np.isfinite(got[~np.isfinite(ref)]).any()
    far = np.isfinite(got)
    assert far.mean() > 0.3 and rel_l2(got[far], ref[far]) <= 4e-6


@pytest.mark.parametrize("scale,partner", RANGES)
@pytest.mark.parametrize("s", [WINO_SHAPES[1], PHASE_SHAPES[0]], ids=_id)
def test_split_winograd_range(s, scale, partner):
    """The filter's transform is fp32 arithmetic of its own (halves and sums), whose results have steps of 2^-149: a
    filter of that size is off by up to one such step before it is multiplied, which is added to the bound."""
    x, w, dy = inputs(s, seed=19)
    op = ucd.BWD_DATA if s.stride > 1 else ucd.FWD
    for first in (True, False):
        a, b = np.float32(scale if first else partner), np.float32(partner if first else scale)
        got = run_hip(s, op, [(WF, s.N)], x=x * a, w=w * b, dy=dy * a)
        ref = run_oracle(s, op, x=x * a, w=w * b, dy=dy * a)
        step = 2.0 ** -149 / np.sqrt(np.mean(np.square((w * b).astype(np.float64))))
        assert rel_l2(got, ref) <= 4e-6 + step, (first, rel_l2(got, ref))


def test_split_winograd_recomputed_blocks_are_not_far_slower():
    """With one NaN in every image each workgroup computes its block twice, the second time on the fp32 instructions:
    2.3 times the ordinary call (143 us against 63), far from the 8 times that are the limit here."""
    import torch
    s = Shape(64, 256, 14, 14, 256, 3, 3, 1, 1)
    plan = ucd.ucd_plan_fixed(ucd.layer(s), ucd.FWD, [(WF, s.N)])
    x, w = (torch.randn(shape, device="cuda:0") for shape in (s.x_shape, s.w_shape))
    y = torch.empty(s.y_shape, device="cuda:0")
    ws = torch.empty(plan.ws_bytes // 4, device="cuda:0")
    ms = []
    for poisoned in (False, True):
        if poisoned:
            x[:, 0, 0, 0] = float("nan")
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ucd.ucd_conv_fwd(plan, x, w, y, ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        ms.append(best)
    assert bool(torch.isnan(y).any()) and not bool(torch.isnan(y).all())
    assert ms[1] <= 8 * ms[0], ms
