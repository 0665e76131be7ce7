"""pointwise_kernel, pointwise_split_stream_kernel, pointwise_bf16_kernel and pointwise_stream_kernel (1x1 layers that keep their input in LDS): edges of its tiles of 128 x 128, of its pairs of 16-channel
steps and of the last round of workgroups, images of a multiple of four pixels and not, values out of range, equal bits in every
run, tensors on any element."""
import numpy as np
import pytest

from paper_1804_04806_amd import ucd
from paper_1804_04806_amd.synth import Shape
from hip_helpers import inputs, recomputed_time_ratio, rel_l2, run_hip, run_oracle
from test_gpu_bf16 import bf16_inputs, check_bf16_output, dev_bf16, run_hip_bf16

pytestmark = pytest.mark.gpu

I, F, D = ucd.ALGO_IMPLICIT, ucd.FWD, ucd.BWD_DATA


def _layer(n, h, w, few, many, op):
    """1x1 layer whose `op` reduces over `few` channels into `many`."""
    return Shape(n, few if op == F else many, h, w, many if op == F else few, 1, 1, 1, 0)


CASES = [(21, 14, 14, 17, 129), (21, 13, 15, 32, 256), (5, 29, 29, 33, 257), (9, 22, 21, 48, 200), (6, 26, 26, 159, 140),
         (21, 14, 14, 160, 385), (63, 13, 10, 100, 100), (43, 28, 28, 20, 300), (42, 28, 29, 64, 130), (1, 64, 63, 96, 1000)]


# the streaming kernel: steps of 16 channels in threes, 128 rows, 256 pixels, workgroups in eights
STREAM32 = [(42, 28, 28, 33, 97), (21, 28, 28, 161, 200), (43, 27, 28, 249, 129), (10, 28, 29, 176, 500), (42, 28, 28, 256, 100)]


def _fp32_kernel(s, op):
    return ucd.ucd_describe_micro(ucd.layer(s), op, I, s.N)[0].split("<")[0]


def _run(s, op, x, w, dy, parts=None):
    assert parts or _fp32_kernel(s, op) in ("pointwise_kernel", "pointwise_split_stream_kernel")
    return run_hip(s, op, [(I, b) for b in parts or [s.N]], x=x, w=w, dy=dy)


@pytest.mark.parametrize("op", (F, D))
@pytest.mark.parametrize("case", CASES + STREAM32, ids=str)
def test_pointwise_edges(case, op):
    s = _layer(*case, op)
    assert _fp32_kernel(s, op) == ("pointwise_split_stream_kernel" if case in STREAM32 else "pointwise_kernel")
    x, w, dy = inputs(s, seed=61)
    ref = run_oracle(s, op, x=x, w=w, dy=dy)
    for parts in (None, [1, s.N - 1] if s.N > 1 else None):
        assert rel_l2(_run(s, op, x, w, dy, parts), ref) <= 1e-6


# BackwardData takes the streaming kernel for any number of input channels: one chain per sum
@pytest.mark.parametrize("case", [(33, 28, 28, 512, 128), (42, 22, 22, 1000, 130), (33, 28, 28, 1500, 97), (64, 14, 14, 2048, 256),
                                  (36, 31, 30, 4090, 100)], ids=str)
def test_pointwise_long_reductions(case):
    """A sum is rounded once per 16 channels: at 4090 of them a random walk of 256 steps at 2^-25 of the sums, 5e-7 of the
    result; the fp32 instructions, which round once per two, 1.5e-6."""
    s = _layer(*case, D)
    assert _fp32_kernel(s, D) == "pointwise_split_stream_kernel"
    _, w, dy = inputs(s, seed=68)
    assert rel_l2(_run(s, D, None, w, dy), run_oracle(s, D, w=w, dy=dy)) <= 1e-6


@pytest.mark.parametrize("det", (0, 1))
@pytest.mark.parametrize("op", (F, D))
@pytest.mark.parametrize("case", [CASES[4], CASES[9], STREAM32[1], STREAM32[3]], ids=str)
def test_pointwise_gives_the_same_bits_in_every_run(case, op, det):
    """Also with a part of the tiles recomputed (one image holds a value below bf16's range)."""
    s = _layer(*case, op)
    x, w, dy = inputs(s, seed=69)
    (x if op == F else dy)[0, 1, 1, 1] = 0xFFFFFF * 2.0 ** -143
    prev = ucd.ucd_set_deterministic(det)
    try:
        runs = [_run(s, op, x, w, dy) for _ in range(3)]
    finally:
        ucd.ucd_set_deterministic(prev)
    assert all(np.array_equal(runs[0], r) for r in runs[1:])


@pytest.mark.parametrize("op", (F, D))
@pytest.mark.parametrize("case", [CASES[1], CASES[2], CASES[7], STREAM32[0], STREAM32[1]], ids=str)
def test_pointwise_not_finite(case, op):
    """Infinities and NaN come out where, and as, fp32 arithmetic gives them; the other outputs stay exact."""
    s = _layer(*case, op)
    x, w, dy = inputs(s, seed=62)
    t = x if op == F else dy
    t[0, -1, 1, 1], t[-1, 0, -1, -1], t[0, 0, 0, 0] = -np.inf, np.nan, 3.3e38   # the last: infinite when rounded to bf16
    got = _run(s, op, x, w, dy).astype(np.float64)
    ref = run_oracle(s, op, x=x, w=w, dy=dy)
    ref = np.where(np.abs(ref) > np.finfo(np.float32).max, np.sign(ref) * np.inf, ref)
    fine = np.isfinite(ref)
    assert fine.any() and not fine.all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert rel_l2(got[fine], ref[fine]) <= 1e-6


@pytest.mark.parametrize("op", (F, D))
@pytest.mark.parametrize("scale,partner", [(1e-37, 1.0), (1e30, 1.0), (2.0 ** -116, 2.0 ** 30), (2.0 ** -136, 2.0 ** 60)])
def test_pointwise_range(scale, partner, op):
    """Operands whose low parts leave bf16's range, and large ones, next to partners that bring the results back."""
    for case in CASES[3], STREAM32[1]:
        s = _layer(*case, op)
        x, w, dy = inputs(s, seed=63)
        for a, b in ((scale, partner), (partner, scale)):
            xs, ws, dys = x * np.float32(a), w * np.float32(b), dy * np.float32(a)
            assert rel_l2(_run(s, op, xs, ws, dys), run_oracle(s, op, x=xs, w=ws, dy=dys)) <= 1e-6


def test_values_behind_a_filter_row_do_not_reach_it():
    """The last step of a filter row of 17 (33) channels reads into the next row."""
    for case in CASES[0], STREAM32[0]:
        s = _layer(*case, F)
        x, w, dy = inputs(s, seed=64)
        w[3], w[90] = np.inf, np.nan
        got = _run(s, F, x, w, dy)
        fine = [k for k in range(s.K) if k not in (3, 90)]
        assert rel_l2(got[:, fine], run_oracle(s, F, x=x, w=w)[:, fine]) <= 1e-6


# workgroups that walk over one tile row (33 tiles of pixels) and over all four (258)
@pytest.mark.parametrize("op", (F, D))
@pytest.mark.parametrize("case", [(21, 14, 14, 160, 385), (168, 14, 14, 32, 385)], ids=str)
def test_pointwise_recomputes_the_tile_row_of_an_inexact_filter_element(case, op):
    """One filter element that three bf16 parts do not represent (24 significant bits near 2^-120) sends its 128 output
    channels to the fp32 instructions, in every run, and no others: these keep the bits they have without it."""
    s = _layer(*case, op)
    x, w, dy = inputs(s, seed=67)
    clean = _run(s, op, x, w, dy)
    w[(130, 20) if op == F else (20, 130)] = 0xFFFFFF * 2.0 ** -143
    assert w[(130, 20) if op == F else (20, 130)] != 0
    runs = [_run(s, op, x, w, dy) for _ in range(4)]
    assert all(np.array_equal(runs[0], r) for r in runs[1:])
    assert np.array_equal(runs[0][:, :128], clean[:, :128]) and np.array_equal(runs[0][:, 256:], clean[:, 256:])
    assert not np.array_equal(runs[0][:, 128:256], clean[:, 128:256])
    assert rel_l2(runs[0], run_oracle(s, op, x=x, w=w, dy=dy)) <= 1e-6


@pytest.mark.parametrize("s,op,kernel", [(Shape(168, 160, 14, 14, 1024, 1, 1, 1, 0), F, "pointwise_kernel"),
                                         (Shape(64, 256, 28, 28, 1024, 1, 1, 1, 0), D, "pointwise_split_stream_kernel")],
                         ids=("lds", "stream"))
def test_pointwise_recomputed_tiles_are_not_far_slower(s, op, kernel):
    """The fp32 instructions alone take about 1.5 times the ordinary call: 2.5 and 2.7 times in all, 3.5 are the limit."""
    assert _fp32_kernel(s, op) == kernel
    assert recomputed_time_ratio(s, op) <= 3.5


# tiles of 128 pixels (the last three: of 256), 64-channel steps, 128 rows; (op,): the kernel takes that operation only
HALF = [(21, 14, 14, 40, 130), (41, 14, 10, 256, 386), (3, 34, 30, 264, 66), (5, 28, 27, 512, 258), (9, 22, 22, 8, 100),
        (1, 4, 901, 72, 200), (6, 31, 32, 328, 34), (14, 40, 36, 24, 261, (F,)), (41, 22, 23, 256, 300, ()), (27, 28, 27, 256, 260),
        (11, 44, 42, 56, 516)]
# tiles of 128 or 256 rows and 256 pixels, 32-channel steps in threes, workgroups in eights
STREAM = [(14, 40, 36, 24, 129, (F,)), (42, 22, 22, 256, 130), (26, 28, 28, 72, 22), (26, 28, 28, 200, 36), (33, 32, 32, 104, 256),
          (34, 32, 32, 8, 140), (9, 44, 42, 520, 300), (6, 30, 30, 552, 20, (D,)), (3, 34, 30, 1032, 66, (D,)),
          (65, 28, 18, 264, 140), (9, 30, 28, 320, 1000), (35, 32, 31, 648, 250), (1, 148, 149, 96, 66)]


@pytest.mark.parametrize("op", (F, D))
@pytest.mark.parametrize("case", HALF + STREAM, ids=str)
def test_pointwise_bf16_edges(case, op):
    """Products are exact and summed in fp32: outputs are held to their rounding.  Odd numbers of rows in BackwardData and
    images of other than a multiple of four pixels stay with the tile GEMMs."""
    s = _layer(*case[:5], op)
    bits, (x, w, dy) = bf16_inputs(s, seed=65)
    ref = run_oracle(s, op, x=x, w=w, dy=dy)
    kernel = ucd.ucd_describe_micro(ucd.layer(s, dtype=1), op, I, s.N)[0]
    name = "pointwise_stream_kernel<" if case in STREAM else "pointwise_bf16_kernel<"
    assert kernel.startswith(name) == (op in (case[5] if len(case) > 5 else (F, D))), kernel
    for parts in [s.N], [1, s.N - 1]:
        if min(parts) > 0:
            check_bf16_output(run_hip_bf16(s, op, [(I, b) for b in parts], bits), ref, ucd.OP_NAMES[op])


@pytest.mark.parametrize("op", (F, D))
@pytest.mark.parametrize("case", [HALF[0], STREAM[3], STREAM[4]], ids=str)
def test_pointwise_bf16_not_finite(case, op):
    """An infinity or a NaN reaches the outputs of its pixel or of its filter row, and no other."""
    s = _layer(*case, op)
    bits, (x, w, dy) = bf16_inputs(s, seed=66)
    clean = run_hip_bf16(s, op, [(I, s.N)], bits)
    t = bits[0 if op == F else 2]
    t[3, 5, 7, 9], t[-1, -1, -1, -1] = 0x7F80, 0x7FC0
    bits[1][(17, 3) if op == F else (3, 17)] = 0xFF80
    got = run_hip_bf16(s, op, [(I, s.N)], bits)
    hit = np.zeros(got.shape, bool)
    hit[3, :, 7, 9] = hit[-1, :, -1, -1] = hit[:, 17] = True
    assert not np.isfinite(got[hit]).any() and np.array_equal(got[~hit], clean[~hit])


@pytest.mark.parametrize("det", (0, 1))
@pytest.mark.parametrize("op", (F, D))
@pytest.mark.parametrize("case", [HALF[1], HALF[9], STREAM[1], STREAM[10]], ids=str)
def test_pointwise_bf16_gives_the_same_bits_in_every_run(case, op, det):
    s = _layer(*case[:5], op)
    bits, _ = bf16_inputs(s, seed=67)
    prev = ucd.ucd_set_deterministic(det)
    try:
        runs = [run_hip_bf16(s, op, [(I, s.N)], bits) for _ in range(3)]
    finally:
        ucd.ucd_set_deterministic(prev)
    assert all(np.array_equal(runs[0], r) for r in runs[1:])


@pytest.mark.parametrize("op", (F, D))
@pytest.mark.parametrize("dtype,case", [(1, HALF[0]), (1, HALF[1]), (1, HALF[6]), (1, HALF[10]), (1, STREAM[1]), (1, STREAM[2]), (1, STREAM[5]),
                                        (1, STREAM[10]), (0, CASES[0]), (0, CASES[2]), (0, CASES[5]), (0, STREAM32[0]), (0, STREAM32[4])], ids=str)
def test_pointwise_tensors_on_any_element(case, op, dtype):
    """Tensors have to be aligned to their element size only: inputs, filter and output one element behind an aligned
    address give the bits of aligned ones, and the elements before and behind the output stay."""
    import torch
    s = _layer(*case[:5], op)
    kind = torch.bfloat16 if dtype else torch.float32
    if dtype:
        bits, _ = bf16_inputs(s, seed=68)
        ref = run_hip_bf16(s, op, [(I, s.N)], bits)
    else:
        bits = inputs(s, seed=68)
        ref = _run(s, op, *bits)

    def shifted(b):
        t = torch.full((b.size + 64,), 3.0, dtype=kind, device="cuda:0")
        t[1:1 + b.size] = (dev_bf16(b) if dtype else torch.from_numpy(b).to("cuda:0")).flatten()
        return t

    a, w = shifted(bits[0 if op == F else 2]), shifted(bits[1])
    out = torch.full((ref.size + 64,), 3.0, dtype=kind, device="cuda:0")
    plan = ucd.ucd_plan_fixed(ucd.layer(s, dtype=dtype), op, [(I, s.N)])
    run = ucd.ucd_conv_fwd if op == F else ucd.ucd_conv_bwd_data
    run(plan, a[1:], w[1:], out[1:], None, 0)
    got = out.float().cpu().numpy()
    assert np.array_equal(got[1:1 + ref.size], ref.ravel())
    assert got[0] == 3.0 and (got[1 + ref.size:] == 3.0).all()
