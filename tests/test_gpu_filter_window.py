"""filter_window_kernel (BackwardFilter of bf16 3x3 stride-1 layers, all taps of a block of channels at once): channels around the
blocks of 64, rows that are no whole strips of eight pixels, strips that follow each other down and along the rows, images of fewer rows
than a unit, paddings of 0, 1 and 2 and of rows and columns apart, beta = 1, values that are not finite, tensors on any element,
launches that it does not take.

The reference is the sum of products of the same bf16 values in fp64, on the device by unfolded matrix products.  dw is an fp32 sum, off by
2e-7 to 5e-7 of it in L2 with chunks of any size, and by a few times that in single elements; bounds of 2e-6 and 1e-4 rms."""
import numpy as np
import pytest

from paper_1804_04806_amd import ucd
from hip_helpers import desc_of, rect
from test_gpu_bf16 import bf16_inputs, run_hip_bf16

pytestmark = pytest.mark.gpu

B, I = ucd.BWD_FILTER, ucd.ALGO_IMPLICIT


def layer(n, c, h, w, k, ph, pw):
    return rect(n, c, h, w, k, 3, 3, (1, 1), (ph, pw))


def described(s):
    return ucd.ucd_describe_micro(desc_of(s, dtype=1), B, I, s.N)[0]


def reference(s, x, dy):
    import torch
    x, dy = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (x, dy))
    ref = torch.zeros(s.K, s.C * 9, dtype=torch.float64, device="cuda:0")
    step = max(1, int(2e8) // (s.C * 9 * s.P * s.Q * 8))
    for o in range(0, s.N, step):
        cols = torch.nn.functional.unfold(x[o:o + step].double(), 3, padding=(s.pad, s.pad_w)).transpose(0, 1).reshape(s.C * 9, -1)
        ref += dy[o:o + step].double().transpose(0, 1).reshape(s.K, -1) @ cols.t().contiguous()
    return ref.reshape(s.w_shape).cpu().numpy()


def check(got, ref, ctx):
    off = got.astype(np.float64) - ref
    rms = np.sqrt(np.mean(ref ** 2))
    assert np.linalg.norm(off) <= 2e-6 * np.linalg.norm(ref) and np.abs(off).max() <= 1e-4 * rms, (ctx, np.linalg.norm(off) / np.linalg.norm(ref))


CASES = [layer(256, 130, 13, 13, 129, 1, 1), layer(40, 130, 45, 29, 100, 1, 2), layer(30, 70, 61, 70, 130, 0, 1),
         layer(70, 200, 11, 13, 260, 2, 0), layer(8, 100, 80, 100, 200, 1, 1), layer(64, 512, 7, 7, 512, 1, 1),
         layer(451, 190, 5, 22, 193, 0, 2), layer(900, 255, 7, 7, 257, 0, 0), layer(33, 129, 34, 63, 65, 1, 0)]


@pytest.mark.parametrize("s", CASES, ids=[f"n{s.N}c{s.C}h{s.H}w{s.W}k{s.K}p{s.pad}{s.pad_w}" for s in CASES])
def test_filter_window_edges(s):
    assert "filter_window_kernel" in described(s)
    bits, (x, _, dy) = bf16_inputs(s, seed=71)
    ref = reference(s, x, dy)
    check(run_hip_bf16(s, B, [(I, s.N)], bits), ref, s)
    dw0 = np.random.default_rng(5).standard_normal(s.w_shape).astype(np.float32)
    check(run_hip_bf16(s, B, [(I, s.N - 1), (I, 1)], bits, beta=1.0, dw0=dw0), ref + dw0, s)


def test_filter_window_on_any_element():
    import torch
    s = layer(257, 129, 13, 13, 131, 1, 1)
    assert "filter_window_kernel" in described(s)
    bits, (x, _, dy) = bf16_inputs(s, seed=72)
    held = []
    for b in (bits[0], bits[2]):
        t = torch.zeros(b.size + 1, dtype=torch.bfloat16, device="cuda:0")
        t[1:] = torch.from_numpy(b.view(np.int16)).to("cuda:0").view(torch.bfloat16).reshape(-1)
        held.append(t)
    out = torch.full(s.w_shape, float("nan"), device="cuda:0")
    ucd.ucd_conv_bwd_filter(ucd.ucd_plan_fixed(desc_of(s, dtype=1), B, [(I, s.N)]), held[0][1:], held[1][1:], out, 0.0, None, 0)
    torch.cuda.synchronize()
    check(out.cpu().numpy(), reference(s, x, dy), s)


@pytest.mark.parametrize("pad", [0, 1])
def test_filter_window_values_that_are_not_finite(pad):
    """Values of x at the borders reach the taps that meet them with dy, and no other."""
    s = layer(256, 128, 13, 13, 130, pad, pad)
    assert "filter_window_kernel" in described(s)
    bits, (x, _, dy) = bf16_inputs(s, seed=73)
    bits[0][7, 3, 12, 5], bits[0][9, 70, 4, 12], bits[0][255, 127, 12, 12] = 0x7F80, 0xFF80, 0x7FC0
    bits[2][11, 129, 4, 4] = 0x7F80
    hit = np.zeros(s.w_shape, dtype=bool)
    for c, h, w in ((3, 12, 5), (70, 4, 12), (127, 12, 12)):
        for r in range(3):
            for q in range(3):
                hit[:, c, r, q] |= 0 <= h + pad - r < s.P and 0 <= w + pad - q < s.Q
    hit[129] = True
    got = run_hip_bf16(s, B, [(I, s.N)], bits)
    assert not np.isfinite(got[hit]).any() and np.isfinite(got[~hit]).all()


def test_launches_that_filter_window_does_not_take():
    small, strided = layer(32, 128, 13, 13, 128, 1, 1), rect(256, 128, 28, 28, 128, 3, 3, (2, 2), (1, 1))
    assert "filter_window_kernel" not in described(small) and "filter_window_kernel" not in described(strided)
    assert "filter_window_kernel" not in described(layer(900, 256, 20, 3, 256, 1, 1))
    assert "filter_window_kernel" not in described(layer(900, 255, 7, 6, 257, 0, 0))   # a unit's 4 x 8 pixels are mostly padding
    before = ucd.ucd_set_deterministic(1)
    try:
        assert "filter_window_kernel" not in described(CASES[0])
    finally:
        ucd.ucd_set_deterministic(before)
