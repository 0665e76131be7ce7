"""conv_window_kernel (Forward and BackwardData of bf16 3x3 stride-1 layers over a window in LDS): every tile at edges of its
channels and positions, chunks of 16 channels that the last one does not fill, column blocks, tiles over several images, paddings
of 0, 1 and 2 and of rows and columns apart, tensors on any element, infinities and NaN, layers that it does not take.

The reference is torch's convolution of the same bf16 values on the CPU in fp32, whose sums are off by a few 1e-7 of the results' rms: the
bounds are those of test_gpu_bf16.py for products of bf16 operands (half a unit of the result's last place, 1e-5 rms)."""
import numpy as np
import pytest

from paper_1804_04806_amd import ucd
from hip_helpers import desc_of, rect
from test_gpu_bf16 import bf16_inputs, check_bf16_output, run_hip_bf16

pytestmark = pytest.mark.gpu

F, D, I = ucd.FWD, ucd.BWD_DATA, ucd.ALGO_IMPLICIT


def layer(n, c, h, w, k, ph, pw):
    return rect(n, c, h, w, k, 3, 3, (1, 1), (ph, pw))


def reference(s, op, x, w, dy):
    import torch
    x, w, dy = (torch.from_numpy(np.ascontiguousarray(a)) for a in (x, w, dy))
    if op == F:
        return torch.nn.functional.conv2d(x, w, padding=(s.pad, s.pad_w)).numpy()
    return torch.nn.functional.conv_transpose2d(dy, w, padding=(s.pad, s.pad_w)).numpy()


def described(s, op):
    return ucd.ucd_describe_micro(desc_of(s, dtype=1), op, I, s.N)[0]


# (layer, the tile that Forward takes, that of BackwardData): channels around 32, 64 and 128 rows and chunks of 16, images whose
# rows are blocks of columns (56, 57 and 100), rows of four pixels, positions over one and over many images
CASES = [
    (layer(70, 34, 13, 13, 130, 1, 1), "32x256", "32x256"), (layer(33, 62, 28, 30, 70, 1, 0), "64x256", "32x256"),
    (layer(60, 34, 20, 21, 66, 0, 2), "64x256", "32x256"), (layer(129, 98, 13, 13, 130, 1, 1), "32x256", "64x256"),
    (layer(300, 50, 13, 15, 260, 1, 1), "64x512", "64x256"), (layer(40, 48, 56, 57, 200, 2, 1), "64x512", "64x512"),
    (layer(90, 130, 28, 28, 128, 1, 1), "128x512", "64x512"), (layer(130, 256, 14, 14, 256, 1, 1), "64x512", "64x512"),
    (layer(9, 30, 45, 29, 100, 2, 0), "32x256", "32x256"), (layer(7, 22, 30, 100, 70, 1, 1), "32x256", "32x256"),
    (layer(250, 44, 16, 4, 33, 0, 1), "32x256", "32x256"), (layer(256, 254, 13, 13, 250, 0, 2), "64x512", "128x512"),
]


@pytest.mark.parametrize("op", [F, D], ids=["fwd", "bwd_data"])
@pytest.mark.parametrize("s,fwd,bwd", CASES, ids=[f"n{s.N}c{s.C}h{s.H}w{s.W}k{s.K}p{s.pad}{s.pad_w}" for s, _, _ in CASES])
def test_window_edges(s, fwd, bwd, op):
    tile = fwd if op == F else bwd
    assert f"conv_window_kernel<Tile<{tile}>>" in described(s, op)
    bits, (x, w, dy) = bf16_inputs(s, seed=61)
    ref = reference(s, op, x, w, dy)
    for parts in ([s.N], [s.N - 1, 1]):
        check_bf16_output(run_hip_bf16(s, op, [(I, b) for b in parts], bits), ref, (s, op, parts))


@pytest.mark.parametrize("op", [F, D], ids=["fwd", "bwd_data"])
def test_window_on_any_element(op):
    """Micro-batches of an odd number of elements, and tensors one element behind an aligned address."""
    import torch
    s = layer(120, 34, 13, 13, 33, 1, 1)   # y has 33 * 169 elements per image
    assert "conv_window_kernel" in described(s, op)
    bits, (x, w, dy) = bf16_inputs(s, seed=62)
    ref = reference(s, op, x, w, dy)
    check_bf16_output(run_hip_bf16(s, op, [(I, 1), (I, 118), (I, 1)], bits), ref, op)
    held = []
    for b in (bits[0] if op == F else bits[2], bits[1]):
        t = torch.zeros(b.size + 1, dtype=torch.bfloat16, device="cuda:0")
        t[1:] = torch.from_numpy(b.view(np.int16)).to("cuda:0").view(torch.bfloat16).reshape(-1)
        held.append(t)
    out = torch.full((ref.size + 1,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    plan = ucd.ucd_plan_fixed(desc_of(s, dtype=1), op, [(I, s.N)])
    run = ucd.ucd_conv_fwd if op == F else ucd.ucd_conv_bwd_data
    run(plan, held[0][1:], held[1][1:], out[1:], None, 0)
    torch.cuda.synchronize()
    assert torch.isnan(out[0])
    check_bf16_output(out[1:].float().cpu().numpy().reshape(ref.shape), ref, op)


@pytest.mark.parametrize("op", [F, D], ids=["fwd", "bwd_data"])
def test_window_values_that_are_not_finite(op):
    """They reach the outputs whose windows hold them, and no other; a filter's reach the channel that they belong to."""
    s = layer(70, 34, 13, 13, 66, 1, 1)
    bits, (x, w, dy) = bf16_inputs(s, seed=63)
    src = bits[0] if op == F else bits[2]
    last = src.shape[1] - 1
    src[3, last, 0, 0], src[68, 0, 12, 12], src[40, 5, 6, 0] = 0x7F80, 0x7FC0, 0xFF80
    bits[1][65, 33, 1, 1] = 0x7FC0   # the last channels' centre tap
    got = run_hip_bf16(s, op, [(I, s.N)], bits)
    hit = np.zeros(got.shape, dtype=bool)
    hit[3, :, 0:2, 0:2] = hit[68, :, 11:13, 11:13] = hit[40, :, 5:8, 0:2] = True
    hit[:, 65 if op == F else 33] = True
    assert not np.isfinite(got[hit]).any() and np.isfinite(got[~hit]).all()


@pytest.mark.parametrize("s", [layer(200, 33, 13, 13, 64, 1, 1), layer(200, 64, 30, 3, 64, 1, 1),
                               rect(100, 64, 20, 20, 64, 3, 3, (2, 2), (1, 1)), rect(100, 64, 20, 20, 64, 3, 5, (1, 1), (1, 2))], ids=str)
def test_layers_that_window_does_not_take(s):
    assert "conv_window_kernel" not in described(s, F) and "conv_window_kernel" not in described(s, D)
