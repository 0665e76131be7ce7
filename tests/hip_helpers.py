"""Shared helpers of the GPU parity tests: run the HIP path through the C-ABI binding on torch
device buffers and return numpy results; run the oracle on the same bits."""
from dataclasses import dataclass

import numpy as np

from oracle import conv as oc
from paper_1804_04806_amd import synth, ucd


@dataclass(frozen=True)
class RectShape(synth.Shape):
    """A layer whose rows have `stride` and `pad`, its columns strides and paddings of their own."""
    stride_w: int = 1
    pad_w: int = 0

    @property
    def Q(self):
        return (self.W + 2 * self.pad_w - self.S) // self.stride_w + 1


def rect(n, c, h, w, k, r, s, strides, pads):
    return RectShape(n, c, h, w, k, r, s, strides[0], pads[0], "", strides[1], pads[1])


def _columns(s):
    return getattr(s, "stride_w", s.stride), getattr(s, "pad_w", s.pad)


def desc_of(s, dtype=0):
    stride_w, pad_w = _columns(s)
    return ucd.layer(N=s.N, C=s.C, H=s.H, W=s.W, K=s.K, R=s.R, S=s.S, stride_h=s.stride, stride_w=stride_w, pad_h=s.pad,
                     pad_w=pad_w, dtype=dtype)


def oracle_layer(s):
    stride_w, pad_w = _columns(s)
    return oc.Layer(s.N, s.C, s.H, s.W, s.K, s.R, s.S, s.stride, stride_w, s.pad, pad_w)


def rel_l2(got, ref):
    got = np.asarray(got, dtype=np.float64).ravel()
    ref = np.asarray(ref, dtype=np.float64).ravel()
    den = np.linalg.norm(ref)
    return float(np.linalg.norm(got - ref) / den) if den > 0 else float(np.linalg.norm(got))


def ws_need(desc, op, micro):
    need = 0
    for a, b in micro:
        n = ucd.ucd_workspace_size(desc, op, a, b)
        assert n != ucd.WS_NA, (op, a, b)
        need = max(need, n)
    return need


# Relative-L2 bounds by what a configuration runs.  The benchmark spec gives 1e-5 for the direct /
# GEMM paths and 1e-3 for Winograd; the Winograd kernels measure 3e-7 (2x2 tiles) to 4e-6 (4x4
# tiles) and the tiled FFT 1e-7 to 2e-7, so Winograd is held to 1e-4 and the FFT to the GEMM bound.
def l2_tol(micro):
    return 1e-4 if any(a in ucd.WINOGRAD_ALGOS for a, _ in micro) else 1e-5


# Elementwise bound, as a multiple of the reference's rms: |got - ref| <= elementwise_tol * rms(ref).
# An fp32 result of rms-sized terms is off by a few 1e-7 rms per element (1e-5 rms for 4x4 Winograd
# tiles): one wrong term (a dropped tap, a neighbour's pixel) is off by about 1/sqrt(reduction
# length) of an rms, i.e. 1e-2 or more.
# With bf16 tensors the fused Winograd kernel multiplies on the bf16 matrix pipe: the transformed filter
# and patches are rounded to bf16 (a relative 2^-9 each, 16 x Ci products per output), which in a numpy
# model of the kernel leaves elements up to 1.8e-2 rms off (4.2e-3 relative L2): 3e-2 there.
def elementwise_tol(micro, bf16=False):
    if bf16 and any(a == ucd.ALGO_WINOGRAD_FUSED for a, _ in micro):
        return 3e-2
    return 1e-3 if any(a in ucd.WINOGRAD_ALGOS for a, _ in micro) else 1e-4


class GuardedWorkspace:
    """A device workspace of exactly `nbytes` usable bytes followed by a guard region; the whole
    buffer is poisoned with NaN and `check_guard` asserts that nothing outside the byte ranges a
    run was entitled to has been written."""
    GUARD = 4096
    PATTERN = 0x7FC00000   # float32 NaN as torch writes it

    def __init__(self, nbytes):
        import torch
        self.nbytes = int(nbytes)
        words = (self.nbytes + 3) // 4
        self.buf = torch.empty(words + self.GUARD // 4, dtype=torch.float32, device="cuda:0")
        self.tensor = self.buf[:max(words, 1)]
        self.ptr = self.buf.data_ptr()
        self.poison()

    def poison(self):
        self.buf.fill_(float("nan"))

    def check_guard(self, used):
        """used: a byte count (the run may have written [0, used)) or a list of (offset, bytes)."""
        import torch
        ranges = [(0, used)] if isinstance(used, int) else list(used)
        dirty = self.buf.view(torch.int32) != self.PATTERN
        for off, n in ranges:
            dirty[off // 4:(off + n + 3) // 4] = False
        bad = torch.nonzero(dirty)
        assert bad.numel() == 0, f"workspace written outside its ranges {ranges}: first at byte {4 * int(bad[0])}"


def run_hip(s, op, micro, x=None, w=None, dy=None, beta=0.0, dw0=None, poison=True):
    """Execute a forced configuration in a workspace of exactly the size the plan reports (a guard
    region behind it must stay untouched); inputs are numpy float32 arrays. Returns numpy float32."""
    import torch
    dev = torch.device("cuda:0")
    desc = desc_of(s)
    plan = ucd.ucd_plan_fixed(desc, op, micro)
    need = plan.ws_bytes
    guarded = GuardedWorkspace(need)
    ws = guarded.tensor
    fill = float("nan") if poison else 0.0
    if op == ucd.FWD:
        xd, wd = torch.from_numpy(x).to(dev), torch.from_numpy(w).to(dev)
        out = torch.full(s.y_shape, fill, dtype=torch.float32, device=dev)
        ucd.ucd_conv_fwd(plan, xd, wd, out, ws, need)
    elif op == ucd.BWD_DATA:
        dyd, wd = torch.from_numpy(dy).to(dev), torch.from_numpy(w).to(dev)
        out = torch.full(s.x_shape, fill, dtype=torch.float32, device=dev)
        ucd.ucd_conv_bwd_data(plan, dyd, wd, out, ws, need)
    else:
        xd, dyd = torch.from_numpy(x).to(dev), torch.from_numpy(dy).to(dev)
        if dw0 is not None:
            out = torch.from_numpy(dw0).to(dev).clone()
        else:
            out = torch.full(s.w_shape, fill, dtype=torch.float32, device=dev)
        ucd.ucd_conv_bwd_filter(plan, xd, dyd, out, beta, ws, need)
    torch.cuda.synchronize()
    guarded.check_guard(need)
    return out.cpu().numpy()


def run_oracle(s, op, x=None, w=None, dy=None, beta=0.0, dw0=None):
    L = oracle_layer(s)
    if op == ucd.FWD:
        return oc.conv_fwd(L, x, w)
    if op == ucd.BWD_DATA:
        return oc.conv_bwd_data(L, dy, w)
    return oc.conv_bwd_filter(L, x, dy, beta=beta, dw=dw0)


def run_oracle_zeros(s, op, x=None, w=None, dy=None):
    """The oracle with the padding (BackwardData: what surrounds dy) as zeros in the tensors: an infinity that meets one is a NaN, as in the
    kernels, where the oracle leaves such products out."""
    sw, pw = _columns(s)
    if op == ucd.BWD_DATA:
        a = [s.R + s.pad, s.S + pw]
        dy = np.pad(dy, ((0, 0), (0, 0), (a[0], a[0]), (a[1], a[1])))
        h, v = (s.P + 2 * a[0] - 1) * s.stride + s.R, (s.Q + 2 * a[1] - 1) * sw + s.S
        dx = oc.conv_bwd_data(oc.Layer(s.N, s.C, h, v, s.K, s.R, s.S, s.stride, sw, 0, 0), dy, w)
        top, left = a[0] * s.stride + s.pad, a[1] * sw + pw
        return dx[:, :, top:top + s.H, left:left + s.W]
    x = np.pad(x, ((0, 0), (0, 0), (s.pad, s.pad), (pw, pw)))
    L = oc.Layer(s.N, s.C, s.H + 2 * s.pad, s.W + 2 * pw, s.K, s.R, s.S, s.stride, sw, 0, 0)
    return oc.conv_fwd(L, x, w) if op == ucd.FWD else oc.conv_bwd_filter(L, x, dy)


def check_specials(got, ref, bound):
    """Infinities and NaN where, and as, they are in ref, and the other values within bound of it."""
    fine = np.isfinite(ref)
    assert fine.any() and not fine.all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    assert rel_l2(got[fine], ref[fine]) <= bound


def inputs(s, seed=0, idx=0):
    return synth.make_x(s, seed, idx), synth.make_w(s, seed, idx), synth.make_dy(s, seed, idx)


def not_finite_time_ratio(s, op, dtype):
    """Time of an implicit-GEMM launch on tensors that hold nothing but infinities and NaN, over its ordinary time: the larger of the two for
    the data and for the filter (best of four runs of three launches)."""
    import torch
    plan = ucd.ucd_plan_fixed(desc_of(s, dtype=dtype), op, [(ucd.ALGO_IMPLICIT, s.N)])
    kind = torch.bfloat16 if dtype else torch.float32
    t, w = (torch.randn(shape, device="cuda:0").to(kind) for shape in (s.x_shape if op == ucd.FWD else s.y_shape, s.w_shape))
    out = torch.empty(s.y_shape if op == ucd.FWD else s.x_shape, device="cuda:0", dtype=kind)
    run = ucd.ucd_conv_fwd if op == ucd.FWD else ucd.ucd_conv_bwd_data

    def best(t, w):
        ms = float("inf")
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(3):
                run(plan, t, w, out, None, 0)
            b.record()
            torch.cuda.synchronize()
            ms = min(ms, a.elapsed_time(b))
        return ms
    plain, inf = best(t, w), float("inf")
    return max(best(t2, w2) for t2, w2 in ((t * inf, w), (t * float("nan"), w), (t, w * inf), (t, w * float("nan")))) / plain


def recomputed_time_ratio(s, op):
    """Time of an implicit-GEMM launch whose filter lies below bf16's range, so that every tile is computed a second time on
    the fp32 instructions, over its ordinary time (best of six runs of five launches)."""
    import torch
    plan = ucd.ucd_plan_fixed(desc_of(s), op, [(ucd.ALGO_IMPLICIT, s.N)])
    t, w = (torch.randn(shape, device="cuda:0") for shape in (s.x_shape if op == ucd.FWD else s.y_shape, s.w_shape))
    out = torch.empty(s.y_shape if op == ucd.FWD else s.x_shape, device="cuda:0")
    run = ucd.ucd_conv_fwd if op == ucd.FWD else ucd.ucd_conv_bwd_data
    ms = []
    for scale in (1.0, 2.0 ** -120):
        w *= scale
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                run(plan, t, w, out, None, 0)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        ms.append(best)
    return ms[1] / ms[0]
