"""The C-ABI library loads without a GPU and exports every symbol include/*.h declares."""
import ctypes
import itertools
import os
import re

from paper_1804_04806_amd import ucd

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = "".join(open(os.path.join(ROOT, "include", h)).read() for h in ("ucd.h", "ucd_calib.h"))
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ucd_[a-z_0-9]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = declared_symbols()
    assert len(names) >= 18 and "ucd_plan" in names and "ucd_conv_bwd_filter" in names
    lib = ctypes.CDLL(ucd.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(ucd.EXPORTS) == names


def test_version_and_strerror():
    assert ucd.ucd_version() >= 100
    assert ucd.strerror(0) == "ok" and "workspace" in ucd.strerror(ucd.E_WS_TOO_SMALL)


def test_workspace_formulas():
    L = ucd.layer(N=8, C=16, H=16, W=16, K=32, R=3, S=3, pad_h=1, pad_w=1)
    assert ucd.ucd_workspace_size(L, ucd.FWD, ucd.ALGO_IMPLICIT, 8) == 0
    # im2col: 4 bytes x C*R*S x (b*P*Q rounded up to 4): 144 KiB per image here
    assert ucd.ucd_workspace_size(L, ucd.FWD, ucd.ALGO_IM2COL, 1) == 4 * 144 * 256 == 147456
    assert ucd.ucd_workspace_size(L, ucd.BWD_FILTER, ucd.ALGO_IM2COL, 3) == 3 * 147456
    assert ucd.ucd_workspace_size(L, ucd.FWD, ucd.ALGO_IM2COL, 9) == ucd.WS_NA      # b > N
    # Winograd: 64 bytes x (C*K + b*T*(C+K)), T = 8*8 tiles: 32 + 64 + 128 KiB at b = 1
    assert ucd.ucd_workspace_size(L, ucd.FWD, ucd.ALGO_WINOGRAD, 1) == 64 * (16 * 32 + 64 * 48) == 224 * 1024
    assert ucd.ucd_workspace_size(L, ucd.BWD_DATA, ucd.ALGO_WINOGRAD, 2) == 64 * (16 * 32 + 128 * 48)
    assert ucd.ucd_workspace_size(L, ucd.BWD_FILTER, ucd.ALGO_WINOGRAD, 1) == 64 * (16 * 32 + 64 * 48)
    # Winograd F(4x4,3x3): 36 planes of 4 bytes, T = 4*4 tiles
    assert ucd.ucd_workspace_size(L, ucd.FWD, ucd.ALGO_WINOGRAD4, 1) == 144 * (16 * 32 + 16 * 48)
    assert ucd.ucd_workspace_size(L, ucd.BWD_DATA, ucd.ALGO_WINOGRAD4, 3) == 144 * (16 * 32 + 48 * 48)
    assert ucd.ucd_workspace_size(L, ucd.BWD_FILTER, ucd.ALGO_WINOGRAD4, 2) == 144 * (16 * 32 + 32 * 48)
    # FFT: 144 planes of 4 bytes, 14 x 14 output tiles: T = 2*2, 2C*2K + ld*(2C + 2K)
    assert ucd.ucd_workspace_size(L, ucd.FWD, ucd.ALGO_FFT, 3) == 4 * 144 * (32 * 64 + 12 * 96)
    assert ucd.ucd_workspace_size(L, ucd.BWD_FILTER, ucd.ALGO_FFT, 1) == 4 * 144 * (4 * 32 * 16 + 4 * 96)
    # fused Winograd: the transformed filter, 64 bytes x Ci (rounded up to 8) x Co (rounded up to 4)
    assert ucd.ucd_workspace_size(L, ucd.FWD, ucd.ALGO_WINOGRAD_FUSED, 8) == 64 * 16 * 32
    assert ucd.ucd_workspace_size(L, ucd.BWD_FILTER, ucd.ALGO_WINOGRAD_FUSED, 8) == 64 * 16 * 32
    Lc3 = ucd.layer(N=8, C=3, H=16, W=16, K=30, R=3, S=3, pad_h=1, pad_w=1)
    assert ucd.ucd_workspace_size(Lc3, ucd.FWD, ucd.ALGO_WINOGRAD_FUSED, 1) == 64 * 8 * 32
    assert ucd.ucd_workspace_size(Lc3, ucd.BWD_DATA, ucd.ALGO_WINOGRAD_FUSED, 1) == 64 * 32 * 4
    # strided BackwardData with three taps per phase and axis: a 3x3 convolution from K to C * stride^2 channels
    L11s4 = ucd.layer(N=4, C=3, H=35, W=35, K=20, R=11, S=11, pad_h=2, pad_w=2, stride_h=4, stride_w=4)
    assert ucd.ucd_workspace_size(L11s4, ucd.BWD_DATA, ucd.ALGO_WINOGRAD_FUSED, 4) == 64 * 24 * 48
    assert ucd.ucd_workspace_size(L11s4, ucd.FWD, ucd.ALGO_WINOGRAD_FUSED, 4) == ucd.WS_NA
    assert ucd.ucd_workspace_size(L11s4, ucd.BWD_FILTER, ucd.ALGO_WINOGRAD_FUSED, 4) == ucd.WS_NA
    # mirrored filter copy: BackwardData of stride-1 layers only, the filter's own size (16-byte multiple)
    assert ucd.ucd_workspace_size(L, ucd.BWD_DATA, ucd.ALGO_IMPLICIT_MIRROR, 5) == 4 * 32 * 16 * 9
    assert ucd.ucd_workspace_size(L, ucd.FWD, ucd.ALGO_IMPLICIT_MIRROR, 5) == ucd.WS_NA
    assert ucd.ucd_workspace_size(L, ucd.BWD_FILTER, ucd.ALGO_IMPLICIT_MIRROR, 5) == ucd.WS_NA
    Lb = ucd.layer(N=8, C=3, H=16, W=16, K=5, R=3, S=3, pad_h=1, pad_w=1, dtype=1)
    assert ucd.ucd_workspace_size(Lb, ucd.BWD_DATA, ucd.ALGO_IMPLICIT_MIRROR, 1) == 272   # 2 x 135 -> 16-byte multiple
    # Winograd F(2x2,5x5), fused: 36 planes of the transformed filter (Ci rounded up to 8, Co to 4);
    # BackwardFilter: the 36 K x C product planes; 5x5 stride-1 layers with horizontal padding 2, fp32
    L5 = ucd.layer(N=8, C=20, H=16, W=16, K=30, R=5, S=5, pad_h=2, pad_w=2)
    assert ucd.ucd_workspace_size(L5, ucd.FWD, ucd.ALGO_WINOGRAD5_FUSED, 8) == 144 * 24 * 32
    assert ucd.ucd_workspace_size(L5, ucd.BWD_DATA, ucd.ALGO_WINOGRAD5_FUSED, 3) == 144 * 32 * 20
    assert ucd.ucd_workspace_size(L5, ucd.BWD_FILTER, ucd.ALGO_WINOGRAD5_FUSED, 1) == 144 * 30 * 20
    assert ucd.ucd_workspace_size(L, ucd.FWD, ucd.ALGO_WINOGRAD5_FUSED, 1) == ucd.WS_NA          # 3x3
    assert ucd.ucd_workspace_size(ucd.layer(N=8, C=20, H=16, W=16, K=30, R=5, S=5, pad_h=2, pad_w=1),
                                  ucd.FWD, ucd.ALGO_WINOGRAD5_FUSED, 1) == ucd.WS_NA             # padding 1
    assert ucd.ucd_workspace_size(ucd.layer(N=8, C=20, H=16, W=16, K=30, R=5, S=5, pad_h=2, pad_w=2, dtype=1),
                                  ucd.FWD, ucd.ALGO_WINOGRAD5_FUSED, 1) == ucd.WS_NA             # bf16
    Ls2 = ucd.layer(N=8, C=16, H=16, W=16, K=32, R=3, S=3, pad_h=1, pad_w=1, stride_h=2, stride_w=2)
    assert ucd.ucd_workspace_size(Ls2, ucd.BWD_FILTER, ucd.ALGO_WINOGRAD, 1) == ucd.WS_NA  # stride 2
    assert ucd.ucd_workspace_size(Ls2, ucd.BWD_DATA, ucd.ALGO_IMPLICIT_MIRROR, 1) == ucd.WS_NA
    assert ucd.ucd_workspace_size(Ls2, ucd.BWD_DATA, ucd.ALGO_WINOGRAD_FUSED, 1) == ucd.WS_NA  # two taps per phase
    L11 = ucd.layer(N=4, C=8, H=7, W=7, K=8, R=1, S=1)
    assert ucd.ucd_workspace_size(L11, ucd.FWD, ucd.ALGO_IM2COL, 1) == ucd.WS_NA    # col == x
    assert ucd.ucd_workspace_size(L11, ucd.FWD, ucd.ALGO_WINOGRAD, 1) == ucd.WS_NA  # not 3x3
    bad = ucd.layer(N=4, C=8, H=2, W=2, K=8, R=5, S=5)
    assert ucd.ucd_workspace_size(bad, ucd.FWD, ucd.ALGO_IMPLICIT, 1) == ucd.WS_NA


def test_plan_fixed_validation_and_query():
    import pytest
    L = ucd.layer(N=8, C=16, H=16, W=16, K=32, R=3, S=3, pad_h=1, pad_w=1)
    p = ucd.ucd_plan_fixed(L, ucd.FWD, [(0, 3), (1, 5)])
    assert p.query() == ([(0, 3), (1, 5)], 0, 5 * 147456)
    for micro, status in (([(0, 3), (0, 4)], ucd.E_INVALID), ([(0, 0), (0, 8)], ucd.E_INVALID),
                          ([(ucd.N_ALGO, 8)], ucd.E_INVALID)):
        with pytest.raises(ucd.UcdError) as e:
            ucd.ucd_plan_fixed(L, ucd.FWD, micro)
        assert e.value.status == status


def test_execution_rejects_bad_calls_before_any_launch():
    import pytest
    L = ucd.layer(N=8, C=16, H=16, W=16, K=32, R=3, S=3, pad_h=1, pad_w=1)
    p = ucd.ucd_plan_fixed(L, ucd.FWD, [(1, 8)])
    lib = ucd.lib()
    # null tensors
    assert lib.ucd_conv_fwd(p.handle, None, None, None, None, 0, None) == ucd.E_NULLPTR
    # workspace one byte short (fake non-null addresses are never dereferenced on this path)
    assert lib.ucd_conv_fwd(p.handle, 4096, 4096, 4096, 4096, 8 * 147456 - 1, None) == ucd.E_WS_TOO_SMALL
    # wrong operation for this plan
    assert lib.ucd_conv_bwd_data(p.handle, 4096, 4096, 4096, 4096, 1 << 30, None) == ucd.E_INVALID
    pf = ucd.ucd_plan_fixed(L, ucd.BWD_FILTER, [(0, 8)])
    assert lib.ucd_conv_bwd_filter(pf.handle, 4096, 4096, 4096, 0.5, None, 0, None) == ucd.E_INVALID
    # a table plan has no layer attached
    t = [[ucd.TIME_INF, 5, 9]]
    pt = ucd.ucd_plan_from_table(2, 0, ucd.POLICY_ALL, t, [[ucd.WS_NA, 0, 0]])
    assert lib.ucd_conv_fwd(pt.handle, 4096, 4096, 4096, None, 0, None) == ucd.E_INVALID


def test_run_micro_rejects_a_micro_batch_beyond_the_descriptor():
    """The descriptor's N is the extent of the caller's buffers: b > N (or b < 1) is an error
    before anything is launched, and so is a bf16 tensor pointer that is not 2-byte aligned."""
    import ctypes as C
    L = ucd.layer(N=8, C=16, H=16, W=16, K=32, R=3, S=3, pad_h=1, pad_w=1)
    lib = ucd.lib()
    for b in (0, 9, 1 << 20):
        assert lib.ucd_run_micro(C.byref(L), ucd.FWD, ucd.ALGO_IMPLICIT, b, 4096, 4096, 4096, 0.0,
                                 None, 0, None) == ucd.E_INVALID
    Lh = ucd.layer(N=8, C=16, H=16, W=16, K=32, R=3, S=3, pad_h=1, pad_w=1, dtype=1)
    assert lib.ucd_run_micro(C.byref(Lh), ucd.FWD, ucd.ALGO_IMPLICIT, 8, 4097, 4096, 4096, 0.0,
                             None, 0, None) == ucd.E_INVALID
    Lbad = ucd.layer(N=8, C=16, H=16, W=16, K=32, R=3, S=3, pad_h=1, pad_w=1, dtype=2)
    assert lib.ucd_run_micro(C.byref(Lbad), ucd.FWD, ucd.ALGO_IMPLICIT, 8, 4096, 4096, 4096, 0.0,
                             None, 0, None) == ucd.E_INVALID


def test_reproducible_mode_workspace_sizes():
    """In the reproducible mode BackwardFilter is the implicit GEMM's alone and needs one K*C*R*S
    plane per reduction chunk; Forward / BackwardData sizes do not change."""
    L = ucd.layer(N=64, C=64, H=28, W=28, K=96, R=3, S=3, pad_h=1, pad_w=1)
    before = [[ucd.ucd_workspace_size(L, op, a, 64) for a in range(ucd.N_ALGO)] for op in range(3)]
    assert before[ucd.BWD_FILTER][ucd.ALGO_IMPLICIT] == 0
    assert ucd.ucd_set_deterministic(1) == 0
    try:
        assert ucd.ucd_set_deterministic(-1) == 1
        after = [[ucd.ucd_workspace_size(L, op, a, 64) for a in range(ucd.N_ALGO)] for op in range(3)]
        assert after[ucd.FWD] == before[ucd.FWD] and after[ucd.BWD_DATA] == before[ucd.BWD_DATA]
        need = after[ucd.BWD_FILTER][ucd.ALGO_IMPLICIT]
        plane = 4 * 96 * 64 * 9
        assert need % plane == 0 and 2 <= need // plane and need <= 32 << 20
        assert all(after[ucd.BWD_FILTER][a] == ucd.WS_NA for a in range(1, ucd.N_ALGO))
    finally:
        assert ucd.ucd_set_deterministic(0) == 1
    assert [[ucd.ucd_workspace_size(L, op, a, 64) for a in range(ucd.N_ALGO)] for op in range(3)] == before


def test_reproducible_backward_filter_prices_the_planes_it_launches():
    """One K*C*R*S plane per reduction chunk, for both element types: the bytes that ucd_workspace_size reports
    are those of the `splits=` planes that the launch writes (and the sum that follows reads), no more and no fewer."""
    planes_of = {}
    assert ucd.ucd_set_deterministic(1) == 0
    try:
        for dtype in (0, 1):
            for n, h, w, c, k, r, stride, pad in itertools.product((1, 8, 32), (13, 28), (14, 28), (16, 65), (24, 64, 130),
                                                                  (1, 3, 7), (1, 2), (0, 1)):
                L = ucd.layer(N=n, C=c, H=h, W=w, K=k, R=r, S=r, pad_h=pad, pad_w=pad, stride_h=stride,
                              stride_w=stride, dtype=dtype)
                text = ucd.ucd_describe_micro(L, ucd.BWD_FILTER, ucd.ALGO_IMPLICIT, n)[0]
                need = ucd.ucd_workspace_size(L, ucd.BWD_FILTER, ucd.ALGO_IMPLICIT, n)
                planes = int(re.search(r"splits=(\d+)", text).group(1))
                assert need == (4 * planes * k * c * r * r if "reduce_partials_kernel" in text else 0), text
                assert ("reduce_partials_kernel" in text) == (planes > 1), text
                planes_of.setdefault("bf16q" in text, set()).add(planes)
    finally:
        assert ucd.ucd_set_deterministic(0) == 1
    assert all(len(v) > 3 for v in planes_of.values()) and len(planes_of) == 2   # both kernels, many chunk counts


def _bwd_filter_launch(n, c, hw, k, r, stride=1):
    L = ucd.layer(N=n, C=c, H=hw, W=hw, K=k, R=r, S=r, pad_h=r // 2, pad_w=r // 2, stride_h=stride, stride_w=stride, dtype=1)
    text = ucd.ucd_describe_micro(L, ucd.BWD_FILTER, ucd.ALGO_IMPLICIT, n)[0]
    return text, int(re.search(r"tiles=(\d+)", text).group(1)) * int(re.search(r"splits=(\d+)", text).group(1))


def test_bf16_backward_filter_launch_rules():
    """Workgroups of the kernel that reads runs of pixels: one round of two per CU (three of 64 x 64 and 32 x 128 tiles),
    not a second one of half as long chunks; and wide tiles that are mostly padding stay with the element-wise kernel."""
    for case, most in (((16, 128, 56, 128, 3), 512), ((64, 128, 32, 128, 3), 512), ((64, 64, 32, 64, 3), 768),
                       ((64, 32, 32, 24, 5), 768), ((64, 32, 56, 32, 3), 768), ((16, 128, 56, 256, 1), 512)):
        text, wgs = _bwd_filter_launch(*case)
        assert "gemm_kernel_bf16q" in text and 0.7 * most <= wgs <= most, (case, wgs, text)
    for case in ((64, 3, 32, 256, 3), (32, 3, 56, 96, 3), (16, 32, 56, 192, 1)):
        text, _ = _bwd_filter_launch(*case)
        assert "gemm_kernel_bf16<" in text, (case, text)


def test_fp32_forward_short_reductions_stay_on_the_fp32_kernel():
    """Layers whose tiles have few reduction steps, by which kernel they run (the split kernel's tiles start and end
    slower): first layers, small launches, and the same layers with more input channels."""
    def kernel(n, c, hw, k, r):
        L = ucd.layer(N=n, C=c, H=hw, W=hw, K=k, R=r, S=r, pad_h=r // 2, pad_w=r // 2)
        return ucd.ucd_describe_micro(L, ucd.FWD, ucd.ALGO_IMPLICIT, n)[0].split("gemm_kernel")[1].split("<")[0]
    for case in ((8, 3, 224, 64, 3), (32, 1, 56, 96, 5), (32, 8, 56, 40, 3), (2, 16, 28, 128, 3), (8, 192, 14, 64, 1)):
        assert kernel(*case) == "", case
    for case in ((8, 16, 224, 64, 3), (32, 16, 56, 96, 3), (32, 8, 56, 128, 3), (2, 32, 28, 128, 3), (8, 512, 14, 64, 1)):
        assert kernel(*case) == "_split", case


def test_fused_winograd_kernel_by_channels():
    """fp32 layers of few input channels: the split kernel from 32 on, with more than 64 output channels from 41 on."""
    def split(c, k, op=ucd.FWD):
        L = ucd.layer(N=8, C=c, H=28, W=28, K=k, R=3, S=3, pad_h=1, pad_w=1)
        return "wino_fused_split_kernel" in ucd.ucd_describe_micro(L, op, ucd.ALGO_WINOGRAD_FUSED, 8)[0]
    assert [split(c, 64) for c in (31, 32, 40)] == [False, True, True]
    assert [split(c, 128) for c in (32, 40, 41)] == [False, False, True]
    assert [split(k, c, ucd.BWD_DATA) for c, k in ((128, 40), (41, 128))] == [True, True]
    assert not split(128, 40, ucd.BWD_DATA)


def test_fp32_backward_filter_kernel_by_layer():
    """Strided layers whose runs of four pixels break, and padded ones of more than 31 taps, run on the split kernel from
    a number of multiplications on; other layers of more than 32 output channels do unless they are small."""
    def split(n, c, hw, k, r, stride=1, pad=None):
        p = r // 2 if pad is None else pad
        L = ucd.layer(N=n, C=c, H=hw, W=hw, K=k, R=r, S=r, pad_h=p, pad_w=p, stride_h=stride, stride_w=stride)
        text = ucd.ucd_describe_micro(L, ucd.BWD_FILTER, ucd.ALGO_IMPLICIT, n)[0]
        return "gemm_kernel_split" in text or "filter_few_kernel" in text
    for case in ((16, 3, 14, 64, 7, 2), (128, 3, 28, 256, 7, 2), (64, 32, 14, 128, 3, 2), (16, 16, 14, 64, 7, 1), (8, 64, 28, 32, 3),
                 (64, 3, 32, 128, 3)):
        assert not split(*case), case
    for case in ((128, 3, 224, 64, 7, 2), (128, 64, 58, 128, 3, 2), (64, 16, 14, 64, 7, 1), (8, 64, 28, 33, 3), (168, 64, 14, 64, 1),
                 (256, 3, 227, 96, 11, 4, 0)):
        assert split(*case), case


def test_small_layers_by_tiles_and_rows():
    """fp32 layers run on gemm_kernel_small up to a number of 16 x 16 output tiles and reduction rows, whatever their
    channels: no layer is taken while a smaller one of its kind is not."""
    def small(op, n, c, hw, k, r=3, stride=1):
        L = ucd.layer(N=n, C=c, H=hw, W=hw, K=k, R=r, S=r, pad_h=r // 2, pad_w=r // 2, stride_h=stride, stride_w=stride)
        return "gemm_kernel_small" in ucd.ucd_describe_micro(L, op, ucd.ALGO_IMPLICIT, n)[0]
    for r, stride in ((1, 1), (3, 1), (3, 2), (5, 1), (7, 2)):
        for hw in (7, 14, 28):
            for c in (16, 64, 128):
                for op in (ucd.FWD, ucd.BWD_FILTER):
                    got = [small(op, 1, c, hw, k, r, stride) for k in range(16, 513, 16)]
                    assert got == sorted(got, reverse=True), (op, c, hw, r, stride, got)
    # Forward up to 256 tiles and 2560 rows
    assert all(small(ucd.FWD, n, *layer) for layer in ((128, 14, 128), (256, 7, 256)) for n in (1, 2))
    assert small(ucd.FWD, 4, 256, 7, 256) and not small(ucd.FWD, 3, 128, 14, 128, 5) and not small(ucd.FWD, 8, 256, 7, 256)
    # BackwardFilter up to 128 tiles with 4096 rows of each, 512 tiles with 512 rows
    assert all(small(ucd.BWD_FILTER, 1, 16, 28, k) for k in (32, 33, 64)) and small(ucd.BWD_FILTER, 2, 64, 14, 128)
    assert not small(ucd.BWD_FILTER, 8, 64, 28, 33) and not small(ucd.BWD_FILTER, 3, 64, 14, 128)


def test_descriptions_name_kernels_of_the_sources():
    """ucd_describe_micro's names are those of the kernels that a trace of the same call shows."""
    kernels = set()
    for name in os.listdir(os.path.join(ROOT, "paper_1804_04806_amd", "csrc")):
        with open(os.path.join(ROOT, "paper_1804_04806_amd", "csrc", name)) as f:
            kernels |= set(re.findall(r"__global__[^;{]*?\bvoid\s+(\w+)\(", f.read()))
    seen = set()
    for dtype in (0, 1):
        for n, c, hw, k, r, stride, pad in ((8, 16, 16, 32, 3, 1, 1), (64, 64, 56, 128, 3, 2, 1), (64, 128, 28, 512, 1, 1, 0),
                                            (64, 512, 28, 128, 1, 1, 0), (64, 3, 224, 64, 7, 2, 3), (64, 96, 27, 256, 5, 1, 2),
                                            (64, 256, 14, 256, 3, 1, 1), (16, 768, 28, 64, 1, 1, 0), (16, 24, 33, 40, 3, 1, 0)):
            L = ucd.layer(N=n, C=c, H=hw, W=hw, K=k, R=r, S=r, pad_h=pad, pad_w=pad, stride_h=stride, stride_w=stride, dtype=dtype)
            for op in range(3):
                for algo in range(ucd.N_ALGO):
                    if ucd.ucd_workspace_size(L, op, algo, n) != ucd.WS_NA:
                        text, launches = ucd.ucd_describe_micro(L, op, algo, n)
                        parts = [re.match(r"\w+", p.strip()).group(0) for p in text.split(";") if p.strip()]
                        assert len(parts) == launches, text
                        seen |= set(parts)
    assert seen <= kernels, seen - kernels
    assert seen >= {"conv_halo_kernel", "gemm_kernel_small", "pointwise_kernel", "pointwise_split_stream_kernel",
                    "pointwise_bf16_kernel", "pointwise_stream_kernel"}, seen


def test_bf16_1x1_layers_of_few_output_channels_by_rounds_of_workgroups():
    """The streaming kernel's tiles are mostly padding there: layers with one more round of few workgroups, or many rounds,
    run on the tile GEMMs."""
    def stream(op, n, few, many):
        L = ucd.layer(N=n, C=many if op == ucd.FWD else few, H=28, W=28, K=few if op == ucd.FWD else many, R=1, S=1, dtype=1)
        return "pointwise_stream_kernel" in ucd.ucd_describe_micro(L, op, ucd.ALGO_IMPLICIT, n)[0]
    # 65536 pixels are a round: b = 83 fills the first, 84 begins the second, 160 fills most of it, 168 begins the third
    assert [stream(ucd.FWD, n, 32, 256) for n in (50, 83, 84, 110, 160, 168, 336)] == [True, True, False, False, True, False, False]
    assert [stream(ucd.FWD, n, 32, 128) for n in (83, 84, 110, 168)] == [True, False, True, False]
    assert [stream(ucd.FWD, n, 64, 512) for n in (83, 84, 160, 168)] == [True, False, True, False]
    assert all(stream(ucd.FWD, n, 64, 128) for n in (83, 84, 168, 336)) and all(stream(ucd.FWD, n, 32, 32) for n in (83, 84, 336))
    assert [stream(ucd.BWD_DATA, n, 32, 256) for n in (83, 84, 160, 168)] == [True, True, True, False]
    assert [stream(ucd.BWD_DATA, n, 64, 256) for n in (84, 168)] == [True, False] and stream(ucd.BWD_DATA, 168, 64, 640)


def test_strided_backward_data_of_many_channels_and_few_pixels_splits_the_reduction():
    """conv_halo_kernel walks over all channels in one workgroup: only with enough pixels to fill the chip that way."""
    def halo(n, c, hw, k, r, stride_h=2):
        L = ucd.layer(N=n, C=c, H=hw, W=hw, K=k, R=r, S=r, pad_h=r // 2, pad_w=r // 2, stride_h=stride_h, stride_w=2)
        return "conv_halo_kernel" in ucd.ucd_describe_micro(L, ucd.BWD_DATA, ucd.ALGO_IMPLICIT, n)[0]
    assert halo(4, 256, 14, 384, 3) and all(halo(n, 256, 28, k, 3) for n, k in ((4, 256), (8, 512), (16, 1024), (16, 2048)))
    assert not any(halo(n, 256, 14, 1024, 3) for n in (1, 2, 8)) and not any(halo(n, 512, 14, 2048, 3) for n in (1, 8))
    assert [halo(n, 128, 28, 768, 3) for n in (1, 4, 24)] == [False, False, True]
    assert halo(40, 96, 28, 512, 5) and halo(4, 96, 28, 160, 5) and halo(32, 128, 28, 768, 5) and not halo(1, 512, 14, 1024, 5)
    # a row stride of 1: more filter rows per workgroup, fewer launches of the other kernels
    assert [halo(n, 128, 28, 384, 3, 1) for n in (1, 8, 24)] == [False, False, True] and halo(8, 128, 28, 64, 3, 1)
    assert halo(4, 96, 28, 96, 5, 1) and halo(24, 96, 28, 96, 5, 1)
    # few channels, all phases in one launch that splits no sum: 853 us against 386 (17x17, 5x3), or with few products 12 against 20
    def few(n, c, hw, k, r, s, stride_h):
        L = ucd.layer(N=n, C=c, H=hw, W=hw, K=k, R=r, S=s, pad_h=r // 2, pad_w=s // 2, stride_h=stride_h, stride_w=2)
        return "conv_halo_kernel" in ucd.ucd_describe_micro(L, ucd.BWD_DATA, ucd.ALGO_IMPLICIT, n)[0]
    assert few(1, 20, 17, 1703, 5, 3, 2) and few(5, 19, 83, 890, 5, 3, 2) and few(10, 21, 34, 1364, 4, 3, 2)
    assert not few(3, 20, 75, 58, 3, 5, 3) and not few(34, 19, 27, 36, 4, 5, 3)


def test_reproducible_mode_keeps_layers_whose_reduction_the_other_kernels_would_split():
    """Strided and 1x1 BackwardData: the implicit GEMMs are the faster ones there only where they may split a sum."""
    strided = ucd.layer(N=1, C=256, H=14, W=14, K=1024, R=3, S=3, pad_h=1, pad_w=1, stride_h=2, stride_w=2)
    wide = ucd.layer(N=1, C=512, H=14, W=14, K=1024, R=5, S=5, pad_h=2, pad_w=2, stride_h=2, stride_w=2)
    deep = ucd.layer(N=18, C=224, H=28, W=28, K=2344, R=1, S=1)
    second_round = ucd.layer(N=201, C=80, H=20, W=20, K=1016, R=1, S=1)
    prev = ucd.ucd_set_deterministic(0)
    try:
        for det in (0, 1):
            ucd.ucd_set_deterministic(det)
            for layer, kernel in ((strided, "conv_halo_kernel<"), (wide, "conv_halo_kernel<"),
                                  (deep, "pointwise_split_stream_kernel<"), (second_round, "pointwise_split_stream_kernel<")):
                text, _ = ucd.ucd_describe_micro(layer, ucd.BWD_DATA, ucd.ALGO_IMPLICIT, layer.N)
                assert (kernel in text) == bool(det), (det, text)
    finally:
        ucd.ucd_set_deterministic(prev)
