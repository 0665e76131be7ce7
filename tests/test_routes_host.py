"""Which layers the kernels for windows in LDS take, from the dry run (no GPU)."""
import time

from paper_1804_04806_amd import ucd


def described(op, n, c, h, w, k, r, s, strides=(1, 1), pads=(0, 0), dtype=0):
    L = ucd.layer(N=n, C=c, H=h, W=w, K=k, R=r, S=s, stride_h=strides[0], stride_w=strides[1], pad_h=pads[0], pad_w=pads[1], dtype=dtype)
    return ucd.ucd_describe_micro(L, op, ucd.ALGO_IMPLICIT, n)[0]


def test_rows_kernel_keeps_the_offsets_of_its_stores_below_32_bits():
    """Rows of a tile past the last output channel are stored to 2^31 + row * plane, which the range check has to see as such: planes
    such that the tile's last row begins at 2^31 and more are not taken."""
    for n, c, h, k, r, stride in ((1, 3, 6060, 58, 7, 2), (1, 4, 4500, 26, 4, 1)):
        assert "conv_rows_kernel" not in described(ucd.FWD, n, c, h, h, k, r, r, (stride, stride))
    for n, c, h, k, r, stride in ((1, 3, 5600, 58, 7, 2), (1, 4, 4100, 26, 4, 1)):
        assert "conv_rows_kernel" in described(ucd.FWD, n, c, h, h, k, r, r, (stride, stride))


def test_loads_of_channels_past_the_last_one_keep_their_offsets_below_32_bits():
    """The same for the channels that fill up a chunk: planes such that the chunk's last one begins at 2^31 and more."""
    assert "conv_window_kernel" not in described(ucd.FWD, 1, 2, 12500, 12500, 2, 3, 3, pads=(1, 1), dtype=1)
    assert "conv_window_kernel" in described(ucd.FWD, 1, 2, 12000, 12000, 2, 3, 3, pads=(1, 1), dtype=1)
    for pad, kernel in ((560, False), (1, True)):   # planes of 294 MB and of 17
        assert ("conv_halo_kernel" in described(ucd.BWD_DATA, 1, 64, 64, 1 << 16, 1, 3, 3, pads=(pad, 1))) == kernel


def test_rows_kernel_with_windows_of_two_thousand_million_elements():
    """Rows of 2^23 pixels: the size of a window with all of their columns begins at 2^31."""
    for w in (8388606, 8388607, 8388608, 8388610):
        assert "conv_rows_kernel" not in described(ucd.FWD, 1, 16, 1, w, 31, 8, 4, pads=(4, 0))


def test_choice_of_a_window_does_not_take_longer_for_wider_images():
    """The blocks of columns are found without a walk over all their numbers: microseconds also for the widest images (a walk takes 0.3 to
    80 ms for these)."""
    for op, layer, dtype in ((ucd.BWD_DATA, (1, 1, 8, 500000, 32, 8, 8, (1, 1), (3, 3)), 0), (ucd.BWD_DATA, (2, 3, 64, 60000, 32, 7, 7, (1, 1), (3, 3)), 1),
                             (ucd.FWD, (1, 1, 8, 500000, 32, 8, 8, (1, 1), (3, 3)), 0), (ucd.BWD_FILTER, (1, 1, 8, 500000, 32, 8, 8, (1, 1), (3, 3)), 0),
                             (ucd.FWD, (4, 64, 3, 100000, 64, 3, 3, (1, 1), (0, 0)), 1), (ucd.BWD_DATA, (4, 64, 3, 100000, 64, 3, 3, (1, 1), (0, 0)), 0)):
        least = float("inf")
        for _ in range(20):
            t = time.perf_counter()
            described(op, *layer, dtype=dtype)
            least = min(least, time.perf_counter() - t)
        assert least < 150e-6, (op, layer, least)


def test_loads_of_the_filter_past_its_last_channel_keep_their_offsets_below_32_bits():
    """Filters of close to 2 GB, of which the channels that fill up two chunks would begin behind 2^31."""
    for k, kernel in ((58240, False), (58000, True)):
        assert ("conv_halo_kernel" in described(ucd.BWD_DATA, 1, 1024, 90, 90, k, 3, 3, pads=(1, 1))) == kernel
    for k, kernel in ((116494, False), (112000, True)):
        assert ("conv_few_kernel" in described(ucd.BWD_DATA, 1, 16, 60, 60, k, 18, 16, (2, 1), (9, 8))) == kernel


def test_layers_that_the_tile_gemms_are_faster_on():
    """Few channels, reductions or pixels that leave a window kernel's tiles mostly empty; beside each a layer of its kind that is taken."""
    def takes(kernel, *a, **k):
        return kernel in described(*a, **k)
    for dtype in (0, 1):   # BackwardData: filters no larger than the stride, few output channels
        assert not takes("conv_few_kernel", ucd.BWD_DATA, 48, 5, 136, 248, 70, 2, 2, (2, 2), (1, 1), dtype=dtype)
        assert not takes("conv_few_kernel", ucd.BWD_DATA, 12, 1, 214, 214, 1, 11, 11, pads=(5, 5), dtype=dtype)
        assert takes("conv_few_kernel", ucd.BWD_DATA, 48, 3, 136, 248, 70, 7, 7, (2, 2), (3, 3), dtype=dtype)
    assert not takes("conv_window_kernel", ucd.FWD, 59, 4, 172, 67, 36, 3, 3, dtype=1) and takes("conv_window_kernel", ucd.FWD, 59, 4, 172, 67, 36, 3, 3, pads=(1, 1), dtype=1)
    assert takes("conv_window_kernel", ucd.FWD, 59, 10, 172, 67, 36, 3, 3, dtype=1)
    for k, w, taken in ((3, 27, False), (6, 27, False), (6, 4, True), (9, 27, True)):
        assert takes("conv_window_kernel", ucd.BWD_DATA, 203, 68, 95, w, k, 3, 3, pads=(0, 1), dtype=1) == taken
    assert not takes("filter_window_kernel", ucd.BWD_FILTER, 20, 799, 141, 6, 502, 3, 3, dtype=1) and takes("filter_window_kernel", ucd.BWD_FILTER, 20, 799, 141, 7, 502, 3, 3, dtype=1)
    for r, sw, taken in ((4, 2, False), (4, 1, True), (5, 2, True)):
        assert takes("conv_rows_kernel", ucd.FWD, 100, 5, 100, 100, 64, r, 4, (2, sw), (2, 2)) == taken
    for n, taken in ((4, False), (5, True)):
        assert takes("conv_rows_kernel", ucd.FWD, n, 3, 130, 147, 640, 11, 7, (2, 2), (5, 3)) == taken
