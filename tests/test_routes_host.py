"""Which layers the kernels for windows in LDS take, from the dry run (no GPU)."""
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
