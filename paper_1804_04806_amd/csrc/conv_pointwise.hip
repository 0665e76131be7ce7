// Launch of pointwise_kernel: Forward and BackwardData of fp32 1x1 stride-1 layers.
#include "conv_pointwise.hpp"
#include "gemm_launch.hpp"
#include "implicit_common.hpp"

namespace ucd {

// Where it is the faster one: its input channels fit LDS and are enough that the products outweigh the stores, and its
// pixels give most CUs a workgroup.  Time of the tile GEMMs / of this kernel over 430 layers, least and mean, more than 128
// output channels: 17 to 160 input channels and 4000 pixels or more 0.99 / 1.24 (128 -> 512 28x28 b = 128 131 / 94 us, 160 ->
// 1024 up to 1.77), 800 to 4000 pixels 0.87 to 1.6, 16 channels 0.82 / 1.0.  Up to 128 output channels the input is used once:
// 8000 to 20000 pixels, a single round, 1.04 / 1.36, more 0.83 to 1.28.
bool pointwise_pays(const Dims &d, int op, int b)
{
    if (d.dtype != 0 || d.R * d.S != 1 || d.sh != 1 || d.sw != 1 || d.ph != 0 || d.pw != 0) return false;
    const int K = op == 0 ? d.C : d.K, M = op == 0 ? d.K : d.C;
    const long cols = (long)b * d.H * d.W;
    if (K <= 16 || K > PointwiseTile::kMaxK || (long)d.H * d.W > 1l << 22) return false;   // (rows of a tile below 2^31 bytes apart)
    return M > 128 ? cols >= 4000 : M > 64 && cols >= 8000 && cols <= 20000;
}

hipError_t pointwise_conv(const Dims &d, int op, int b, const void *in, const void *w, void *out, hipStream_t s)
{
    PointwiseParams p{};
    p.x = in; p.w = w; p.y = out;
    p.w_bytes = wbytes(d);
    p.x_bytes = op == 0 ? xbytes(d, b) : ybytes(d, b);
    p.y_bytes = op == 0 ? ybytes(d, b) : xbytes(d, b);
    p.K = op == 0 ? d.C : d.K;
    p.M = op == 0 ? d.K : d.C;
    p.px = d.H * d.W; p.cols = b * p.px;
    p.w_row = op == 0 ? d.C : 1;
    p.w_k = op == 0 ? 1 : d.C;
    p.div_px = FastDiv(p.px);
    typedef PointwiseTile T;
    const int tiles = (p.cols + T::NT - 1) / T::NT, slots = device_cus();
    p.m_tiles = (p.M + T::MT - 1) / T::MT;
    p.whole = tiles / slots * slots;
    const int over = tiles - p.whole;
    p.splits = over == 0 ? 1 : slots / over < 1 ? 1 : slots / over < p.m_tiles ? slots / over : p.m_tiles;
    const unsigned grid = (unsigned)(p.whole + over * p.splits);
    if (LaunchLog *log = launch_log()) {
        log->add("gemm_kernel_split_pointwise<Tile<" + std::to_string(T::MT) + "x" + std::to_string(T::NT) + ">," +
                 (op == 0 ? "forward" : "backward data") + "> tiles=" + std::to_string(tiles) + " splits=1 batch=1 M=" +
                 std::to_string(p.M) + " N=" + std::to_string(p.cols) + " K=" + std::to_string(p.K));
        return hipSuccess;
    }
    if (p.px % 4 == 0) {
        if (op == 0) pointwise_kernel<true, true><<<grid, T::THREADS, 0, s>>>(p);
        else pointwise_kernel<false, true><<<grid, T::THREADS, 0, s>>>(p);
    } else {
        if (op == 0) pointwise_kernel<true, false><<<grid, T::THREADS, 0, s>>>(p);
        else pointwise_kernel<false, false><<<grid, T::THREADS, 0, s>>>(p);
    }
    return hipGetLastError();
}

}  // namespace ucd
