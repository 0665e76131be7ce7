// Launch of pointwise_kernel and pointwise_bf16_kernel: Forward and BackwardData of 1x1 stride-1 layers.
#include "conv_pointwise_bf16.hpp"
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

// bf16: from here on tiles of 256 pixels, up to here of 128, which give the chip twice the workgroups (narrow / wide tiles of
// one layer below 1.2 to 1.5, above 0.75 to 1.05 by output channels)
constexpr long kWideCols = 20000;

// The same for bf16 tensors, whose tile GEMMs are slower against it.  Time of the tile GEMMs / of this kernel, least and mean
// over 1200 layers of 800 to 800000 pixels: more than 64 output channels, up to 256 input channels 1.0 / 1.55 (256 -> 1024
// 14x14 b = 256 77 / 46 us, BackwardData 90 / 50), up to 512 below 20000 pixels 0.98 / 1.6 (320 -> 192 3.0); from there on, with
// their narrower tiles, 1.07 / 1.2 above 192 output channels, 0.8 / 0.95 up to 128.  33 to 64 output channels 1.0 / 1.2, but
// 0.66 to 1.05 with no more than 32 input channels in BackwardData.
bool pointwise_bf16_pays(const Dims &d, int op, int b)
{
    if (d.dtype != 1 || d.R * d.S != 1 || d.sh != 1 || d.sw != 1 || d.ph != 0 || d.pw != 0) return false;
    const int K = op == 0 ? d.C : d.K, M = op == 0 ? d.K : d.C;
    const long cols = (long)b * d.H * d.W;
    if (d.H * d.W % 4 != 0 || K % 8 != 0 || (op == 1 && M % 2 != 0) || (long)d.H * d.W > 1l << 22) return false;
    if (M <= 32 || (M <= 64 && K <= 32)) return false;
    return K <= PointwiseHalfTile<2>::kMaxK || (K <= PointwiseHalfTile<1>::kMaxK && (cols < kWideCols || M > 192));
}

// pixel tiles that take all tile rows, and how many workgroups share each of the last round's
static unsigned pointwise_grid(PointwiseParams &p, int mt, int nt)
{
    const int tiles = (p.cols + nt - 1) / nt, slots = device_cus();
    p.m_tiles = (p.M + mt - 1) / mt;
    p.whole = tiles / slots * slots;
    const int over = tiles - p.whole;
    p.splits = over == 0 ? 1 : slots / over < 1 ? 1 : slots / over < p.m_tiles ? slots / over : p.m_tiles;
    return (unsigned)(p.whole + over * p.splits);
}

static std::string pointwise_text(const PointwiseParams &p, const char *name, const char *op, int mt, int nt)
{
    return std::string(name) + "<Tile<" + std::to_string(mt) + "x" + std::to_string(nt) + ">," + op + "> tiles=" +
           std::to_string((p.cols + nt - 1) / nt) + " splits=1 batch=1 M=" + std::to_string(p.M) + " N=" +
           std::to_string(p.cols) + " K=" + std::to_string(p.K);
}

static PointwiseParams pointwise_params(const Dims &d, int op, int b, const void *in, const void *w, void *out)
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
    return p;
}

hipError_t pointwise_conv(const Dims &d, int op, int b, const void *in, const void *w, void *out, hipStream_t s)
{
    PointwiseParams p = pointwise_params(d, op, b, in, w, out);
    typedef PointwiseTile T;
    const unsigned grid = pointwise_grid(p, T::MT, T::NT);
    if (LaunchLog *log = launch_log()) {
        log->add(pointwise_text(p, "gemm_kernel_split_pointwise", op == 0 ? "forward" : "backward data", T::MT, T::NT));
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

template <class T>
static hipError_t launch_bf16(PointwiseParams &p, int op, hipStream_t s)
{
    const unsigned grid = pointwise_grid(p, T::MT, T::NT);
    if (LaunchLog *log = launch_log()) {
        log->add(pointwise_text(p, "gemm_kernel_bf16_pointwise", op == 0 ? "forward" : "backward data", T::MT, T::NT));
        return hipSuccess;
    }
    if (op == 0) pointwise_bf16_kernel<T, true><<<grid, T::THREADS, 0, s>>>(p);
    else pointwise_bf16_kernel<T, false><<<grid, T::THREADS, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t pointwise_bf16(const Dims &d, int op, int b, const void *in, const void *w, void *out, hipStream_t s)
{
    PointwiseParams p = pointwise_params(d, op, b, in, w, out);
    if (p.K <= PointwiseHalfTile<2>::kMaxK && p.cols >= kWideCols) return launch_bf16<PointwiseHalfTile<2>>(p, op, s);
    return launch_bf16<PointwiseHalfTile<1>>(p, op, s);
}

}  // namespace ucd
