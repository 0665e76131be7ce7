// Launch of conv_halo_kernel: BackwardData of fp32 layers.
#include <algorithm>
#include <cmath>

#include "conv_halo.hpp"
#include "gemm_launch.hpp"
#include "implicit_common.hpp"

namespace ucd {

// The position grid of BackwardData under tile T; false where the window of a tile does not fit.
template <class T>
static bool halo_params(const Dims &d, int b, HaloParams &p)
{
    p.K = d.K; p.P = d.P; p.Q = d.Q;
    p.C = d.C; p.H = d.H; p.W = d.W;
    p.R = d.R; p.RS = d.R * d.S; p.CRS = d.crs();
    p.sh = d.sh; p.ph = d.ph; p.dc = d.pw / T::NPH + T::kFirst;
    p.Gh = (d.H + d.sh - 1) / d.sh;
    const int Gw = (d.W + T::NPH - 1) / T::NPH;
    // as few blocks of columns as the window's size in LDS allows
    const int U = (d.R + d.sh - 1) / d.sh;
    for (int widest = 32;;) {
        p.nb = (Gw + widest - 1) / widest;
        p.Wc = (Gw + p.nb - 1) / p.nb;
        if (p.Wc < 4 && p.nb > 1) return false;
        p.pitch = p.Wc + T::kSpan;
        const int rows = (T::NT - 2) / p.Wc + 2, segments = (rows - 2) / p.Gh + 2;
        p.cells = (rows + segments * (U - 1)) * p.pitch;
        while (p.cells % 16 < 4 || p.cells % 16 > 12) ++p.cells;   // the halves on other banks
        if (p.cells <= T::kMaxCells) break;
        // narrower blocks hold as many rows or more: the next to try is as wide as the window of these rows may be
        widest = std::min(p.Wc - 1, T::kMaxCells / (rows + segments * (U - 1)) - T::kSpan);
        if (widest < 4) return false;
    }
    p.images = b * p.nb;
    const long cols = (long)p.images * p.Gh * p.Wc;
    if (cols >= 1l << 30) return false;
    p.cols = (int)cols;
    p.tiles_m = (d.C + T::MT - 1) / T::MT;
    p.div_wc = FastDiv(p.Wc); p.div_gh = FastDiv(p.Gh); p.div_nb = FastDiv(p.nb); p.div_pitch = FastDiv(p.pitch);
    return true;
}

template <class T>
static hipError_t launch(const Dims &d, int b, const void *dy, const void *w, void *dx, hipStream_t s)
{
    HaloParams p{};
    if (!halo_params<T>(d, b, p)) return hipErrorInvalidValue;
    p.in = dy; p.in_bytes = ybytes(d, b);
    p.w = w; p.w_bytes = wbytes(d);
    p.out = dx; p.out_bytes = xbytes(d, b);
    const int tiles_n = (p.cols + T::NT - 1) / T::NT;
    const dim3 grid((unsigned)(p.tiles_m * tiles_n), (unsigned)d.sh);
    if (LaunchLog *log = launch_log()) {
        log->add("conv_halo_kernel<Tile<" + std::to_string(T::MT) + "x" + std::to_string(T::NT) + ">,phases " +
                 std::to_string(d.sh * T::NPH) + "> tiles=" + std::to_string(grid.x * grid.y) + " splits=1 batch=1 M=" +
                 std::to_string(d.C) + " N=" + std::to_string(p.cols) + " K=" + std::to_string(d.K * d.R * d.S));
        return hipSuccess;
    }
    conv_halo_kernel<T><<<grid, T::THREADS, 0, s>>>(p);
    return hipGetLastError();
}

// two workgroups per CU where their LDS allows
template <int S, int PAR> using Strided = HaloTile<2, S, PAR, 1, 2, 2, S == 3 ? 2 : 4>;
template <int S> using Plain = HaloTile<1, S, 0, S == 3 ? 2 : 1, 2, 2, 4>;

template <class F>
static auto with_tile(const Dims &d, F f)
{
    if (d.sw == 1) return d.S == 3 ? f(Plain<3>{}) : f(Plain<5>{});
    if (d.pw % 2) return d.S == 3 ? f(Strided<3, 1>{}) : f(Strided<5, 1>{});
    return d.S == 3 ? f(Strided<3, 0>{}) : f(Strided<5, 0>{});
}
// Column stride 2: a workgroup walks over all channels of dy and all filter rows of its phase, which takes a launch that leaves
// CUs idle as long as a full one; the implicit GEMMs split their reductions there, but not in reproducible mode nor with merged
// phases.  Time in us as measured over the layers of implicit_bwd_data_us (model / measured 0.71 to 1.31, 0.82 to 1.17 in 98 of
// 100): two workgroups share a CU with 3 columns, one at a time has it with 5.  Where the two are within a tenth of each other
// this kernel, which adds no parts of a sum by atomics.
static bool strided_pays(const Dims &d, int b, long wgs)
{
    const int rows = (d.R + d.sh - 1) / d.sh;
    const double cus = (double)wgs / device_cus(), more = (d.S == 3 ? cus : std::ceil(cus)) - 1;
    const double here = d.S == 3 ? 8.2 + d.K * (0.067 * rows + 0.031) * (1 + 0.92 * (more > 0 ? more : 0))
                                 : 12.4 + d.K * (0.14 * rows + 0.032) * (1 + 1.04 * (more > 0 ? more : 0));
    return here <= 1.1 * implicit_bwd_data_us(d, b);
}

// Where it is the faster one.  Measured over 470 layers (1 to 128 images of 7x7 to 150x150, 16 to 512 channels, filters of
// 3x3 to 7x7), time of the implicit GEMMs otherwise taken / of this kernel, least and mean:
//   column stride 2: 3 columns 1.6 / 2.4, 5 columns 1.4 / 2.2 (128 -> 64 3x3/2 56x56 b = 128: 224 / 124 us, 256 -> 96 5x5/2
//   28x28 b = 64 237 / 71).  With 16 input channels three quarters of a tile's rows are padding, 0.96 and 0.8.  Over 1041 more
//   layers of 1 to 256 images, 17 to 1024 -> 16 to 2048 channels and strides of 1 to 4 rows, where strided_pays is true (815) 0.75 /
//   2.4, four below 0.9 (reproducible mode 934, 0.84 / 2.7); where it is false this kernel / the others 0.69 / 1.3 (eleven
//   below 0.9), 6.9 at most (31 -> 1574 3x3 13x19 stride (1, 2) b = 8: 374 / 54 us)
//   column stride 1, by filled part of the last round of workgroups times useful part of a tile's rows: from 0.5 on 1.29 /
//   1.6 (384 -> 384 3x3 13x13 b = 256: 923 / 512; as the Winograd kernel 410), 0.38 1.1 to 1.4, 0.25 0.65 to 1.2
// Filters of 7 columns: their operands and window do not fit LDS together often enough.
bool halo_pays(const Dims &d, int b)
{
    if (d.dtype != 0 || (d.S != 3 && d.S != 5) || d.sw > 2 || d.R < d.sh) return false;
    if (d.C <= 16 || (long)d.H * d.W > 1l << 22) return false;   // (rows of a tile below 2^31 bytes apart)
    if (!offsets_in_reach((d.K + kHaloC - 1) / kHaloC * kHaloC - 8, 4l * d.P * d.Q)) return false;   // loads of channels past the last one
    if (!offsets_in_reach(d.K + 2 * kHaloC, 4l * d.crs())) return false;                                                             // and of the filter's
    return with_tile(d, [&](auto t) {
        typedef decltype(t) T;
        HaloParams p{};
        if (!halo_params<T>(d, b, p)) return false;
        const long wgs = (long)p.tiles_m * ((p.cols + T::NT - 1) / T::NT) * d.sh;
        if (T::NPH == 2) return strided_pays(d, b, wgs);
        const long slots = (T::THREADS == 256 ? 2l : 1l) * device_cus();
        return 2.0 * wgs * d.C >= (double)((wgs + slots - 1) / slots * slots) * p.tiles_m * T::MT;
    });
}

hipError_t halo_bwd_data(const Dims &d, int b, const void *dy, const void *w, void *dx, hipStream_t s)
{
    return with_tile(d, [&](auto t) { return launch<decltype(t)>(d, b, dy, w, dx, s); });
}

}  // namespace ucd
