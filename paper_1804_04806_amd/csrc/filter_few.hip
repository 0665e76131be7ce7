// Launch of filter_few_kernel: BackwardFilter of layers with few input channels.
#include <algorithm>

#include "filter_few.hpp"
#include "gemm_launch.hpp"

namespace ucd {

// The grid of groups under tile T with blocks of gw groups of columns; false where a tile's window does not fit.
template <class T>
static bool few_groups(const Dims &d, int b, int gw, FilterFewParams &p)
{
    const int whole = d.S / d.sw, last = d.S % d.sw;   // runs of taps that begin on the same element, and the rest
    p.taps[0] = (whole + 1) / 2 * d.sw + (whole % 2 ? 0 : last);
    p.taps[1] = d.S - p.taps[0];
    p.CB = std::min(d.C, 32 * T::NE / (d.R * p.taps[0]));
    if (p.taps[1]) p.CB = std::min(p.CB, 32 * T::NO / (d.R * p.taps[1]));
    if (p.CB < 1 || d.R < d.sh) return false;
    p.c_blocks = (d.C + p.CB - 1) / p.CB;
    p.CB = (d.C + p.c_blocks - 1) / p.c_blocks;
    p.k_blocks = (d.K + T::MT - 1) / T::MT;
    const int across = (d.Q + 7) / 8;
    p.gw = gw;
    p.nb = (across + gw - 1) / gw;
    if (8l * gw * d.sw >= 1 << 15) return false;   // columns of a row in 16 bits
    p.half = (8 * gw + (d.S - 1) / d.sw + 2 + 1) / 2 | 1;   // an operand's fifth word too; odd: rows begin on different banks
    const int rows = (T::G - 2) / gw + 2, segments = (rows - 2) / d.P + 2;   // of groups, and virtual images they lie in
    p.rows = d.sh * rows + segments * (d.R - d.sh);
    p.pairs = p.CB * p.rows * d.sw * p.half;
    if (p.CB * p.rows > T::kRows || 2 * p.pairs > T::kMaxElements) return false;
    p.images = b * p.nb;
    const long groups = (long)p.images * d.P * gw;
    if (groups >= 1l << 30) return false;
    p.groups = (int)groups;
    p.tiles = (p.groups + T::G - 1) / T::G;
    return true;
}

// The blocks of columns with which the launch is shortest: a tile's time goes up with the pairs that it splits, and with narrow blocks, whose
// rows of dy are parts of a cache line (stem as above, one group 341 us, two 280, three 290, with 7 % of the groups padding).
template <class T>
static bool few_blocks(const Dims &d, int b, FilterFewParams &best)
{
    double least = 1e30;
    const int across = (d.Q + 7) / 8;
    // of blocks as wide as each other the fewest; none wider than a window of 2 R rows may be, whose phases have 4 gw pairs and more
    for (int gw = std::min(across, T::kMaxElements / (16 * d.R * d.sw)); gw >= 1;) {
        const int nb = (across + gw - 1) / gw;
        gw = (across + nb - 1) / nb;
        FilterFewParams p{};
        if (few_groups<T>(d, b, gw, p)) {
            const double cycles = (double)p.tiles * (2000. + 60. * ((p.pairs + 511) / 512) + 700. / gw);
            if (cycles < least) { least = cycles; best = p; }
        }
        --gw;
    }
    return least < 1e30;
}

template <class T>
static int splits_of(const FilterFewParams &p) { return std::max(1, std::min(p.tiles, device_cus() / (p.k_blocks * p.c_blocks))); }

template <class T>
static hipError_t launch(const Dims &d, int b, const void *x, const void *dy, float *dw, hipStream_t s, FilterFewParams &p)
{
    p.C = d.C; p.H = d.H; p.W = d.W; p.K = d.K; p.P = d.P; p.Q = d.Q; p.R = d.R; p.S = d.S; p.CRS = d.crs();
    p.sh = d.sh; p.sw = d.sw; p.ph = d.ph; p.pw = d.pw;
    p.div_gw = FastDiv(p.gw); p.div_p = FastDiv(d.P); p.div_nb = FastDiv(p.nb); p.div_len = FastDiv(d.sh * (d.P - 1) + d.R);
    p.div_rows = FastDiv(p.rows); p.div_half = FastDiv(p.half); p.div_sw = FastDiv(d.sw); p.div_r = FastDiv(d.R);
    p.div_taps[0] = FastDiv(p.taps[0]); p.div_taps[1] = FastDiv(std::max(1, p.taps[1]));
    p.x = x; p.x_bytes = xbytes(d, b);
    p.dy = dy; p.dy_bytes = ybytes(d, b);
    p.dw = dw;
    const long blocks = (long)p.k_blocks * p.c_blocks, splits = splits_of<T>(p);
    if (LaunchLog *log = launch_log()) {
        log->add("filter_few_kernel<Tile<" + std::to_string(T::MT) + "x" + std::to_string(32 * T::NJ) + ">> tiles=" + std::to_string(blocks) +
                 " splits=" + std::to_string(splits) + " batch=1 M=" + std::to_string(d.K) + " N=" + std::to_string(d.crs()) +
                 " K=" + std::to_string(b * d.P * d.Q));
        return hipSuccess;
    }
    filter_few_kernel<T><<<(unsigned)(blocks * splits), 512, 0, s>>>(p);
    return hipGetLastError();
}

typedef FilterFewTile<1, 3, 2> Narrow;
typedef FilterFewTile<2, 3, 2> Wide;

// Whether tile T has enough pixels per workgroup and few enough products that are padding.
template <class T>
static bool fills(const Dims &d, int b, int pixels, double share, FilterFewParams &p)
{
    // the least that few_blocks could come to, before it is asked
    if ((double)b * d.P * d.Q < (double)pixels * (device_cus() / (((d.K + T::MT - 1) / T::MT) * d.C))) return false;
    if (!few_blocks<T>(d, b, p) || (double)b * d.P * d.Q < (double)pixels * splits_of<T>(p)) return false;
    return (double)d.K * d.crs() >= share * ((double)p.k_blocks * T::MT) * (p.c_blocks * 32. * T::NJ);
}

// Launches are short of work below some thousand pixels per workgroup (its sums go through LDS and atomics at the end), and tiles of
// 64 rows split and multiply no faster than the implicit GEMMs do unless they are full; up to 32 output channels those run on the fp32 instructions.
// Of 260 layers (8 to 256 images of 20x20 to 227x227, 1 to 12 channels in, 16 to 64 out, filters of 3x3 to 11x11, strides 1, 2 and 4) their
// time / this kernel's is 1.79 in the geometric mean of 35 with up to 32 output channels, 1000 pixels and two fifths of the products
// real, 1.00 at least; 1.31 of 7 with more channels, 3200 pixels and four fifths real, 1.19 at least (2000 pixels 0.94, seven tenths 0.92).  Of 130
// other layers that it takes none is below 1.00.  (A strided window does not fit beside the 256 pixels of Narrow's tiles.)
bool filter_few(const Dims &d, int b, const void *x, const void *dy, float *dw, float beta, hipStream_t s, hipError_t &e)
{
    if (d.dtype != 0 || d.det || d.C > 16 || d.R * d.S == 1 || d.K > 64) return false;
    FilterFewParams p{};
    if (!(d.K <= 32 ? fills<Narrow>(d, b, 1000, 0.4, p) : fills<Wide>(d, b, 3200, 0.8, p))) return false;
    e = hipSuccess;
    if (beta == 0.f) e = fill_zero(dw, (size_t)d.K * d.crs(), s);
    if (e == hipSuccess) e = d.K <= 32 ? launch<Narrow>(d, b, x, dy, dw, s, p) : launch<Wide>(d, b, x, dy, dw, s, p);
    return true;
}

}  // namespace ucd
