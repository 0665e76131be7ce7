// Launch of conv_rows_kernel: Forward of layers with few input channels.
#include <algorithm>

#include "conv_rows.hpp"
#include "gemm_launch.hpp"

namespace ucd {

// The position grid under tile T with nb blocks of columns; false where a tile's window does not fit.
template <class T>
static bool rows_blocks(const Dims &d, int b, int nb, RowsParams &p)
{
    p.delta = d.pw & 1;
    p.SQ = (d.S + p.delta + 3) / 4;
    const int per_channel = d.R * p.SQ;
    if ((long)d.C * per_channel > kRowsQuads) return false;
    p.nb = nb;
    p.Wc = (d.Q + p.nb - 1) / p.nb;
    if (p.nb > 1 && d.sw % 2) p.Wc += p.Wc & 1;   // blocks begin on even columns
    const long pitch = ((p.Wc - 1l) * d.sw + 4 * p.SQ + 1) / 2 * 2;
    if (pitch > 1024 * T::NB) return false;   // (as integers its window has no size any more)
    p.pitch = (int)pitch;
    const int rows = (T::NT - 2) / p.Wc + 2, segments = (rows - 2) / d.P + 2;   // of positions, and virtual images they lie in
    p.rows = d.sh * rows + segments * (d.R - d.sh);
    const int elements = d.C * p.rows * p.pitch;
    p.quads = d.C * per_channel;
    p.steps = (p.quads + 3) / 4;
    p.pairs = elements / 2;
    p.b_part = (2 * (elements + 4) + 15) / 16 * 16;   // an odd column's third word may lie behind the last row
    if (p.quads > kRowsQuads || d.C * p.rows > kRowsMost || p.pairs > 512 * T::NB || p.steps * T::A_STEP + T::PARTS * p.b_part > kRowsLds) return false;
    p.images = b * p.nb;
    const long cols = (long)p.images * d.P * p.Wc;
    if (cols >= 1l << 30) return false;
    p.cols = (int)cols;
    p.tiles_m = (d.K + T::MT - 1) / T::MT;
    p.tiles_n = (p.cols + T::NT - 1) / T::NT;
    return true;
}

// Cycles of a workgroup's tile: its barriers and sums, the pairs that a thread splits, the matrix instructions of the two waves of a SIMD.
template <class T>
static double tile_cycles(const RowsParams &p)
{
    return 4000 + 70. * ((p.pairs + 511) / 512) * 2 + p.steps * (T::F32 ? 192 : 32) * T::WM * 2;
}

// The blocks of columns with which that is least over the launch: narrow ones keep more of a window's rows, and of its columns fewer.  Of those
// as wide as each other the fewest; none wider than a tile, whose windows hold columns that it does not read, nor than a window of 2 R rows per
// channel may be.
template <class T>
static bool rows_grid(const Dims &d, int b, RowsParams &best)
{
    if (d.R < d.sh || !offsets_in_reach(T::MT, (long)d.esize() * d.P * d.Q)) return false;   // stores of rows past the last one
    const int room = 512 * T::NB / (d.C * d.R) - 4 * ((d.S + (d.pw & 1) + 3) / 4);
    if (room < 0) return false;
    double least = 1e30;
    for (int widest = std::min(std::max(T::NT, d.Q < 2 * T::NT ? d.Q : 0), room / d.sw + 1);;) {
        const int nb = (d.Q + widest - 1) / widest, Wc = (d.Q + nb - 1) / nb;
        if (nb > 1 && Wc < 8) break;
        RowsParams p{};
        if (rows_blocks<T>(d, b, nb, p)) {
            const double cycles = tile_cycles<T>(p) * p.cols;
            if (cycles < least) { least = cycles; best = p; }
        }
        widest = Wc - 1;
        if (widest < 1) break;
    }
    return least < 1e30;
}

static int per_row(const RowsParams &p) { return std::max(1, std::min(p.tiles_n, device_cus() / p.tiles_m)); }

template <class T>
static hipError_t launch(const Dims &d, int b, const void *x, const void *w, void *y, hipStream_t s, RowsParams &p)
{
    p.C = d.C; p.H = d.H; p.W = d.W; p.K = d.K; p.P = d.P; p.Q = d.Q; p.R = d.R; p.S = d.S; p.CRS = d.crs();
    p.sh = d.sh; p.sw = d.sw; p.ph = d.ph; p.pw = d.pw;
    p.div_wc = FastDiv(p.Wc); p.div_p = FastDiv(d.P); p.div_nb = FastDiv(p.nb); p.div_half = FastDiv(p.pitch / 2);
    p.div_rows = FastDiv(p.rows); p.div_sq = FastDiv(p.SQ); p.div_r = FastDiv(d.R);
    p.div_len = FastDiv(d.sh * (d.P - 1) + d.R);
    p.in = x; p.in_bytes = xbytes(d, b);
    p.w = w; p.w_bytes = wbytes(d);
    p.out = y; p.out_bytes = ybytes(d, b);
    const unsigned blocks = (unsigned)(per_row(p) * p.tiles_m);
    if (LaunchLog *log = launch_log()) {
        log->add("conv_rows_kernel<Tile<" + std::to_string(T::MT) + "x" + std::to_string(T::NT) + ">> tiles=" + std::to_string((long)p.tiles_m * p.tiles_n) +
                 " splits=1 batch=1 M=" + std::to_string(d.K) + " N=" + std::to_string(p.cols) + " K=" + std::to_string(d.crs()));
        return hipSuccess;
    }
    if (d.sw % 2) conv_rows_kernel<T, true><<<blocks, 512, 0, s>>>(p);
    else conv_rows_kernel<T, false><<<blocks, 512, 0, s>>>(p);
    return hipGetLastError();
}

// Rows of a tile / 32, 0 where none pays.  The filter is split by every workgroup and stays there, so launches of few tiles per workgroup lose
// what longer ones gain, and so do products of zeros: rows, taps and quads that only fill up a tile.  Of 260 layers (fp32 and bf16, 8 to
// 256 images of 7x7 to 227x227, 1 to 16 channels in, 16 to 512 out, filters of 3x3 to 11x11, strides 1, 2 and 4) the implicit GEMMs' time / this
// kernel's is 0.85 to 1.7 in fp32 from three tiles per workgroup on; with three quarters of the products real and sums of 60 products, 1.41 in the
// geometric mean of 37 and 1.17 at least, with fewer of either 0.96 and 0.87, below two tiles down to 0.54.  bf16 (a sixth of the
// multiplications for the same window): eight tiles and 100 products 1.29, 1.18 at least; six tiles 1.06; three 0.79; more than one row
// tile 0.87.  The tile GEMMs hold the 16 taps of 4x4 filters without a rest: under a column stride 1.04 and 0.77 (55 layers); and with many row
// tiles few workgroups share the columns: from six on, a last round of less than 0.85 of them 1.18 and 0.86 (55 layers).  Of 600 other layers
// that it takes 1.32 and 0.89, six below 0.97.
template <class E>
static int pick(const Dims &d, int b, RowsParams &p)
{
    if (d.C > 16 || d.crs() < (d.dtype == 1 ? 100 : 60)) return 0;
    const int wm = d.K <= 32 ? 1 : (d.K + 95) / 96 * 96 < (d.K + 63) / 64 * 64 ? 3 : 2;
    // blocks of eight columns and more fill up less than half of them: too few positions are, before the grid is worked out
    if (1.5 * b * d.P * d.Q < 256. * (d.dtype == 1 ? 8 : 3) * (device_cus() / ((d.K + 32 * wm - 1) / (32 * wm)) - 1)) return 0;
    if (!(wm == 1 ? rows_grid<RowsTile<E, 1>>(d, b, p) : wm == 2 ? rows_grid<RowsTile<E, 2>>(d, b, p) : rows_grid<RowsTile<E, 3>>(d, b, p))) return 0;
    if ((long)p.tiles_n < (d.dtype == 1 ? 8l : 3l) * per_row(p) || (d.dtype == 1 && p.tiles_m > 1)) return 0;
    if (d.dtype == 0 && d.R == 4 && d.S == 4 && d.sw > 1) return 0;
    const int per = per_row(p), rounds = (p.tiles_n + per - 1) / per;
    if (p.tiles_m > 5 && p.tiles_n < 0.85 * per * rounds) return 0;
    return 4.0 * d.crs() * d.K > 3.0 * (16.0 * p.steps) * (32.0 * wm * p.tiles_m) ? wm : 0;
}

template <class E>
static bool rows_fwd_t(const Dims &d, int b, const void *x, const void *w, void *y, hipStream_t s, hipError_t &e)
{
    RowsParams p{};
    switch (pick<E>(d, b, p)) {
    case 1: e = launch<RowsTile<E, 1>>(d, b, x, w, y, s, p); return true;
    case 2: e = launch<RowsTile<E, 2>>(d, b, x, w, y, s, p); return true;
    case 3: e = launch<RowsTile<E, 3>>(d, b, x, w, y, s, p); return true;
    }
    return false;
}

bool rows_fwd(const Dims &d, int b, const void *x, const void *w, void *y, hipStream_t s, hipError_t &e)
{
    return d.dtype == 1 ? rows_fwd_t<bf16>(d, b, x, w, y, s, e) : rows_fwd_t<float>(d, b, x, w, y, s, e);
}

}  // namespace ucd
