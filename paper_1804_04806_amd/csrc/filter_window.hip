// Launch of filter_window_kernel: BackwardFilter of 3x3 stride-1 layers with bf16 tensors.
#include <algorithm>

#include "filter_window.hpp"
#include "gemm_launch.hpp"

namespace ucd {

typedef FilterWindowTile<4, 2, 2, 2> Tile4;

static void filter_window_params(const Dims &d, int b, FilterWindowParams &p)
{
    typedef Tile4 T;
    p.x_bytes = xbytes(d, b); p.dy_bytes = ybytes(d, b);
    p.b = b; p.C = d.C; p.H = d.H; p.W = d.W; p.K = d.K; p.P = d.P; p.Q = d.Q; p.ph = d.ph; p.pw = d.pw;
    const int strips = (d.Q + 7) / 8, chunks = (d.P + T::RB - 1) / T::RB;
    p.div_strips = FastDiv(strips); p.div_chunks = FastDiv(chunks);
    p.k_blocks = (d.K + T::KT - 1) / T::KT; p.c_blocks = (d.C + T::CT - 1) / T::CT;
    // Along the rows a line of many strips is used at once (8 strips and more: 1.09 to 1.15 times as fast in the mean, 1.5 at most); down the
    // rows of narrow images 0.94 to 1.0 times as fast, and 1.23 for 64 channels 56x56 b = 256, whose images all workgroups begin at
    // the same time a multiple of 4 KB apart.
    p.down = strips < 8;
    const long rows = (long)b * strips;
    p.units = (int)(p.down ? (rows + 1) / 2 * chunks : (rows * chunks + 1) / 2);   // fewer than the pixels of x
    // Workgroups per block of channels: up to a round of one per CU, whose steps of two units take 1.9 us while every workgroup's atomics add
    // 0.085 us to the launch (665 layers, standard deviation 16 %; the number so chosen takes 1.01 times the best of four in the mean).
    const long blocks = (long)p.k_blocks * p.c_blocks, cus = device_cus();
    double best = 1e30;
    for (int eighths = 2; eighths <= 8; ++eighths) {
        const long n = std::max(1l, cus * eighths / (8 * blocks));
        const int per = (int)((p.units + n * T::WR - 1) / (n * T::WR)) * T::WR;
        const long wgs = blocks * ((p.units + per - 1) / per);
        const double us = 1.9 * (double)((wgs + cus - 1) / cus) * (per / T::WR) + 0.085 * wgs;
        if (us < best) { best = us; p.per_wg = per; }
    }
}

// From 20 Gflop on where images are whole runs of four pixels (113 layers of 1 to 256 images of 7x7 to 227x227 and 9 to 1024 channels, time of
// gemm_kernel_bf16q / of this kernel 1.31 in the geometric mean, 1.00 at least; 16 Gflop 0.85, 12 0.78: the atomics outweigh
// the rest), from 8 where they are not (74 layers, gemm_kernel_bf16, 1.51 and 1.13; 6 Gflop 0.89).  Rows of four pixels and
// more, because they are loaded in fours from inside the row.  Where less than three fifths of the units' 4 x 8 pixels are dy's, gemm_kernel_bf16q
// loses nothing to padding: 13 layers 1.09, 0.82 at least; gemm_kernel_bf16 is the slower one there too (37 layers, 1.41 and 0.99).  Of 960 other
// layers that it takes 1.55, two below 0.92 (9 Gflop).
static bool filter_window_pays(const Dims &d, int b)
{
    if (d.dtype != 1 || d.det || d.R != 3 || d.S != 3 || d.sh != 1 || d.sw != 1 || d.W < 4 || d.Q < 4 || d.ph > 2 || d.pw > 2) return false;
    const double flops = 2. * d.K * d.crs() * ((double)b * d.P * d.Q), units = (d.P + 3) / 4 * 4. * ((d.Q + 7) / 8 * 8.);
    return d.P * d.Q % 4 == 0 ? flops >= 20e9 && d.P * d.Q >= 0.6 * units : flops >= 8e9;
}

bool filter_window(const Dims &d, int b, const void *x, const void *dy, float *dw, float beta, hipStream_t s, hipError_t &e)
{
    if (!filter_window_pays(d, b)) return false;
    FilterWindowParams p{};
    filter_window_params(d, b, p);
    p.x = x; p.dy = dy; p.dw = dw;
    if (beta == 0.f) {
        e = fill_zero(dw, (size_t)d.K * d.crs(), s);
        if (e != hipSuccess) return true;
    }
    const long blocks = (long)p.k_blocks * p.c_blocks, splits = (p.units + p.per_wg - 1) / p.per_wg;
    if (LaunchLog *log = launch_log()) {
        log->add("filter_window_kernel<Tile<" + std::to_string(Tile4::KT) + "x" + std::to_string(9 * Tile4::CT) + ">> tiles=" + std::to_string(blocks) +
                 " splits=" + std::to_string(splits) + " batch=1 M=" + std::to_string(d.K) + " N=" + std::to_string(d.crs()) +
                 " K=" + std::to_string(b * d.P * d.Q));
        e = hipSuccess;
        return true;
    }
    filter_window_kernel<Tile4><<<(unsigned)(blocks * splits), 512, 0, s>>>(p);
    e = hipGetLastError();
    return true;
}

}  // namespace ucd
