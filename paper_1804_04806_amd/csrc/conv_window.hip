// Launch of conv_window_kernel: Forward and BackwardData of 3x3 stride-1 layers with bf16 tensors.
#include <algorithm>
#include <cmath>

#include "conv_window.hpp"
#include "gemm_launch.hpp"

namespace ucd {

// The position grid under tile T; false where a tile's window does not fit.
template <class T>
static bool window_params(const Dims &d, int b, WindowParams &p)
{
    if (T::OP == 0) {
        p.Ci = d.C; p.Hi = d.H; p.Wi = d.W; p.Co = d.K; p.Ho = d.P; p.Wo = d.Q; p.ph = d.ph; p.pw = d.pw;
    } else {
        p.Ci = d.K; p.Hi = d.P; p.Wi = d.Q; p.Co = d.C; p.Ho = d.H; p.Wo = d.W; p.ph = 2 - d.ph; p.pw = 2 - d.pw;
    }
    if (p.ph < 0 || p.ph > 2 || p.pw < 0 || p.pw > 2 || p.Wi < 4) return false;
    if (!offsets_in_reach((p.Ci + kWinC - 1) / kWinC * kWinC - 8, 2l * p.Hi * p.Wi)) return false;   // loads of channels past the last one
    // As few blocks of columns as the window's size in LDS and its 512 runs of four pixels allow.  Narrower blocks hold as many rows or
    // more: after one that does not fit, the next to try is as wide as the window of its rows may be.
    for (int widest = 62;;) {
        p.nb = (p.Wo + widest - 1) / widest;
        p.Wc = (p.Wo + p.nb - 1) / p.nb;
        if (p.Wc < 4 && p.nb > 1) return false;
        p.runs = (p.Wc + 2 + 3) / 4;
        p.pitch = 4 * p.runs + 1;   // odd: the rows' runs begin on different banks
        const int rows = (T::NT - 2) / p.Wc + 2, more = (rows - 2) / p.Ho + 1;   // of positions, and how often an image ends in them
        p.rows = rows + more * (2 - p.ph) + 2;
        p.cells = p.rows * p.pitch;
        if (p.cells <= T::kMaxCells && 2 * p.rows * p.runs <= 512) break;
        widest = std::min(p.Wc - 1, 4 * std::min(256 / p.rows, (T::kMaxCells / p.rows - 1) / 4) - 2);
        if (widest < 4) return false;
    }
    p.images = b * p.nb;
    const long cols = (long)p.images * p.Ho * p.Wc;
    if (cols >= 1l << 30) return false;
    p.cols = (int)cols;
    p.tiles_m = (p.Co + T::MT - 1) / T::MT;
    p.div_wc = FastDiv(p.Wc); p.div_ho = FastDiv(p.Ho); p.div_nb = FastDiv(p.nb);
    p.div_runs = FastDiv(p.runs); p.div_rows = FastDiv(p.rows); p.div_step = FastDiv(p.Hi + p.ph);
    return true;
}

template <class T>
static hipError_t launch(const Dims &d, int b, const void *in, const void *w, void *out, hipStream_t s, WindowParams &p)
{
    p.in = in; p.in_bytes = T::OP == 0 ? xbytes(d, b) : ybytes(d, b);
    p.w = w; p.w_bytes = wbytes(d);
    p.out = out; p.out_bytes = T::OP == 0 ? ybytes(d, b) : xbytes(d, b);
    const unsigned blocks = (unsigned)(p.tiles_m * ((p.cols + T::NT - 1) / T::NT));
    if (LaunchLog *log = launch_log()) {
        log->add("conv_window_kernel<Tile<" + std::to_string(T::MT) + "x" + std::to_string(T::NT) + ">> tiles=" + std::to_string(blocks) +
                 " splits=1 batch=1 M=" + std::to_string(p.Co) + " N=" + std::to_string(p.cols) + " K=" + std::to_string(p.Ci * 9));
        return hipSuccess;
    }
    conv_window_kernel<T><<<blocks, 512, 0, s>>>(p);
    return hipGetLastError();
}

// A launch takes whole rounds of workgroups, one per CU, of 12 + 3.2 us a chunk (128 x 512), 5.4 + 2.1 (64 x 512), 4.1 + 1.57
// (64 x 256); of 32 x 256 two share a CU: 0.5 + 1.13 a round and one launch.  Fitted to 934 layers (1 to 256 images of 7x7 to 227x227, 8 to
// 1024 channels in and 16 to 1024 out, both operations): the tile so chosen takes 1.002 times the best of these four and of
// 128 x 256 and 128 x 128 in the mean, 1.18 at most.  Time of the kernels before / of this one 2.26 in the geometric mean of 634 of them,
// least 0.99 (384 -> 384 13x13 b = 256: Forward 216 -> 100 us, BackwardData 403 -> 104, on a mirrored filter 220 -> 107, as Winograd
// 183 and 180; 128 -> 128 28x28 b = 32: 28.9 -> 17.0 us, as Winograd 21.3).
struct WindowPick {
    int tile = -1;
    double us = 1e30;
    WindowParams p;
};

template <class T>
static void consider(const Dims &d, int b, int cus, int tile, double start, double chunk, WindowPick &best)
{
    WindowParams p{};
    if (!window_params<T>(d, b, p)) return;
    const double wgs = (double)p.tiles_m * ((p.cols + T::NT - 1) / T::NT);
    const double rounds = T::kPair ? 0.6 * std::ceil(wgs / cus) + 0.4 * std::max(1., wgs / cus) : std::ceil(wgs / cus);
    const double us = (T::kPair ? 3.5 : 0.) + rounds * (start + chunk * ((p.Ci + kWinC - 1) / kWinC));
    if (us < best.us) { best.us = us; best.tile = tile; best.p = p; }
}

// Wherever a tile's window fits: rows of four pixels and more (a run is loaded from inside its row), padding of up to two.  With an odd
// number of channels every other row of the filter begins in the middle of a word (BackwardData: every other channel of it), and the last
// word that holds elements ends behind the tensor, which the range check, by whole words, lets read as zero.
// Of few channels most of a chunk is zeros, and the element-wise GEMM, which stops at the last one, is as fast or faster (time of it / of
// this kernel): up to 8 channels in Forward 1.04 in the mean of 152 layers, 0.67 at least, where rows are not as long as the image's; where they
// are, the GEMM with vector loads 1.88 and 1.34 (172 layers); BackwardData of up to 4 channels 1.04 and 0.70 (278 layers), of 5 to 8 1.28 and
// 0.97 (87) up to 16 M pixels of dx, 0.88 at least beyond.  With 9 and 10 1.3 to 1.5, 0.99 at least.
template <int OP>
static bool window_conv_op(const Dims &d, int b, const void *in, const void *w, void *out, hipStream_t s, hipError_t &e)
{
    if (d.dtype != 1 || d.R != 3 || d.S != 3 || d.sh != 1 || d.sw != 1 || d.C % 2) return false;
    if (OP == 0 ? d.C <= 8 && d.Q != d.W : d.K <= 4 || (d.K <= 8 && (double)b * d.C * d.H * d.W >= 16e6)) return false;
    typedef WindowTile<OP, 4, 2, 8> T0;
    typedef WindowTile<OP, 2, 2, 8> T1;
    typedef WindowTile<OP, 2, 1, 8> T2;
    typedef WindowTile<OP, 1, 1, 8> T3;
    WindowPick best{};
    const int cus = device_cus();
    consider<T0>(d, b, cus, 0, 12., 3.2, best);
    consider<T1>(d, b, cus, 1, 5.4, 2.1, best);
    consider<T2>(d, b, cus, 2, 4.1, 1.57, best);
    consider<T3>(d, b, cus, 3, 0.5, 1.13, best);
    switch (best.tile) {
    case 0: e = launch<T0>(d, b, in, w, out, s, best.p); return true;
    case 1: e = launch<T1>(d, b, in, w, out, s, best.p); return true;
    case 2: e = launch<T2>(d, b, in, w, out, s, best.p); return true;
    case 3: e = launch<T3>(d, b, in, w, out, s, best.p); return true;
    }
    return false;
}

bool window_conv(const Dims &d, int op, int b, const void *in, const void *w, void *out, hipStream_t s, hipError_t &e)
{
    return op == 0 ? window_conv_op<0>(d, b, in, w, out, s, e) : window_conv_op<1>(d, b, in, w, out, s, e);
}

}  // namespace ucd
