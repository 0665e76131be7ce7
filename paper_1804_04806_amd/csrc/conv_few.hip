// Launch of conv_few_kernel: BackwardData of layers with few input channels.
#include <algorithm>
#include <cmath>

#include "conv_few.hpp"
#include "gemm_launch.hpp"

namespace ucd {

// The grid of blocks of fh x fw strides, with as many pairs of taps in LDS at a time as leave room for a window; false where none fits.
static bool few_grid(const Dims &d, int b, int fh, int fw, FewParams &p)
{
    const int parts = d.dtype == 0 ? 3 : 1;
    p.fh = fh; p.fw = fw;
    p.vsh = fh * d.sh; p.vsw = fw * d.sw;
    p.U = (d.R + d.sh - 1) / d.sh + fh - 1; p.V = (d.S + d.sw - 1) / d.sw + fw - 1;
    p.taps = p.U * p.V;
    if (p.taps > kFewTaps) return false;
    const int pairs = (p.taps + 1) / 2, Wb = (d.W - 1 + d.pw) / p.vsw + 1, more = (p.V - 1) / fw;
    p.Hb = (d.H - 1 + d.ph) / p.vsh + 1;
    bool fits = false;
    for (int at_a_time : {12, 8, 5}) {
        p.groups = (pairs + at_a_time - 1) / at_a_time;
        p.pairs = (pairs + p.groups - 1) / p.groups;
        if (2 * p.pairs * p.groups > kFewTaps) continue;
        const int most = std::min(1536, (kFewLds - 2 * parts * p.pairs * 1024) / (2 * parts * 16));
        // As few blocks of columns as the window's size in LDS allows.  Narrower blocks hold as many rows or more: after one that does not
        // fit, the next to try is as wide as the window of its rows may be.
        for (int widest = 256; !fits && widest >= 4;) {
            p.nb = (Wb + widest - 1) / widest;
            p.Wc = (Wb + p.nb - 1) / p.nb;
            if (p.Wc < 4 && p.nb > 1) break;
            const int rows = (kFewN - 2) / p.Wc + 2, segments = (rows - 2) / p.Hb + 2, held = fh * rows + segments * (p.U - fh);
            p.span = p.Wc + more;
            p.pitch = fw * p.span;
            p.cells = held * p.pitch;
            fits = p.cells <= most;
            widest = std::min(p.Wc - 1, most / (held * fw) - more);
        }
        if (fits) break;
    }
    if (!fits) return false;
    p.images = b * p.nb;
    const long cols = (long)p.images * p.Hb * p.Wc;
    if (cols >= 1l << 30) return false;
    p.cols = (int)cols;
    return true;
}

// Time in us: whole rounds of workgroups, one per CU, of a start and, per chunk of eight channels, the pairs of taps multiplied, a step's filter
// cells and the window's cells.  Fitted to 813 launches (1 to 256 images of 7x7 to 227x227, 1 to 32 channels in, 16 to 512 out, filters of 3x3
// to 11x11, strides 1, 2 and 4), standard deviation 6 % fp32 and 5 % bf16; the block so chosen takes 1.01 times the best one's time in the mean.
// Of 3000 launches of the kernel as it is now the model is 1.05 (fp32) and 1.1 times the time, standard deviation 7 and 10 %.
static double few_us(const Dims &d, const FewParams &p, long cus)
{
    const long wgs = (p.cols + kFewN - 1) / kFewN, rounds = (wgs + cus - 1) / cus;
    const int chunks = (d.K + kFewC - 1) / kFewC;
    const bool f32 = d.dtype == 0;
    return (f32 ? 1.2 : 1.8) + rounds * ((f32 ? 6.3 : 5.3) + chunks * (p.groups * ((f32 ? 0.2 : 0.048) * p.pairs + 0.7) + (f32 ? 0.3 : 0.34) * p.cells / 512));
}

static double few_pick(const Dims &d, int b, FewParams &best)   // its time
{
    const bool f32 = d.dtype == 0;
    const int chunks = (d.K + kFewC - 1) / kFewC, cus = device_cus();
    double least = 1e30;
    for (int fh = std::min(4, 32 / (d.C * d.sh * d.sw)); fh >= 1; --fh)
        for (int fw = std::min(8, 32 / (d.C * d.sh * d.sw * fh)); fw >= 1; --fw) {
            // less than few_us can be: no position that only fills up, all taps in as few steps as there can be, and of windows of 255 / Wc rows
            // of positions and two images the smallest
            const int Hb = (d.H - 1 + d.ph) / (fh * d.sh) + 1, Wb = (d.W - 1 + d.pw) / (fw * d.sw) + 1;
            const int u = (d.R + d.sh - 1) / d.sh - 1, V = (d.S + d.sw - 1) / d.sw + fw - 1, taps = (u + fh) * V, more = (V - 1) / fw;
            const double cells = fw * (255. * fh + 2. * u * more + 2. * std::sqrt(510. * fh * more * u));
            if (cells > 1536. || taps > kFewTaps) continue;
            const double rounds = std::max(1., (double)b * Hb * Wb / (256. * cus));
            if (rounds * ((f32 ? 6.3 : 5.3) + chunks * ((f32 ? 0.1 : 0.024) * taps + 0.029 * taps + (f32 ? 0.3 : 0.34) / 512 * cells)) > least) continue;
            FewParams p{};
            if (!few_grid(d, b, fh, fw, p)) continue;
            const double us = few_us(d, p, cus);
            if (us <= least) { least = us; best = p; }
        }
    return least;
}

// Up to 16 input channels, filters whose every stride phase has a tap, where the model of the implicit GEMMs comes to 1.15 times this kernel's.
// fp32 layers of stride 1 whose launch has fewer than 128 workgroups split their reductions there (not in reproducible mode: where
// it was not taken for them 0.75 to 0.09); bf16 layers of up to nine taps and 47 output channels are bound by memory either way.  Of 1500 layers drawn
// at random that it takes (1 to 256 images of 7x7 to 227x600, 1 to 1024 channels out, filters of 2x2 to 11x11, strides 1 to 4) their time / this
// kernel's is 2.3 in the geometric mean, 0.90 at least, one below 0.97; of 1390 that the models leave to them it would be 0.8, 0.27 at least (few
// output channels, filters no larger than the stride: 6 -> 39 2x2/2 100x218 b = 60 30 us against 70).  3 -> 64 7x7/2 224x224 b = 128:
// 807 -> 413 us, bf16 482 -> 225; 3 -> 64 7x7 112x112 b = 64 1760 -> 508; 3 -> 64 11x11 64x64 b = 32 809 -> 428.
static bool few_pays(const Dims &d, int b, FewParams &p)
{
    if (d.C > 16 || d.R < d.sh || d.S < d.sw || d.R * d.S == 1 || (long)d.H * d.W > 1l << 22) return false;
    if (d.dtype == 1 && d.R * d.S <= 9 && d.K < 48) return false;
    if (!offsets_in_reach(d.K + 2 * kFewC, (long)d.esize() * d.crs())) return false;   // loads of the filter's channels past the last one
    if (1.15 * few_pick(d, b, p) > implicit_bwd_data_us(d, b)) return false;
    return d.dtype == 1 || d.det || d.sh * d.sw > 1 || p.cols > 127 * kFewN;
}

bool few_bwd_data(const Dims &d, int b, const void *dy, const void *w, void *dx, hipStream_t s, hipError_t &e)
{
    FewParams p{};
    if (!few_pays(d, b, p)) return false;
    p.K = d.K; p.P = d.P; p.Q = d.Q; p.C = d.C; p.H = d.H; p.W = d.W; p.R = d.R; p.S = d.S; p.CRS = d.crs();
    p.sh = d.sh; p.sw = d.sw; p.ph = d.ph; p.pw = d.pw;
    p.div_wc = FastDiv(p.Wc); p.div_hb = FastDiv(p.Hb); p.div_nb = FastDiv(p.nb); p.div_pitch = FastDiv(p.pitch); p.div_span = FastDiv(p.span);
    p.div_v = FastDiv(p.V); p.div_block = FastDiv(p.vsh * p.vsw); p.div_vsw = FastDiv(p.vsw);
    p.in = dy; p.in_bytes = ybytes(d, b);
    p.w = w; p.w_bytes = wbytes(d);
    p.out = dx; p.out_bytes = xbytes(d, b);
    const unsigned blocks = (unsigned)((p.cols + kFewN - 1) / kFewN);
    if (LaunchLog *log = launch_log()) {
        log->add("conv_few_kernel<Tile<32x256>,block " + std::to_string(p.vsh) + "x" + std::to_string(p.vsw) + "> tiles=" + std::to_string(blocks) +
                 " splits=1 batch=1 M=" + std::to_string(p.C * p.vsh * p.vsw) + " N=" + std::to_string(p.cols) + " K=" + std::to_string(p.K * p.taps));
        e = hipSuccess;
        return true;
    }
    if (d.dtype == 1) conv_few_kernel<bf16><<<blocks, 512, 0, s>>>(p);
    else conv_few_kernel<float><<<blocks, 512, 0, s>>>(p);
    e = hipGetLastError();
    return true;
}

}  // namespace ucd
