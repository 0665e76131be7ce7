// Launch of conv_few_kernel: BackwardData of layers with few input channels.
#include <algorithm>

#include "conv_few.hpp"
#include "gemm_launch.hpp"

namespace ucd {

// The grid of blocks of fh x fw strides with at most at_a_time pairs of taps in LDS; false where a tile's window does not fit.
static bool few_grid(const Dims &d, int b, int fh, int fw, int at_a_time, FewParams &p)
{
    const int parts = d.dtype == 0 ? 3 : 1;
    p.fh = fh; p.fw = fw;
    p.vsh = fh * d.sh; p.vsw = fw * d.sw;
    p.U = (d.R + d.sh - 1) / d.sh + fh - 1; p.V = (d.S + d.sw - 1) / d.sw + fw - 1;
    p.taps = p.U * p.V;
    if (p.taps > kFewTaps) return false;
    const int pairs = (p.taps + 1) / 2;
    p.groups = (pairs + at_a_time - 1) / at_a_time;
    p.pairs = (pairs + p.groups - 1) / p.groups;
    if (2 * p.pairs * p.groups > kFewTaps) return false;
    const int most = std::min(1536, (kFewLds - 2 * parts * p.pairs * 1024) / (2 * parts * 16));
    p.Hb = (d.H - 1 + d.ph) / p.vsh + 1;
    const int Wb = (d.W - 1 + d.pw) / p.vsw + 1;
    // as few blocks of columns as the window's size in LDS allows
    for (p.nb = (Wb + 255) / 256;; ++p.nb) {
        p.Wc = (Wb + p.nb - 1) / p.nb;
        if (p.Wc < 4 && p.nb > 1) return false;
        p.span = (fw * p.Wc + p.V - fw + fw - 1) / fw;
        p.pitch = fw * p.span;
        const int rows = (kFewN - 2) / p.Wc + 2, segments = (rows - 2) / p.Hb + 2;
        p.cells = (fh * rows + segments * (p.U - fh)) * p.pitch;
        if (p.cells <= most) break;
    }
    p.images = b * p.nb;
    const long cols = (long)p.images * p.Hb * p.Wc;
    if (cols >= 1l << 30) return false;
    p.cols = (int)cols;
    return true;
}

// Time in us: whole rounds of workgroups, one per CU, of a start and, per chunk of eight channels, the pairs of taps multiplied, a step's filter
// cells and the window's cells.  Fitted to 813 launches (1 to 256 images of 7x7 to 227x227, 1 to 32 channels in, 16 to 512 out, filters of 3x3
// to 11x11, strides 1, 2 and 4), standard deviation 6 % fp32 and 5 % bf16; the block so chosen takes 1.01 times the best one's time in the mean.
static double few_us(const Dims &d, const FewParams &p)
{
    const long wgs = (p.cols + kFewN - 1) / kFewN, rounds = (wgs + device_cus() - 1) / device_cus();
    const int chunks = (d.K + kFewC - 1) / kFewC;
    const bool f32 = d.dtype == 0;
    return (f32 ? 1.2 : 1.8) + rounds * ((f32 ? 6.3 : 5.3) + chunks * (p.groups * ((f32 ? 0.2 : 0.048) * p.pairs + 0.7) + (f32 ? 0.3 : 0.34) * p.cells / 512));
}

static bool few_pick(const Dims &d, int b, FewParams &best)
{
    double least = 1e30;
    for (int fh = 1; fh <= 4 && d.C * fh * d.sh * d.sw <= 32; ++fh)
        for (int fw = 1; fw <= 8 && d.C * fh * d.sh * fw * d.sw <= 32; ++fw)
            for (int at_a_time : {12, 8, 5}) {
                FewParams p{};
                if (!few_grid(d, b, fh, fw, at_a_time, p)) continue;
                const double us = few_us(d, p);
                if (us < least) { least = us; best = p; }
                break;
            }
    return least < 1e30;
}

// Up to 16 input channels, filters whose every stride phase has a tap.  fp32 layers of stride 1 whose launch has fewer than 128 workgroups split
// their reductions in the implicit GEMMs (not in reproducible mode); bf16 layers of up to nine taps and 47 output channels are
// bound by memory either way.  Of 372 other layers drawn as above the implicit GEMMs' time / this kernel's is 2.2 in the
// geometric mean, 0.91 at least, two below 0.97 (3 -> 64 7x7/2 224x224 b = 128: 818 -> 432 us, bf16 482 -> 280; 3 -> 64 7x7 112x112 b = 64 1759 -> 526;
// 3 -> 64 11x11 64x64 b = 32 810 -> 430); where it is not taken for its workgroups 0.75 to 0.09.
bool few_pays(const Dims &d, int b)
{
    if (d.C > 16 || d.R < d.sh || d.S < d.sw || d.R * d.S == 1 || (long)d.H * d.W > 1l << 22) return false;
    if (d.dtype == 1 && d.R * d.S <= 9 && d.K < 48) return false;
    if (!offsets_in_reach((d.K + kFewC - 1) / kFewC * kFewC, (long)d.esize() * d.P * d.Q)) return false;   // loads of channels past the last one
    FewParams p{};
    if (!few_pick(d, b, p)) return false;
    return d.dtype == 1 || d.det || d.sh * d.sw > 1 || p.cols > 127 * kFewN;
}

hipError_t few_bwd_data(const Dims &d, int b, const void *dy, const void *w, void *dx, hipStream_t s)
{
    FewParams p{};
    if (!few_pick(d, b, p)) return hipErrorInvalidValue;
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
        return hipSuccess;
    }
    if (d.dtype == 1) conv_few_kernel<bf16><<<blocks, 512, 0, s>>>(p);
    else conv_few_kernel<float><<<blocks, 512, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace ucd
