// Implicit-GEMM BackwardData: one GEMM per stride phase, or all phases merged (see conv_implicit.hip for the scheme).
#include "implicit_common.hpp"

namespace ucd {

// Merged stride phases.  With few input channels a phase GEMM (M = C rows) leaves most of a
// 32-row tile empty.  Writing h + ph = vs*t + a with vs = f*stride, the pixels a = 0..vs-1 of
// block t are all reached from the same window of dy rows p = f*t + (f-1) - u, u = 0..U'-1,
// U' = ceil(R/stride) + f - 1, through filter row r = a - stride*(f-1) + stride*u (no such tap:
// zero).  One GEMM with M = C*vs_h*vs_w rows then computes all phases; R*S of every
// (stride*U')*(stride*V') taps it multiplies are real.  f = 1 or 2, whichever wastes least;
// 0 = keep the phases separate.
static int merged_phase_factor(const Dims &d)
{
    if (d.sh * d.sw == 1 || d.C >= 32) return 0;
    auto tile_eff = [](int M) {  // useful rows of the tiles x relative speed of the tile shape
        const int rows = pick_rows(M, true);
        const double speed = rows == 32 ? 0.7 : rows == 64 ? 0.9 : rows == 96 ? 0.96 : 1.0;
        return (double)M / ((M + rows - 1) / rows * rows) * speed;
    };
    int best = 0;
    double best_s = tile_eff(d.C);  // separate phases multiply no zero taps
    for (int f = 1; f <= 2; ++f) {
        const int M = d.C * f * d.sh * f * d.sw;
        const int U = (d.R + d.sh - 1) / d.sh + f - 1, V = (d.S + d.sw - 1) / d.sw + f - 1;
        if (M > 128 || U > 31 || V > 31) continue;
        const double s = tile_eff(M) * d.R / (double)(d.sh * U) * d.S / (double)(d.sw * V);
        if (s > best_s * 1.1) { best = f; best_s = s; }
    }
    return best;
}

template <class E>
static hipError_t implicit_bwd_data_merged(const Dims &d, int b, const void *dy, const void *w, void *dx, int f,
                                           hipStream_t s)
{
    typedef Loaders<E> L;
    const int vsh = f * d.sh, vsw = f * d.sw;
    const int U = (d.R + d.sh - 1) / d.sh + f - 1, V = (d.S + d.sw - 1) / d.sw + f - 1;
    const int Hb = (d.H - 1 + d.ph) / vsh + 1, Wb = (d.W - 1 + d.pw) / vsw + 1;  // blocks that hold a pixel
    GemmShape g{d.C * vsh * vsw, b * Hb * Wb, d.K * U * V};
    KLaneParams pa{};
    pa.t = w; pa.bytes = wbytes(d); pa.col_stride = d.R * d.S; pa.k_stride = d.crs(); pa.s_mem = d.S;
    pa.taps = FastDiv(U * V); pa.taps_w = FastDiv(V);
    pa.col_taps = FastDiv(vsh * vsw); pa.col_taps_w = FastDiv(vsw);
    pa.tap_mul_h = d.sh; pa.tap_add_h = -d.sh * (f - 1); pa.tap_mul_w = d.sw; pa.tap_add_w = -d.sw * (f - 1);
    pa.n_tap_h = d.R; pa.n_tap_w = d.S;
    GatherParams pb{};
    pb.t = dy; pb.bytes = ybytes(d, b); pb.Ct = d.K; pb.Ht = d.P; pb.Wt = d.Q;
    pb.grid_hw = FastDiv(Hb * Wb); pb.grid_w = FastDiv(Wb);
    pb.mul_h = f; pb.add_h = f - 1; pb.mul_w = f; pb.add_w = f - 1; pb.dir = -1;
    pb.taps = pa.taps; pb.taps_w = pa.taps_w;
    pb.n_tap_h = U; pb.n_tap_w = V;
    pb.shift_thread = 0; pb.shift_row = (U - 1) * d.Q + (V - 1);
    EpiPhasesParams pe{};
    pe.out = dx; pe.grid_hw = pb.grid_hw; pe.grid_w = pb.grid_w; pe.block = pa.col_taps; pe.block_w = pa.col_taps_w;
    pe.C = d.C; pe.H = d.H; pe.W = d.W; pe.vs_h = vsh; pe.vs_w = vsw; pe.pad_h = d.ph; pe.pad_w = d.pw;
    if (U * V <= 31)
        return launch_gemm<L::template PhaseFilterKLane, L::template GatherNLane, EpiPhasesT<E>, true>(pa, pb, pe, g, s);
    return launch_gemm<L::template PhaseFilterKLane, L::template GatherNLaneBig, EpiPhasesT<E>, true>(pa, pb, pe, g, s);
}

// One phase GEMM with the gather loader that fits its tap count.
template <template <int> class AL, template <int> class GatherSmall, template <int> class GatherBig, class Epi,
          bool ROWS96>
static hipError_t launch_phase(bool small, const KLaneParams &pa, const GatherParams &pb, const EpiNCHWParams &pe,
                               const GemmShape &g, hipStream_t s)
{
    return small ? launch_gemm<AL, GatherSmall, Epi, ROWS96>(pa, pb, pe, g, s)
                 : launch_gemm<AL, GatherBig, Epi, ROWS96>(pa, pb, pe, g, s);
}

// Stride-1 BackwardData with bf16 tensors and vector loads of dy (see vector_gather_applies): one
// GEMM dX[C x bHW] = W^T[C x KRS] * gather(dY), the gather running backwards through the taps.
static hipError_t implicit_bwd_data_bf16_vec(const Dims &d, int b, const void *dy, const void *w, void *dx,
                                             hipStream_t s)
{
    typedef Loaders<bf16> L;
    const int px = d.H * d.W, px_pad = (px + 3) / 4 * 4;
    GemmShape g{d.C, b * px_pad, d.K * d.R * d.S};
    KLaneParams pa{};
    pa.t = w; pa.bytes = wbytes(d); pa.col_stride = d.R * d.S;
    pa.taps = FastDiv(d.R * d.S); pa.taps_w = FastDiv(d.S);
    pa.k_stride = d.crs(); pa.s_mem = d.S;
    pa.tap_add_h = 0; pa.tap_mul_h = 1; pa.tap_add_w = 0; pa.tap_mul_w = 1;
    pa.unit_taps = 1;
    RunParams pb{};
    pb.t = dy; pb.bytes = ybytes(d, b); pb.Ct = d.K; pb.Ht = d.P; pb.Wt = d.Q;
    pb.plane_px = px; pb.grid_pad = FastDiv(px_pad); pb.grid_w = FastDiv(d.W);
    pb.add_h = d.ph; pb.add_w = d.pw; pb.dir = -1;
    pb.taps = pa.taps; pb.taps_w = pa.taps_w;
    pb.n_tap_h = d.R; pb.n_tap_w = d.S;
    pb.shift_thread = 0; pb.shift_row = (d.R - 1) * d.Q + (d.S - 1);
    EpiNCHWParams pe{};
    pe.out = dx; pe.grid_hw = pb.grid_pad; pe.grid_w = pb.grid_w;
    pe.M = d.C; pe.HWo = px; pe.Wo = d.W; pe.h0 = 0; pe.hs = 1; pe.w0 = 0; pe.ws = 1; pe.cols = px;
    const bool plain = d.R * d.S == 1 && d.ph == 0 && d.pw == 0;
    // filter operand: lanes along the input channels for filters of at most 9 taps (see below)
    if (pick_rows(d.C, true) != 96 && d.R * d.S <= 9)
        return plain ? launch_gemm<L::template FilterNLane, RunNLane, EpiNCHWT<bf16>, false>(pa, pb, pe, g, s)
                     : launch_gemm<L::template FilterNLane, RunNLaneMasked, EpiNCHWT<bf16>, false>(pa, pb, pe, g, s);
    return plain ? launch_gemm<L::template FilterKLane, RunNLane, EpiNCHWT<bf16>, true>(pa, pb, pe, g, s)
                 : launch_gemm<L::template FilterKLane, RunNLaneMaskedBig, EpiNCHWT<bf16>, true>(pa, pb, pe, g, s);
}

static void phase_shape(const Dims &d, int a, int c, int &h0, int &w0, int &Hh, int &Ww, int &Ra, int &Sc)
{
    h0 = ((a - d.ph) % d.sh + d.sh) % d.sh;
    w0 = ((c - d.pw) % d.sw + d.sw) % d.sw;
    Hh = h0 < d.H ? (d.H - h0 + d.sh - 1) / d.sh : 0;
    Ww = w0 < d.W ? (d.W - w0 + d.sw - 1) / d.sw : 0;
    Ra = a < d.R ? (d.R - a + d.sh - 1) / d.sh : 0;
    Sc = c < d.S ? (d.S - c + d.sw - 1) / d.sw : 0;
}

// Time in us of the launches below, as measured: a workgroup's reduction rows follow one another, and beyond one
// workgroup per CU the rows of all share its matrix pipes; both go with the size of the tile.  1700 strided layers (1 to 128
// images of 7x7 to 112x112, 17 to 1024 -> 32 to 2048 channels, 3 to 7 filter rows, 3 and 5 columns, row strides 1 to 4), both
// modes: model / measured within a fifth in four of five (least 0.5, most 2); 2000 layers of 1 to 16 -> 1 to 1024 channels 0.7 to 1.2 in four of five.
// bf16: 1020 layers of 1 to 16 channels, standard deviation 12 % (0.7 to 1.25).
double implicit_bwd_data_us(const Dims &d, int b)
{
    const bool bf = d.dtype == 1;
    const int cus = device_cus();
    auto launch_us = [&](int M, int N, int Kd, int splits) {
        const TilePick t = pick_tile(M, N, true, splits);
        const double size = t.bm * t.bn / 16384., more = (double)t.blocks(M, N, splits) / cus - 1;
        if (bf) return 1.9 + Kd * (0.022 + size * (0.03 + 0.043 * (more > 0 ? more : 0))) + 1.5e-6 * M * N;
        return 5.9 + Kd / splits * (0.012 + size * (0.088 + 0.12 * (more > 0 ? more : 0)));
    };
    if (const int f = merged_phase_factor(d)) {
        const int Hb = (d.H - 1 + d.ph) / (f * d.sh) + 1, Wb = (d.W - 1 + d.pw) / (f * d.sw) + 1;
        const int U = (d.R + d.sh - 1) / d.sh + f - 1, V = (d.S + d.sw - 1) / d.sw + f - 1;
        return (bf ? 2.8 : 0) + launch_us(d.C * f * d.sh * f * d.sw, b * Hb * Wb, d.K * U * V, 1);
    }
    double us = bf ? 2.8 : 0;
    bool any_split = false;
    for (int a = 0; a < d.sh; ++a)
        for (int c = 0; c < d.sw; ++c) {
            int h0, w0, Hh, Ww, Ra, Sc;
            phase_shape(d, a, c, h0, w0, Hh, Ww, Ra, Sc);
            if (Hh == 0 || Ww == 0 || Ra == 0 || Sc == 0) continue;
            const int splits = output_splits(d.C, b * Hh * Ww, d.K * Ra * Sc, !bf && !d.det);
            any_split = any_split || splits > 1;
            us += launch_us(d.C, b * Hh * Ww, d.K * Ra * Sc, splits);
        }
    return us + (any_split ? 3.5 : 0);
}

// Stride phases: input pixels h with (h + ph) % sh == a are reached only by filter rows
// r = a, a + sh, ...; within a phase the gather is a dense stride-1 correlation with the
// sub-sampled, index-reversed filter.  Pixels of a phase with no tap get zeros (Kd = 0).
template <class E>
static hipError_t implicit_bwd_data_t(const Dims &d, int b, const void *dy, const void *w, void *dx, hipStream_t s)
{
    typedef Loaders<E> L;
    constexpr bool F32 = std::is_same<E, float>::value;
    if constexpr (!F32) {
        // measured slower than the element-wise kernel (its filter operand cannot be fetched in cells
        // and, run four times per step, costs the kernel its second workgroup per CU): opt-in only
        static const bool on = [] { const char *e = std::getenv("UCD_BF16_VEC_BWD_DATA"); return e && e[0] == '1'; }();
        if (on && vector_gather_applies(d, d.W, d.Q)) return implicit_bwd_data_bf16_vec(d, b, dy, w, dx, s);
    }
    if (const int f = merged_phase_factor(d)) return implicit_bwd_data_merged<E>(d, b, dy, w, dx, f, s);
    // phases whose GEMM has too few tiles split their reduction (atomics); dx is zero-filled once
    // if any phase does
    bool any_split = false;
    for (int a = 0; a < d.sh; ++a)
        for (int c = 0; c < d.sw; ++c) {
            int h0, w0, Hh, Ww, Ra, Sc;
            phase_shape(d, a, c, h0, w0, Hh, Ww, Ra, Sc);
            if (Hh && Ww && Ra && Sc && output_splits(d.C, b * Hh * Ww, d.K * Ra * Sc, F32 && !d.det) > 1) any_split = true;
        }
    if (any_split) {
        hipError_t e = fill_zero((float *)dx, (size_t)b * d.C * d.H * d.W, s);
        if (e != hipSuccess) return e;
    }
    for (int a = 0; a < d.sh; ++a)
        for (int c = 0; c < d.sw; ++c) {
            int h0, w0, Hh, Ww, Ra, Sc;
            phase_shape(d, a, c, h0, w0, Hh, Ww, Ra, Sc);
            if (Hh == 0 || Ww == 0) continue;
            GemmShape g{d.C, b * Hh * Ww, d.K * Ra * Sc};
            if (any_split && g.Kd == 0) continue;  // dx is already zero there
            g.splits = output_splits(g.M, g.N, g.Kd, F32 && !d.det);
            const bool split = g.splits > 1;
            KLaneParams pa{};
            pa.t = w; pa.bytes = wbytes(d); pa.col_stride = d.R * d.S;
            pa.taps = FastDiv(Ra * Sc); pa.taps_w = FastDiv(Sc);
            pa.k_stride = d.crs(); pa.s_mem = d.S;
            pa.tap_add_h = a; pa.tap_mul_h = d.sh; pa.tap_add_w = c; pa.tap_mul_w = d.sw;
            pa.unit_taps = (d.sh == 1 && d.sw == 1) ? 1 : 0;
            GatherParams pb{};
            pb.t = dy; pb.bytes = ybytes(d, b); pb.Ct = d.K; pb.Ht = d.P; pb.Wt = d.Q;
            pb.grid_hw = FastDiv(Hh * Ww); pb.grid_w = FastDiv(Ww);
            pb.mul_h = 1; pb.add_h = (h0 + d.ph - a) / d.sh; pb.mul_w = 1; pb.add_w = (w0 + d.pw - c) / d.sw;
            pb.dir = -1;
            pb.taps = pa.taps; pb.taps_w = pa.taps_w;
            pb.n_tap_h = Ra; pb.n_tap_w = Sc;
            pb.shift_thread = 0; pb.shift_row = (Ra > 0 ? Ra - 1 : 0) * d.Q + (Sc > 0 ? Sc - 1 : 0);
            EpiNCHWParams pe{};
            pe.out = dx; pe.grid_hw = pb.grid_hw; pe.grid_w = pb.grid_w;
            pe.M = d.C; pe.HWo = d.H * d.W; pe.Wo = d.W; pe.h0 = h0; pe.hs = d.sh; pe.w0 = w0; pe.ws = d.sw;
            // With 2-byte elements the filter operand is read with lanes along the input channels
            // instead of the reduction rows (FilterNLaneT: fewer cache accesses per load; AlexNet
            // conv4 at b = 256: 0.56 -> 0.44 ms), where the tile is not the one that loader lacks (96
            // rows) and the filter has at most 9 taps: its lanes are R*S elements apart, and
            // on a 5x5 filter it is the slower one by far (conv2: 0.76 -> 1.46 ms).  In fp32, where
            // vector and scalar instruction issue is the limit and not the memory pipeline, it
            // measured 5-10 % slower even on 1x1 filters, whose channels are contiguous in memory.
            const bool nlane = !F32 && pick_rows(d.C, true) != 96 && d.R * d.S <= 9;
            const bool small = Ra * Sc <= 31;
            hipError_t e = hipSuccess;
            bool done = false;
            if constexpr (F32) {
                if (split) {
                    e = launch_phase<FilterKLane, GatherNLane, GatherNLaneBig, EpiNCHWAtomic, true>(small, pa, pb, pe, g, s);
                    done = true;
                }
            }
            g.tail_split = !d.det;
            if constexpr (!F32) {
                if (nlane) {
                    e = launch_phase<L::template FilterNLane, L::template GatherNLane, L::template GatherNLaneBig,
                                     EpiNCHWT<E>, false>(small, pa, pb, pe, g, s);
                    done = true;
                }
            }
            if (!done)
                e = launch_phase<L::template FilterKLane, L::template GatherNLane, L::template GatherNLaneBig,
                                 EpiNCHWT<E>, true>(small, pa, pb, pe, g, s);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

hipError_t implicit_bwd_data(const Dims &d, int b, const void *dy, const void *w, void *dx, hipStream_t s)
{
    if (small_pays(d, 1, b)) return small_conv(d, 1, b, dy, w, dx, 0.f, s);
    if (pointwise_stream_pays(d, 1, b)) return pointwise_stream(d, 1, b, dy, w, dx, s);
    if (pointwise_pays(d, 1, b)) return pointwise_conv(d, 1, b, dy, w, dx, s);
    if (pointwise_bf16_pays(d, 1, b)) return pointwise_bf16(d, 1, b, dy, w, dx, s);
    hipError_t e;
    if (window_conv(d, 1, b, dy, w, dx, s, e) || few_bwd_data(d, b, dy, w, dx, s, e)) return e;
    if (halo_pays(d, b)) return halo_bwd_data(d, b, dy, w, dx, s);
    return d.dtype == 1 ? implicit_bwd_data_t<bf16>(d, b, dy, w, dx, s) : implicit_bwd_data_t<float>(d, b, dy, w, dx, s);
}

}  // namespace ucd
