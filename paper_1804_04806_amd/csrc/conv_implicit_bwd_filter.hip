// Implicit-GEMM BackwardFilter: reduction over the output pixels, split over workgroups (see conv_implicit.hip for the scheme).
#include "implicit_common.hpp"

namespace ucd {

// Number of reduction splits so that tiles * splits covers the chip a few times over, with
// chunks of at least 256 reduction rows.
int filter_splits(int M, int N, int Kd, int batch)
{
    const TilePick shape = pick_tile(M, N, true, 1 << 20);  // the default shape
    const long tiles = shape.blocks(M, N, batch);
    long want = (1024 + tiles - 1) / tiles;
    long cap = Kd / 256;
    if (cap < 1) cap = 1;
    if (want > cap) want = cap;
    if (want < 1) want = 1;
    // three workgroups of the 96- and 128-row BackwardFilter kernels fit a CU, four of the others
    const long slots = shape.bm >= 96 ? slots_filter() : slots_output();
    if (tiles >= 4 * slots) return (int)want;  // many rounds anyway
    return best_fill(tiles, want, (want + 1) / 2, want * 2 < cap ? want * 2 : cap, slots);
}

// The same for the split kernel, whose 128-column workgroups fit a CU twice and whose 256-column ones once.
static int split_kernel_filter_splits(int M, int N, int Kd)
{
    const bool wide = wide_shape(M, N);
    const TilePick shape = pick_tile(M, N, true, 1 << 20);
    const long tiles = wide ? (long)((M + 127) / 128) * ((N + 255) / 256) : shape.blocks(M, N, 1);
    const long slots = (wide ? 1l : shape.bm * shape.bn <= 64 * 64 ? 3l : 2l) * device_cus();
    const long cap = Kd / 256 < 1 ? 1 : Kd / 256;
    long want = (slots + tiles - 1) / tiles;
    if (want > cap) want = cap;
    if (want < 1) want = 1;
    if (tiles >= 4 * slots) return (int)want;
    return best_fill(tiles, want, (want + 1) / 2, want * 2 < cap ? want * 2 : cap, slots);
}

// Reproducible BackwardFilter: at most this much workspace holds the reduction chunks' partial
// results (one K x CRS plane per chunk); a filter too large for several planes gets fewer, longer chunks.
constexpr size_t kDetPartialCap = (size_t)32 << 20;

static int det_filter_splits(const Dims &d, int b)
{
    const int Kd = b * d.P * d.Q;
    long want = filter_splits(d.K, d.crs(), Kd);
    const long cap = (long)(kDetPartialCap / ((size_t)4 * d.K * d.crs()));
    if (want > cap) want = cap;
    int chunk;
    return effective_splits(Kd, (int)(want < 1 ? 1 : want), chunk);
}

size_t implicit_det_ws_bytes(const Dims &d, int b)
{
    const int splits = det_filter_splits(d, b);
    return splits > 1 ? (size_t)4 * splits * d.K * d.crs() : 0;  // one chunk: a single addition per element
}

// dw = beta * dw + part[0] + part[1] + ... in that order
__global__ void reduce_partials_kernel(const float *part, int splits, size_t plane, float *dw, float beta, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += step) {
        float acc = beta == 0.f ? 0.f : dw[i];
        for (int sp = 0; sp < splits; ++sp) acc += part[(size_t)sp * plane + i];
        dw[i] = acc;
    }
}

// fp32 tensors: the split kernel, masks by padding and tap count (see QuadXT)
template <class Epi>
static hipError_t launch_filter_gemm(const Dims &d, const KLaneParams &pa, const KLaneParams &pb,
                                     const typename Epi::Params &pe, const GemmShape &g, hipStream_t s)
{
    const bool two = d.sw == 2;
    if (d.ph == 0 && d.pw == 0)
        return two ? launch_gemm<QuadDyFree, QuadXFree2, Epi, true>(pa, pb, pe, g, s)
                   : launch_gemm<QuadDyFree, QuadXFree, Epi, true>(pa, pb, pe, g, s);
    if (d.R * d.S <= 31)
        return two ? launch_gemm<QuadDy, QuadX2, Epi, true>(pa, pb, pe, g, s)
                   : launch_gemm<QuadDy, QuadX, Epi, true>(pa, pb, pe, g, s);
    return two ? launch_gemm<QuadDyFree, QuadXBig2, Epi, true>(pa, pb, pe, g, s)
               : launch_gemm<QuadDyFree, QuadXBig, Epi, true>(pa, pb, pe, g, s);
}

template <class E>
static hipError_t implicit_bwd_filter_t(const Dims &d, int b, const void *x, const void *dy, float *dw, float beta,
                                        float *ws, hipStream_t s)
{
    typedef Loaders<E> L;
    hipError_t e;
    GemmShape g{d.K, d.crs(), b * d.P * d.Q};
    g.splits = d.det ? det_filter_splits(d, b)
               : std::is_same<E, float>::value && g.M > 32 ? split_kernel_filter_splits(g.M, g.N, g.Kd)
                                               : filter_splits(g.M, g.N, g.Kd);
    const bool partials = d.det && g.splits > 1;
    if (!partials && beta == 0.f && (e = fill_zero(dw, (size_t)d.K * d.crs(), s)) != hipSuccess) return e;
    KLaneParams pa{};
    pa.t = dy; pa.bytes = ybytes(d, b);
    pa.grid_hw = FastDiv(d.P * d.Q); pa.grid_w = FastDiv(d.Q);
    pa.col_taps = FastDiv(1); pa.col_taps_w = FastDiv(1);
    pa.n_stride = d.K * d.P * d.Q; pa.Ht = d.P; pa.Wt = d.Q;
    pa.mul_h = 1; pa.add_h = 0; pa.mul_w = 1; pa.add_w = 0;
    KLaneParams pb{};
    pb.t = x; pb.bytes = xbytes(d, b);
    pb.grid_hw = pa.grid_hw; pb.grid_w = pa.grid_w;
    pb.col_taps = FastDiv(d.R * d.S); pb.col_taps_w = FastDiv(d.S);
    pb.n_stride = d.C * d.H * d.W; pb.Ht = d.H; pb.Wt = d.W;
    pb.mul_h = d.sh; pb.add_h = -d.ph; pb.mul_w = d.sw; pb.add_w = -d.pw;
    pb.shift = d.ph * d.W + d.pw;
    pb.n_tap_h = d.R; pb.n_tap_w = d.S;
    if (partials) {
        const size_t plane = (size_t)d.K * d.crs();
        EpiPartialParams pp{ws, d.crs(), (long)plane};
        if constexpr (std::is_same<E, float>::value)
            e = launch_filter_gemm<EpiPartial>(d, pa, pb, pp, g, s);
        else
            e = d.R * d.S <= 31 ? launch_gemm<L::template DyTab, L::template XTab, EpiPartial, true>(pa, pb, pp, g, s)
                                : launch_gemm<L::template DyKLane, L::template XKLane, EpiPartial, true>(pa, pb, pp, g, s);
        if (e != hipSuccess) return e;
        if (LaunchLog *log = launch_log()) {
            log->add("reduce_partials_kernel");
            return hipSuccess;
        }
        size_t blocks = (plane + 255) / 256;
        if (blocks > 4096) blocks = 4096;
        reduce_partials_kernel<<<(unsigned)blocks, 256, 0, s>>>(ws, g.splits, plane, dw, beta, plane);
        return hipGetLastError();
    }
    EpiDenseParams pe{dw, d.crs()};
    if constexpr (std::is_same<E, float>::value) {
        return launch_filter_gemm<EpiAtomic>(d, pa, pb, pe, g, s);
    } else {
        // filters of at most 31 taps: per-row state in an LDS table; without padding every tap of every pixel is inside x
        const bool tab = d.R * d.S <= 31, free = d.ph == 0 && d.pw == 0;
        if (tab) return launch_gemm<L::template DyTab, L::template XTab, EpiAtomic, true>(pa, pb, pe, g, s);
        if (free) return launch_gemm<L::template DyKLane, L::template XKLaneFree, EpiAtomic, true>(pa, pb, pe, g, s);
        return launch_gemm<L::template DyKLane, L::template XKLane, EpiAtomic, true>(pa, pb, pe, g, s);
    }
}

hipError_t implicit_bwd_filter(const Dims &d, int b, const void *x, const void *dy, float *dw, float beta,
                               float *ws, hipStream_t s)
{
    return d.dtype == 1 ? implicit_bwd_filter_t<bf16>(d, b, x, dy, dw, beta, ws, s)
                        : implicit_bwd_filter_t<float>(d, b, x, dy, dw, beta, ws, s);
}

}  // namespace ucd
