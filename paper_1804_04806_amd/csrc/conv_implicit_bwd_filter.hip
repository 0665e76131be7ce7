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

// The same for gemm_kernel_bf16q: the count whose rounds of workgroups take least, a workgroup's start and end (pixel
// table, first loads, atomics) costing as much as kStart of its 64-row steps.  Filling the last round best, as above,
// took two short rounds for one long one (us, before / now: 128 -> 128 3x3 56x56 b = 16, 112 / 56 chunks, 76 / 53;
// 64 -> 64 3x3 32x32 b = 64, 38 / 28).
static int bf16q_filter_splits(int M, int N, int Kd)
{
    constexpr long kStart = 6;
    const TilePick shape = pick_tile(M, N, true, 1 << 20);
    const int bn = shape.bm == 32 || shape.bm == 96 ? 128 : shape.bn;  // those exist with 128 columns only
    const long tiles = (long)((M + shape.bm - 1) / shape.bm) * ((N + bn - 1) / bn);
    const long slots = (shape.bm * bn <= 64 * 64 ? 3l : 2l) * device_cus();
    // the atomics of a 128-row tile cost as much as eight steps (1x1 128 -> 256 56x56 b = 16: chunks of 256 rows 33 us,
    // of 512 rows 25), where that leaves a quarter of the CUs a workgroup (1x1 128 -> 128 14x14 b = 16: 10.0 us with 256
    // rows, 11.4 with 512)
    const int least = shape.bm == 128 && tiles * (Kd / 512) >= device_cus() / 4 ? 512 : 256;
    const long cap = Kd / least < 1 ? 1 : Kd / least;
    long best = 1, best_cost = 0;
    for (long c = 1; c <= cap && c <= 4 * slots / tiles + 1; ++c) {
        const long steps = (Kd + c * kQuadBK - 1) / (c * kQuadBK);
        const long cost = (tiles * c + slots - 1) / slots * (steps + kStart);
        if (c == 1 || cost < best_cost) { best = c; best_cost = cost; }
    }
    return (int)best;
}

// The same for the split kernel: two workgroups fit a CU, one of 256 columns, three of 64 x 64 tiles.
static int quad_filter_splits(int M, int N, int Kd)
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

// bf16 tensors: runs of four pixels (gemm_kernel_bf16q) or element by element (gemm_kernel_bf16).  The runs have to be
// whole in nearly every wave of 64 rows: images of a multiple of four pixels (13x13, 384 channels: 343 against 283 us;
// 14x14, 256 channels: 127 against 158), whose rows are one after the other in x as well or of a multiple of four pixels
// themselves.  Column stride 1, or 2 where its two loads still pay (4: 454 against 224 us, 11x11 first layer; 2 with
// border masks and few taps: 85 against 77, 64 -> 128 channels 56x56; 1x1 stride 2: 106 against 169).  Short reductions
// do not pay for the table of a 64-row step (196 rows: 11.7 against 10.9 us).  b = 256, 128 for the strided ones.
// Padded filters of more than 31 taps need two masks per pixel, whose table pays later still (us, runs / element by
// element, rows): 11x11 on 8x7 2408 18.6 / 16.2, 38528 66.5 / 90.5; 11x11 on 16x16 11008 83.9 / 79.5; 7x7/2 on 48x48
// 18432 17.3 / 14.5, on 96x96 73728 31.1 / 33.0; 7x7 on 24x24 4608 11.1 / 10.5, 73728 59.4 / 88.6.
// A tile of 96 or 128 rows that has at most 64 columns keeps the element-wise kernel up to 131072 rows (3 -> 256 3x3 32x32
// b = 64 26.3 / 22.7, 32 -> 256 1x1 56x56 b = 16 19.3 / 15.4; 3 -> 128 3x3 56x56 b = 64, 200704 rows 41 / 46).
static bool bf16_quads_pay(const Dims &d, int Kd)
{
    if (Kd < 2048 || d.P * d.Q % 4 != 0) return false;
    const bool masked = d.ph != 0 || d.pw != 0, even_rows = d.Q % 4 == 0;
    // tiles of 96 and more rows whose columns are mostly padding
    if (d.crs() <= 64 && (masked || Kd >= 32768) && Kd < 131072 &&
        pick_tile(d.K, d.crs(), true, bf16q_filter_splits(d.K, d.crs(), Kd)).bm >= 96)
        return false;
    if (masked && d.R * d.S > 31 && Kd < 32768) return false;
    if (d.sw == 1) return even_rows || (d.Q == d.W && d.sh == 1);
    return d.sw == 2 && even_rows && (!masked || d.R * d.S > 31);
}

// Reproducible BackwardFilter: at most this much workspace holds the reduction chunks' partial
// results (one K x CRS plane per chunk); a filter too large for several planes gets fewer, longer chunks.
constexpr size_t kDetPartialCap = (size_t)32 << 20;

// The planes that the launch writes, the sum reads and ucd_workspace_size prices.
static int det_filter_splits(const Dims &d, int b)
{
    const int Kd = b * d.P * d.Q;
    long want = filter_splits(d.K, d.crs(), Kd);
    const long cap = (long)(kDetPartialCap / ((size_t)4 * d.K * d.crs()));
    if (want > cap) want = cap;
    int chunk;
    const int step = d.dtype == 1 && bf16_quads_pay(d, Kd) ? kQuadBK : kBK;  // of the kernel that will run
    return effective_splits(Kd, (int)(want < 1 ? 1 : want), chunk, step);
}

size_t implicit_det_ws_bytes(const Dims &d, int b)
{
    const int splits = det_filter_splits(d, b);
    return splits > 1 ? (size_t)4 * splits * d.K * d.crs() : 0;  // one chunk: a single addition per element
}

// Whether the split kernel is the faster one for fp32 tensors.  Below 33 output channels it is not (see launch_gemm).
// Where its runs of four pixels break (rows of other than a multiple of four pixels under a column stride of 2, other
// strides, padding), or two masks per pixel are needed, it loads element by element or builds a dearer table, which
// pays from a number of multiplications on.  Time of the fp32 kernel / of this one by millions of multiplications:
// column stride 2, runs broken, up to 31 taps: 100 0.92 to 1.0, 200 to 400 0.92 to 0.99 (unpadded 0.94 to 1.02), 400 to 800
// 0.99 to 1.08; padded filters of more taps, broken 100 0.85, 800 0.90 to 1.02, 1100 0.82, 1260 1.06 to 1.12, more 1.14 to
// 1.25; not broken 100 to 180 0.91 to 0.95, 200 to 400 0.97 to 1.14, tiles of 96 rows 180 1.10.  Tiles of 96 rows, which the fp32 kernel cannot
// make smaller in small launches, 1.05 in all but padded filters of many taps.  All other layers 0.95 to 1.5.
static bool split_filter_pays(const Dims &d, int Kd)
{
    if (d.K <= 32) return false;
    // one tile of 96 or 128 rows, most of its columns padding, in about a round of workgroups: with fewer chunks the tiles
    // get smaller, with more the steps outweigh the start (us, fp32 / split: 3 -> 128 3x3, 50176 rows 22.0 / 22.1, 65536 29 /
    // 34, 100352 36 / 40)
    if (d.K > 64 && d.K <= 128 && d.crs() <= 32 && Kd >= 65536 && Kd < 131072) return false;
    const double mul = (double)d.K * d.crs() * Kd;
    const bool masked = d.ph != 0 || d.pw != 0, big = masked && d.R * d.S > 31;
    const bool whole = d.sw == 1 || (d.sw == 2 && d.Q % 4 == 0);
    const bool rows96 = pick_rows(d.K, true) == 96;
    if (big) return mul >= (!whole ? 1.2e9 : rows96 ? 1.5e8 : 2e8);
    if (whole || rows96) return true;
    if (!masked) return d.sw > 2 || mul >= 3e8;
    return mul >= 4e8;
}

// Operands in runs of four pixels, masks by padding and tap count (see QuadXT, QuadHalfX): fp32 tensors on the split
// kernel, bf16 tensors on theirs; or element by element.
template <class E, class Epi>
static hipError_t launch_filter_gemm(const Dims &d, const KLaneParams &pa, const KLaneParams &pb,
                                     const typename Epi::Params &pe, const GemmShape &g, hipStream_t s)
{
    const bool two = d.sw == 2, free = d.ph == 0 && d.pw == 0, few = d.R * d.S <= 31;
    typedef Loaders<E> L;
    constexpr bool F32 = std::is_same<E, float>::value;
    if (F32 ? !split_filter_pays(d, g.Kd) : !bf16_quads_pay(d, g.Kd)) {
        // fp32: without padding the loader without masks or table is the faster one for few taps too (us, table / this:
        // 64 -> 32 3x3 56x56 b = 64 98 / 87, 64 -> 24 3x3/2 28x28 16.2 / 14.5)
        if (few && !(F32 && free)) return launch_gemm<L::template DyTab, L::template XTab, Epi, true>(pa, pb, pe, g, s);
        if (free) return launch_gemm<L::template DyKLane, L::template XKLaneFree, Epi, true>(pa, pb, pe, g, s);
        return launch_gemm<L::template DyKLane, L::template XKLane, Epi, true>(pa, pb, pe, g, s);
    }
    if constexpr (F32) {
        if (free)
            return two ? launch_gemm<QuadDyFree, QuadXFree2, Epi, true>(pa, pb, pe, g, s)
                       : launch_gemm<QuadDyFree, QuadXFree, Epi, true>(pa, pb, pe, g, s);
        if (few)
            return two ? launch_gemm<QuadDy, QuadX2, Epi, true>(pa, pb, pe, g, s)
                       : launch_gemm<QuadDy, QuadX, Epi, true>(pa, pb, pe, g, s);
        return two ? launch_gemm<QuadDyFree, QuadXBig2, Epi, true>(pa, pb, pe, g, s)
                   : launch_gemm<QuadDyFree, QuadXBig, Epi, true>(pa, pb, pe, g, s);
    } else {
        if (free)
            return two ? launch_gemm<QuadHalfDy, QuadHalfXFree2, Epi, true>(pa, pb, pe, g, s)
                       : launch_gemm<QuadHalfDy, QuadHalfXFree, Epi, true>(pa, pb, pe, g, s);
        if (few) return launch_gemm<QuadHalfDy, QuadHalfXTab, Epi, true>(pa, pb, pe, g, s);
        return two ? launch_gemm<QuadHalfDy, QuadHalfXBig2, Epi, true>(pa, pb, pe, g, s)
                   : launch_gemm<QuadHalfDy, QuadHalfXBig, Epi, true>(pa, pb, pe, g, s);
    }
}

template <class E>
static hipError_t implicit_bwd_filter_t(const Dims &d, int b, const void *x, const void *dy, float *dw, float beta,
                                        float *ws, hipStream_t s)
{
    constexpr bool F32 = std::is_same<E, float>::value;
    hipError_t e;
    GemmShape g{d.K, d.crs(), b * d.P * d.Q};
    g.splits = d.det ? det_filter_splits(d, b)
               : F32 && split_filter_pays(d, g.Kd) ? quad_filter_splits(g.M, g.N, g.Kd)
               : !F32 && bf16_quads_pay(d, g.Kd) ? bf16q_filter_splits(g.M, g.N, g.Kd)
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
        e = launch_filter_gemm<E, EpiPartial>(d, pa, pb, pp, g, s);
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
    return launch_filter_gemm<E, EpiAtomic>(d, pa, pb, pe, g, s);
}

hipError_t implicit_bwd_filter(const Dims &d, int b, const void *x, const void *dy, float *dw, float beta,
                               float *ws, hipStream_t s)
{
    if (small_pays(d, 2, b)) return small_conv(d, 2, b, x, dy, dw, beta, s);
    hipError_t e;
    if (filter_window(d, b, x, dy, dw, beta, s, e) || filter_few(d, b, x, dy, dw, beta, s, e)) return e;
    return d.dtype == 1 ? implicit_bwd_filter_t<bf16>(d, b, x, dy, dw, beta, ws, s)
                        : implicit_bwd_filter_t<float>(d, b, x, dy, dw, beta, ws, s);
}

}  // namespace ucd
