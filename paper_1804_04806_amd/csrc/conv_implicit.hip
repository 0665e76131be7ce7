// Zero-workspace implicit-GEMM convolution: Forward, BackwardData, BackwardFilter as tile GEMMs
// whose operand loaders gather straight from the NCHW tensors.
//   Forward        Y[K x bPQ]   = W[K x CRS]      * im2col(X)[CRS x bPQ]
//   BackwardData   dX[C x bHW]  = W^T[C x KRS]    * gather(dY)[KRS x bHW]   (one GEMM per stride phase)
//   BackwardFilter dW[K x CRS] += dY[K x bPQ]     * im2col(X)^T[bPQ x CRS]  (split over bPQ, fp32 atomics)
#include "implicit_common.hpp"

namespace ucd {

__global__ void fill_zero_kernel(float *p, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += step) p[i] = 0.f;
}

LaunchLog *&launch_log()
{
    static thread_local LaunchLog *log = nullptr;
    return log;
}

hipError_t fill_zero(float *p, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    if (LaunchLog *log = launch_log()) {
        log->add("fill_zero_kernel");
        return hipSuccess;
    }
    size_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    fill_zero_kernel<<<(unsigned)blocks, 256, 0, s>>>(p, n);
    return hipGetLastError();
}

static hipError_t implicit_fwd_bf16_vec(const Dims &d, int b, const void *x, const void *w, void *y, hipStream_t s)
{
    const int px = d.P * d.Q, px_pad = (px + 3) / 4 * 4;
    GemmShape g{d.K, b * px_pad, d.crs()};
    RunParams pb{};
    pb.t = x; pb.bytes = xbytes(d, b); pb.Ct = d.C; pb.Ht = d.H; pb.Wt = d.W;
    pb.plane_px = px; pb.grid_pad = FastDiv(px_pad); pb.grid_w = FastDiv(d.Q);
    pb.add_h = -d.ph; pb.add_w = -d.pw; pb.dir = 1;
    pb.taps = FastDiv(d.R * d.S); pb.taps_w = FastDiv(d.S);
    pb.n_tap_h = d.R; pb.n_tap_w = d.S;
    pb.shift_thread = d.ph * d.W + d.pw; pb.shift_row = 0;
    EpiNCHWParams pe{};
    pe.out = y; pe.grid_hw = pb.grid_pad; pe.grid_w = pb.grid_w;
    pe.M = d.K; pe.HWo = px; pe.Wo = d.Q; pe.h0 = 0; pe.hs = 1; pe.w0 = 0; pe.ws = 1; pe.cols = px;
    // 0: every element exists (no border masks); 1: masks, at most 16 taps; 2: masks, more taps
    const int mode = d.R * d.S == 1 && d.ph == 0 && d.pw == 0 ? 0 : d.R * d.S <= 16 ? 1 : 2;
    if (d.crs() % 8 == 0) {  // filter rows are whole 16-byte cells
        CellParams pa{w, wbytes(d), d.crs()};
        if (mode == 0) return launch_gemm<CellKLaneT, RunNLane, EpiNCHWT<bf16>, true>(pa, pb, pe, g, s);
        if (mode == 1) return launch_gemm<CellKLaneT, RunNLaneMasked, EpiNCHWT<bf16>, true>(pa, pb, pe, g, s);
        return launch_gemm<CellKLaneT, RunNLaneMaskedBig, EpiNCHWT<bf16>, true>(pa, pb, pe, g, s);
    }
    KLaneParams pa{};
    pa.t = w; pa.bytes = wbytes(d); pa.row_stride = 1; pa.col_stride = d.crs();
    if (mode == 0) return launch_gemm<Loaders<bf16>::KLane0, RunNLane, EpiNCHWT<bf16>, true>(pa, pb, pe, g, s);
    if (mode == 1) return launch_gemm<Loaders<bf16>::KLane0, RunNLaneMasked, EpiNCHWT<bf16>, true>(pa, pb, pe, g, s);
    return launch_gemm<Loaders<bf16>::KLane0, RunNLaneMaskedBig, EpiNCHWT<bf16>, true>(pa, pb, pe, g, s);
}

// Whether the split kernel is the faster one for an unsplit Forward GEMM.  With short reductions a tile's start and end
// outweigh its steps, and the split kernel's cost more.  The fp32 kernel decodes taps, so layers with several cross
// earlier than 1x1 ones; it also loses more to rows of 128 than to 64.  Its time / the split kernel's:
//   one round of workgroups (tiles of 64 rows): 1x1 128 rows 0.93, 256 0.97, 512 1.00; 3x3 144 0.94, 7x7 196 0.99
//   up to 64 output channels: 1x1 96 rows 0.93, 128 1.00 (b = 80, 24x74); 3x3 on 56x56 b = 32: 27 0.80, 72 0.93, 108 0.98,
//   144 1.05 (3 -> 64 on 224x224, b = 8: 35 us / 50 us); 7x7 147 0.97, 196 1.01
//   tiles of 96 rows: 3x3 27 0.80, 72 0.95, 90 0.98, 108 1.02; of 128 rows: 27 0.91 to 1.00, 36 1.03, 72 1.12
//   more than 64 output channels, 1x1: 64 rows 0.95 to 1.00, 80 1.00 to 1.05
static bool split_forward_pays(const GemmShape &g, int taps)
{
    const TilePick t = pick_tile(g.M, g.N, true, 1);
    if (t.bm != 96 && t.blocks(g.M, g.N, 1) <= device_cus()) return g.Kd >= (taps == 1 ? 384 : 200);
    if (g.M <= 64) return g.Kd >= (taps > 31 ? 196 : 128);
    if (taps == 1) return g.Kd >= 80;
    return g.Kd >= (pick_rows(g.M, true) == 96 ? 96 : 36);
}

template <class E>
static hipError_t implicit_fwd_t(const Dims &d, int b, const void *x, const void *w, void *y, hipStream_t s)
{
    typedef Loaders<E> L;
    constexpr bool F32 = std::is_same<E, float>::value;
    if constexpr (!F32) {
        if (vector_gather_applies(d, d.Q, d.W)) return implicit_fwd_bf16_vec(d, b, x, w, y, s);
    }
    GemmShape g{d.K, b * d.P * d.Q, d.crs()};
    g.splits = output_splits(g.M, g.N, g.Kd, F32 && !d.det);
    KLaneParams pa{};
    pa.t = w; pa.bytes = wbytes(d); pa.row_stride = 1; pa.col_stride = d.crs();
    GatherParams pb{};
    pb.t = x; pb.bytes = xbytes(d, b); pb.Ct = d.C; pb.Ht = d.H; pb.Wt = d.W;
    pb.grid_hw = FastDiv(d.P * d.Q); pb.grid_w = FastDiv(d.Q);
    pb.mul_h = d.sh; pb.add_h = -d.ph; pb.mul_w = d.sw; pb.add_w = -d.pw; pb.dir = 1;
    pb.taps = FastDiv(d.R * d.S); pb.taps_w = FastDiv(d.S);
    pb.n_tap_h = d.R; pb.n_tap_w = d.S;
    pb.shift_thread = d.ph * d.W + d.pw; pb.shift_row = 0;
    EpiNCHWParams pe{};
    pe.out = y; pe.grid_hw = pb.grid_hw; pe.grid_w = pb.grid_w;
    pe.M = d.K; pe.HWo = d.P * d.Q; pe.Wo = d.Q; pe.h0 = 0; pe.hs = 1; pe.w0 = 0; pe.ws = 1;
    if constexpr (F32) {
        if (g.splits > 1) {
            hipError_t e = fill_zero((float *)y, (size_t)b * d.K * d.P * d.Q, s);
            if (e != hipSuccess) return e;
            if (d.R * d.S <= 31) return launch_gemm<CellK32T, GatherCell, EpiNCHWAtomic, true>(pa, pb, pe, g, s);
            return launch_gemm<CellK32T, GatherCellBig, EpiNCHWAtomic, true>(pa, pb, pe, g, s);
        }
    }
    g.tail_split = !d.det;
    // without padding every tap of every output pixel lies inside x: the loader without border masks
    // (filters of more than one tap: 1x1 layers are bound by memory, not by the loader)
    const bool free = d.ph == 0 && d.pw == 0 && d.R * d.S > 1;
    if constexpr (F32) {
        if (split_forward_pays(g, d.R * d.S)) {
            if (free) return launch_gemm<CellK32T, GatherCellFree, EpiNCHW, true>(pa, pb, pe, g, s);
            if (d.R * d.S <= 31) return launch_gemm<CellK32T, GatherCell, EpiNCHW, true>(pa, pb, pe, g, s);
            return launch_gemm<CellK32T, GatherCellBig, EpiNCHW, true>(pa, pb, pe, g, s);
        }
    }
    if (free) return launch_gemm<L::template KLane0, L::template GatherNLaneFree, EpiNCHWT<E>, true>(pa, pb, pe, g, s);
    if (d.R * d.S <= 31) return launch_gemm<L::template KLane0, L::template GatherNLane, EpiNCHWT<E>, true>(pa, pb, pe, g, s);
    return launch_gemm<L::template KLane0, L::template GatherNLaneBig, EpiNCHWT<E>, true>(pa, pb, pe, g, s);
}

hipError_t implicit_fwd(const Dims &d, int b, const void *x, const void *w, void *y, hipStream_t s)
{
    if (small_pays(d, 0, b)) return small_conv(d, 0, b, x, w, y, 0.f, s);
    hipError_t e;
    if (rows_fwd(d, b, x, w, y, s, e)) return e;
    if (pointwise_stream_pays(d, 0, b)) return pointwise_stream(d, 0, b, x, w, y, s);
    if (pointwise_pays(d, 0, b)) return pointwise_conv(d, 0, b, x, w, y, s);
    if (pointwise_bf16_pays(d, 0, b)) return pointwise_bf16(d, 0, b, x, w, y, s);
    if (window_conv(d, 0, b, x, w, y, s, e)) return e;
    return d.dtype == 1 ? implicit_fwd_t<bf16>(d, b, x, w, y, s) : implicit_fwd_t<float>(d, b, x, w, y, s);
}

// ---- BackwardData on a mirrored filter copy ---------------------------------------------------------
// With stride 1, dx[n,c,h,w] = sum_{k,r,s} dy[n,k,h+pad-r,w+pad-s] w[k,c,r,s] is the Forward
// convolution of dy (K channels, P x Q) with wt[c][k][r'][s'] = w[k][c][R-1-r'][S-1-s'] and padding
// (R-1-pad, S-1-pad).  Once the filter is stored that way its rows are contiguous along the
// reduction index, which is what the Forward kernels' filter loaders want (no per-element decode
// in fp32; 16-byte cells for the bf16 vector-load kernel).  The copy costs K*C*R*S elements of
// workspace and one small kernel per run of micro-batches.
template <class E>
__global__ __launch_bounds__(256) void mirror_filter_kernel(const E *__restrict__ w, E *__restrict__ wt, int K, int C,
                                                            int RS)
{
    const long n = (long)K * C * RS;
    for (long i = blockIdx.x * 256l + threadIdx.x; i < n; i += 256l * gridDim.x) {
        const int t = (int)(i % RS);
        const long ck = i / RS;
        const int k = (int)(ck % K), c = (int)(ck / K);
        wt[i] = w[((long)k * C + c) * RS + (RS - 1 - t)];   // (R-1-r)*S + (S-1-s) = RS-1 - (r*S+s)
    }
}

bool implicit_mirror_applies(const Dims &d, int op)
{
    return op == 1 && d.sh == 1 && d.sw == 1 && d.ph <= d.R - 1 && d.pw <= d.S - 1;
}

size_t implicit_mirror_ws_bytes(const Dims &d) { return (d.esize() * d.K * d.crs() + 15) / 16 * 16; }

hipError_t implicit_bwd_data_mirror(const Dims &d, int b, const void *dy, const void *w, void *dx, void *ws,
                                    bool filter_ready, hipStream_t s)
{
    LaunchLog *log = launch_log();
    if (filter_ready) {
        // the copy is still in the workspace from the previous micro-batch
    } else if (log) {
        log->add("mirror_filter_kernel");
    } else {
        const long n = (long)d.K * d.crs();
        const unsigned blocks = (unsigned)((n + 255) / 256 < 2048 ? (n + 255) / 256 : 2048);
        if (d.dtype == 1)
            mirror_filter_kernel<uint16_t><<<blocks, 256, 0, s>>>((const uint16_t *)w, (uint16_t *)ws, d.K, d.C, d.R * d.S);
        else
            mirror_filter_kernel<float><<<blocks, 256, 0, s>>>((const float *)w, (float *)ws, d.K, d.C, d.R * d.S);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    Dims m = d;   // the mirrored layer: dy is its input, dx its output
    m.C = d.K; m.K = d.C;
    m.H = d.P; m.W = d.Q; m.P = d.H; m.Q = d.W;
    m.ph = d.R - 1 - d.ph; m.pw = d.S - 1 - d.pw;
    return implicit_fwd(m, b, dy, ws, dx, s);
}

}  // namespace ucd
