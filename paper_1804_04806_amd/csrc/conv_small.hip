// Small layers: which launches run on gemm_kernel_small, and their launch.
#include "gemm_small.hpp"
#include "gemm_launch.hpp"
#include "implicit_common.hpp"

namespace ucd {

// One stride phase of BackwardData (see implicit_bwd_data): first pixel, pixels and taps per axis.
struct PhaseExtent { int h0, w0, Hh, Ww, Ra, Sc; };
static PhaseExtent phase_extent(const Dims &d, int a, int c)
{
    PhaseExtent e;
    e.h0 = ((a - d.ph) % d.sh + d.sh) % d.sh;
    e.w0 = ((c - d.pw) % d.sw + d.sw) % d.sw;
    e.Hh = e.h0 < d.H ? (d.H - e.h0 + d.sh - 1) / d.sh : 0;
    e.Ww = e.w0 < d.W ? (d.W - e.w0 + d.sw - 1) / d.sw : 0;
    e.Ra = a < d.R ? (d.R - a + d.sh - 1) / d.sh : 0;
    e.Sc = c < d.S ? (d.S - c + d.sw - 1) / d.sw : 0;
    return e;
}

// Whether gemm_kernel_small is the faster one.  Its time is that of one workgroup times the rounds of workgroups, a
// workgroup's grows with the reduction; the tile kernels' hardly changes until they fill the chip.  Measured over 1500
// layers (1 to 16 images of 7x7 to 56x56, 3 to 1024 channels, 1x1 to 7x7, strides 1 and 2): time of the kernels otherwise
// taken / of this one, least and mean, by tiles of 16 x 16 and reduction rows:
//   fp32 Forward: up to 256 tiles, 2560 rows 1.28 / 2.3; up to 256, 2560 to 6000 rows 0.94 / 1.3; 256 to 512, 1024 to 2560
//   rows 0.75 / 1.2
//   fp32 BackwardData: up to 655360 rows of tiles 1.12 / 3.1 (strided layers up to 10: one launch for all phases);
//   512 to 1024 tiles of 1024 to 2560 rows 0.51 / 1.0
//   bf16 (an eighth of the matrix time) Forward and BackwardData: up to 512 tiles 1.08 / 3.0, 512 to 1024 tiles 0.80 / 2.3
//   BackwardFilter: fp32 up to 128 tiles, 524288 rows of tiles 1.22 / 2.0, 128 to 512 tiles up to 512 rows 1.49 / 2.1, 128 to
//   256 tiles of 512 to 2560 rows 0.86 / 1.5; bf16 up to 128 tiles, 2048 rows 1.18 / 1.8, 128 to 512 tiles up to 512 rows 1.39 / 1.9
// Layers of more than 32 output channels by themselves (900 more, fp32): Forward up to 64 tiles, 1024 to 2560 rows 1.08 / 2.0,
// otherwise 1.5 / 3.8 (one image, 128 -> 128 3x3 14x14, which the tile kernels split over a cleared output, 21.9 / 7.9 us);
// BackwardFilter 1.7 / 2.5.
bool small_pays(const Dims &d, int op, int b)
{
    const long M = op == 1 ? d.C : d.K;
    const long N = op == 0 ? (long)b * d.P * d.Q : op == 1 ? (long)b * d.H * d.W : d.crs();
    const long Kd = op == 0 ? d.crs() : op == 1 ? (long)d.K * ((d.R + d.sh - 1) / d.sh) * ((d.S + d.sw - 1) / d.sw)
                                                : (long)b * d.P * d.Q;
    const long tiles = ((M + 15) / 16) * ((N + 15) / 16);
    const bool f32 = d.dtype == 0;
    if (op == 2) {
        if (d.det) return false;   // its chunks keep their planes there
        if (tiles <= 128) return f32 ? tiles * Kd <= 524288 : Kd < 2048;
        return tiles <= 512 && Kd <= 512;
    }
    if (op == 0) {
        // bf16: filter rows are read eight elements at a time, and the tensor's last dword has to be whole
        if (!f32) return tiles <= 512 && Kd <= 9216 && Kd % 2 == 0;
        return tiles <= 256 && Kd <= 2560;
    }
    if (d.sh * d.sw > kSmallPhases) return false;
    if (!f32) return tiles <= 512 && Kd <= 9216;
    return tiles <= 1024 && Kd <= 2560 && tiles * Kd <= 655360;
}

template <class E, int KIND>
static void launch(bool big, bool few, const SmallParams<kSmallBwdData> &all, dim3 grid, int threads, hipStream_t s)
{
    SmallParams<KIND> p;
    static_cast<SmallHead &>(p) = all;
    for (size_t i = 0; i < sizeof(p.ph) / sizeof(p.ph[0]); ++i) p.ph[i] = all.ph[i];
    if constexpr (std::is_same<E, float>::value) {
        if (few) {
            if (big) gemm_kernel_small<E, KIND, true, true><<<grid, threads, 0, s>>>(p);
            else gemm_kernel_small<E, KIND, false, true><<<grid, threads, 0, s>>>(p);
            return;
        }
    }
    if (big) gemm_kernel_small<E, KIND, true><<<grid, threads, 0, s>>>(p);
    else gemm_kernel_small<E, KIND, false><<<grid, threads, 0, s>>>(p);
}

hipError_t small_conv(const Dims &d, int op, int b, const void *a, const void *bsrc, void *out, float beta, hipStream_t s)
{
    SmallParams<kSmallBwdData> p{};
    p.out = out;
    p.RS = d.R * d.S; p.S = d.S; p.CRS = d.crs();
    p.hs = p.ws = 1;
    p.dir = 1;
    p.beta = beta;
    p.ph[0].taps = FastDiv(d.R * d.S); p.ph[0].taps_w = FastDiv(d.S);
    p.ph[0].mul_h = d.sh; p.ph[0].add_h = -d.ph; p.ph[0].mul_w = d.sw; p.ph[0].add_w = -d.pw;
    p.ph[0].grid_hw = FastDiv(d.P * d.Q); p.ph[0].grid_w = FastDiv(d.Q);
    int phases = 1;
    bool big = d.R * d.S > 31;
    if (op == 0) {          // (a, bsrc) = (x, w)
        p.a = bsrc; p.a_bytes = wbytes(d);
        p.b = a; p.b_bytes = xbytes(d, b);
        p.Ct = d.C; p.Ht = d.H; p.Wt = d.W;
        p.M = d.K; p.HWo = d.P * d.Q; p.Wo = d.Q;
        p.ph[0].N = b * d.P * d.Q; p.ph[0].Kd = d.crs();
    } else if (op == 1) {   // (dy, w)
        p.a = bsrc; p.a_bytes = wbytes(d);
        p.b = a; p.b_bytes = ybytes(d, b);
        p.Ct = d.K; p.Ht = d.P; p.Wt = d.Q;
        p.M = d.C; p.HWo = d.H * d.W; p.Wo = d.W;
        p.hs = d.sh; p.ws = d.sw; p.dir = -1;
        phases = 0;
        big = false;
        for (int i = 0; i < d.sh; ++i)
            for (int j = 0; j < d.sw; ++j) {
                const PhaseExtent e = phase_extent(d, i, j);
                if (e.Hh == 0 || e.Ww == 0) continue;
                SmallPhase &q = p.ph[phases++];
                q.grid_hw = FastDiv(e.Hh * e.Ww); q.grid_w = FastDiv(e.Ww);
                q.taps = FastDiv(e.Ra * e.Sc); q.taps_w = FastDiv(e.Sc);
                q.N = b * e.Hh * e.Ww; q.Kd = d.K * e.Ra * e.Sc;
                q.mul_h = q.mul_w = 1;
                q.add_h = (e.h0 + d.ph - i) / d.sh; q.add_w = (e.w0 + d.pw - j) / d.sw;
                q.tap_add_h = i; q.tap_add_w = j;
                q.h0 = e.h0; q.w0 = e.w0;
                big = big || e.Ra * e.Sc > 31;
            }
    } else {                // (x, dy)
        p.a = bsrc; p.a_bytes = ybytes(d, b);
        p.b = a; p.b_bytes = xbytes(d, b);
        p.Ct = d.C; p.Ht = d.H; p.Wt = d.W;
        p.M = d.K; p.HWo = d.P * d.Q; p.Wo = d.crs();
        p.a_n_stride = d.K * d.P * d.Q;
        p.ph[0].N = d.crs(); p.ph[0].Kd = b * d.P * d.Q;
        // (bf16: eight rows of a lane are two such runs)
        p.vec_a = d.P * d.Q % 4 == 0;
        p.vec_b = p.vec_a && d.R * d.S == 1 && d.ph == 0 && d.pw == 0 && d.sh == 1 && d.sw == 1;
    }
    p.tiles_m = (p.M + 15) / 16;
    int n = 0, kd = 0;
    double work = 0, cols = 0;
    for (int i = 0; i < phases; ++i) {
        n = p.ph[i].N > n ? p.ph[i].N : n;
        kd = p.ph[i].Kd > kd ? p.ph[i].Kd : kd;
        work += (double)p.ph[i].N * p.ph[i].Kd;
        cols += p.ph[i].N;
    }
    if (n == 0) return hipSuccess;
    const int step = d.dtype == 1 ? 32 : 16;
    int splits = 1;
    if (op == 2) {
        const int tiles = p.tiles_m * ((n + 15) / 16);
        // chunks of 256 rows meet through atomics in a cleared dw (2048 rows, 18 tiles: 6.8 us, with 512 rows a
        // chunk 8.1, 1024 11.7, one workgroup a tile 16.9)
        int want = kd / 256;
        if (want * tiles > 512) want = 512 / tiles;
        splits = effective_splits(kd, want, p.k_chunk, step);
        if (splits > 1 && beta == 0.f) {
            const hipError_t e = fill_zero((float *)out, (size_t)d.K * d.crs(), s);
            if (e != hipSuccess) return e;
        }
        kd = p.k_chunk < kd ? p.k_chunk : kd;
    }
    const int steps = (kd + step - 1) / step;
    const int waves = steps >= 64 ? 16 : steps >= 24 ? 8 : 4;
    // (up to twice as many rows where the tile kernels split their operands, whose products are exact)
    const bool few = kd <= (op == 2 && p.M > 32 ? 2 * kSmallFew : kSmallFew);
    const dim3 grid((unsigned)(p.tiles_m * ((n + 15) / 16)), (unsigned)phases, (unsigned)splits);
    if (LaunchLog *log = launch_log()) {
        static const char *const kind[3] = {"forward", "backward data", "backward filter"};
        log->add(std::string("gemm_kernel_small<Tile<16x16>,") + kind[op] + (d.dtype == 1 ? "/bf16" : "") + "> tiles=" +
                 std::to_string(grid.x * grid.y) + " splits=" + std::to_string(splits) + " batch=1 M=" + std::to_string(p.M) + " N=" +
                 std::to_string((long)cols) + " K=" + std::to_string((long)(work / cols + 0.5)));
        return hipSuccess;
    }
    if (d.dtype == 1) {
        if (op == 0) launch<bf16, kSmallFwd>(big, false, p, grid, 64 * waves, s);
        else if (op == 1) launch<bf16, kSmallBwdData>(big, false, p, grid, 64 * waves, s);
        else launch<bf16, kSmallBwdFilter>(big, false, p, grid, 64 * waves, s);
    } else {
        if (op == 0) launch<float, kSmallFwd>(big, few, p, grid, 64 * waves, s);
        else if (op == 1) launch<float, kSmallBwdData>(big, few, p, grid, 64 * waves, s);
        else launch<float, kSmallBwdFilter>(big, few, p, grid, 64 * waves, s);
    }
    return hipGetLastError();
}

}  // namespace ucd
