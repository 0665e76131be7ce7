// Launch of pointwise_kernel, pointwise_bf16_kernel and pointwise_stream_kernel: Forward and BackwardData of 1x1 stride-1 layers.
#include "conv_pointwise_bf16.hpp"
#include "conv_pointwise_stream.hpp"
#include "gemm_launch.hpp"
#include "implicit_common.hpp"

namespace ucd {

// Two rows of tiles, few input channels, and outputs of 200 MB and more, beyond the last-level cache: tile GEMMs / pointwise_kernel
// 0.84 to 0.98, pointwise_split_stream_kernel alike (48 -> 160 56x56 b = 128 113 / 128 us).
static bool thin_and_large(int K, int M, long cols) { return M > 128 && M <= 192 && K <= 48 && cols * M >= 50000000l; }

// Where it is the faster one: its input channels fit LDS and are enough that the products outweigh the stores, and its
// pixels give most CUs a workgroup.  Time of the tile GEMMs / of this kernel over 430 layers, least and mean, more than 128
// output channels: 17 to 160 input channels and 4000 pixels or more 0.96 / 1.24 (128 -> 512 28x28 b = 128 131 / 94 us, 160 ->
// 1024 up to 1.77), 800 to 4000 pixels 0.87 to 1.6, 16 channels 0.82 / 1.0.  Up to 128 output channels the input is used once:
// 8000 to 20000 pixels, a single round, 1.04 / 1.36, more 0.83 to 1.28.
bool pointwise_pays(const Dims &d, int op, int b)
{
    if (d.dtype != 0 || d.R * d.S != 1 || d.sh != 1 || d.sw != 1 || d.ph != 0 || d.pw != 0) return false;
    const int K = op == 0 ? d.C : d.K, M = op == 0 ? d.K : d.C;
    const long cols = (long)b * d.H * d.W;
    if (K <= 16 || K > PointwiseTile::kMaxK || (long)d.H * d.W > 1l << 22) return false;   // (rows of a tile below 2^31 bytes apart)
    if (thin_and_large(K, M, cols)) return false;
    return M > 128 ? cols >= 4000 : M > 64 && cols >= 8000 && cols <= 20000;
}

// fp32 layers that pointwise_kernel does not take: input channels beyond LDS, or one tile of output channels and many pixels.
// Tile GEMMs / pointwise_split_stream_kernel over 900 layers of 3000 to 100000 pixels: with 128 workgroups and more, half the chip,
// Forward 1.1 to 1.6 above 96 output channels (fewer workgroups 0.55 to 1.0, up to 64 channels 0.6 to 1.2); not beyond 256
// input channels, where tile GEMMs that split their last tiles' sums are more exact by up to 6 % (352 -> 256 14x14 b = 256).
// BackwardData, whose tile GEMMs run on the fp32 pipe, 1.04 to 2.0 from 96 workgroups and 65 output channels on (512 -> 128
// 28x28 b = 128 142 / 94 us; 97 beyond 1024 input channels, 0.93 below; 128 workgroups beyond 2048, 0.90 with 98).  32 input channels and fewer 0.75 to 1.3.
// BackwardData of up to 96 output channels from more than 256, the second round of workgroups less than a quarter full: 0.91 to
// 0.99 (otherwise 1.0 to 1.6).  Both lines only where the tile GEMMs may split their last tiles' sums: in reproducible mode 1.03 to
// 1.8 on the layers beyond them (752 -> 2328 28x28 b = 5: 267 / 150 us).
bool pointwise_stream_pays(const Dims &d, int op, int b)
{
    if (d.dtype != 0 || d.R * d.S != 1 || d.sh != 1 || d.sw != 1 || d.ph != 0 || d.pw != 0 || d.H * d.W % 2 != 0) return false;
    const int K = op == 0 ? d.C : d.K, M = op == 0 ? d.K : d.C;
    const long cols = (long)b * d.H * d.W;
    if ((long)d.H * d.W > 1l << 22) return false;
    if (K <= 32 || pointwise_pays(d, op, b) || thin_and_large(K, M, cols)) return false;
    const long groups = (cols + 255) / 256 * ((M + 127) / 128);
    const long cus = device_cus();
    if (op == 0) return M > 96 && K <= 256 && groups >= 128;
    if (!d.det && M <= 96 && K > 256 && groups > cus && 4 * groups < 5 * cus) return false;
    return M > (K <= 1024 ? 64 : 96) && groups >= (K <= 2048 || d.det ? 96 : 128);
}

// bf16 layers.  Times of the tile GEMMs / of these kernels over 2600 layers of 800 to 800000 pixels; "narrow" and "wide" are
// pointwise_bf16_kernel with 128 and 256 pixels, up to 512 and 256 input channels, "stream" is pointwise_stream_kernel.
enum class Bf16Route { kTiles, kNarrow, kWide, kStream };
constexpr long kWideCols = 20000;   // below, tiles of 256 pixels leave most CUs idle: narrow / wide 1.3, above 0.75 to 1.05
constexpr int kStreamGroups = 128;  // half the chip

static long stream_groups(int M, long cols) { return (cols + 255) / 256 * ((M + 127) / 128); }

// Up to 64 output channels half or more of a streaming workgroup's rows are padding: a round of workgroups (one per CU) costs
// it what the tile GEMMs take for about 0.7 to 1 rounds of pixels, so that both its number of rounds and how full the last one
// is decide.  Tile GEMMs / stream over 2100 layers of 16000 to 800000 pixels, least and mean:
//   Forward, up to 32 channels from up to 32 0.97 / 1.14, up to 64 from up to 128 0.97 / 1.22 in any number of rounds
//   others: one round 1.0 / 1.25 (up to 32 from up to 256, up to 64 from up to 512), two rounds, the second more than half full (from
//   up to 128 a third) 0.97 / 1.05, otherwise 0.66 / 0.87 (256 -> 32 28x28 b = 84: 11.2 / 16.1 us)
//   BackwardData: up to two rounds 0.95 / 1.2; more, up to 32 channels 0.73 / 0.88, up to 64 from up to 320 0.84 / 0.96, from
//   more 0.94 / 1.05
static bool stream_few_rows_pays(int op, int M, int K, long cols)
{
    const double rounds = (double)((cols + 255) / 256) / device_cus();
    if (op == 1) return rounds <= 2 ? K > 128 || rounds <= 1 || rounds > 1.5 || M > 32 : M > 32 && K > 320;
    if (K <= (M <= 32 ? 32 : 128)) return true;
    if (K > (M <= 32 ? 256 : 512)) return false;
    return rounds <= 1 || (rounds <= 2 && rounds > (K <= 128 ? 1.3 : 1.5));
}

static Bf16Route bf16_route(const Dims &d, int op, int b)
{
    if (d.dtype != 1 || d.R * d.S != 1 || d.sh != 1 || d.sw != 1 || d.ph != 0 || d.pw != 0) return Bf16Route::kTiles;
    const int K = op == 0 ? d.C : d.K, M = op == 0 ? d.K : d.C;
    const long cols = (long)b * d.H * d.W;
    if (d.H * d.W % 4 != 0 || K % 8 != 0 || (op == 1 && M % 2 != 0) || (long)d.H * d.W > 1l << 22) return Bf16Route::kTiles;
    const bool many = cols >= kWideCols;
    // up to 32 output channels most of a tile is empty: stream 0.7 to 0.9 against the Forward tile GEMMs above 256 input
    // channels, 1.05 to 1.5 up to there; BackwardData 0.8 to 1.1 up to 64 input channels, 1.05 to 1.7 above
    if (M <= 16) return Bf16Route::kTiles;
    if (M <= 32) {
        const bool pays = op == 0 ? many : (many && K > 64) || (K > 256 && cols >= 3000);
        return pays && stream_few_rows_pays(op, M, K, cols) ? Bf16Route::kStream : Bf16Route::kTiles;
    }
    if (M <= 64 && many && !stream_few_rows_pays(op, M, K, cols)) return Bf16Route::kTiles;
    if (op == 1 && M <= 64 && K <= (many ? 16 : 32)) return Bf16Route::kTiles;   // 0.85 to 1.2
    // beyond LDS: 128 -> 64 us for 2048 -> 256 28x28 b = 64 in BackwardData, whose tile GEMMs gather the filter; Forward 0.75 to
    // 0.95 with less than half a chip of workgroups or up to 96 output channels, otherwise 1.02 to 1.7 (1024 -> 256 14x14
    // b = 256 57 / 34 us)
    if (K > PointwiseHalfTile<1>::kMaxK)
        return (op == 1 ? cols >= 3000 : M > 96 && stream_groups(M, cols) >= kStreamGroups) ? Bf16Route::kStream : Bf16Route::kTiles;
    // narrow / stream 1.05 to 1.5 where stream has half a chip of workgroups, 0.6 to 0.95 below
    if (K > PointwiseHalfTile<2>::kMaxK)
        return many || stream_groups(M, cols) >= kStreamGroups ? Bf16Route::kStream : Bf16Route::kNarrow;
    // one tile of up to 256 output channels uses the input once either way: wide / stream 0.95 to 1.2; above 0.9 to 1.1
    if (!many) return Bf16Route::kNarrow;   // tile GEMMs / narrow 1.0 to 2.9 (256 -> 192 3.0)
    return M <= 256 ? Bf16Route::kStream : Bf16Route::kWide;   // tile GEMMs / wide 1.2 to 1.8 (256 -> 1024 14x14 b = 256 77 / 46)
}

bool pointwise_bf16_pays(const Dims &d, int op, int b) { return bf16_route(d, op, b) != Bf16Route::kTiles; }

// pixel tiles that take all tile rows, and how many workgroups share each of the last round's
static unsigned pointwise_grid(PointwiseParams &p, int mt, int nt)
{
    const int tiles = (p.cols + nt - 1) / nt, slots = device_cus();
    p.m_tiles = (p.M + mt - 1) / mt;
    p.whole = tiles / slots * slots;
    const int over = tiles - p.whole;
    p.splits = over == 0 ? 1 : slots / over < 1 ? 1 : slots / over < p.m_tiles ? slots / over : p.m_tiles;
    return (unsigned)(p.whole + over * p.splits);
}

static std::string pointwise_text(const PointwiseParams &p, const char *name, const char *op, int mt, int nt)
{
    return std::string(name) + "<Tile<" + std::to_string(mt) + "x" + std::to_string(nt) + ">," + op + "> tiles=" +
           std::to_string((p.cols + nt - 1) / nt) + " splits=1 batch=1 M=" + std::to_string(p.M) + " N=" +
           std::to_string(p.cols) + " K=" + std::to_string(p.K);
}

static PointwiseParams pointwise_params(const Dims &d, int op, int b, const void *in, const void *w, void *out)
{
    PointwiseParams p{};
    p.x = in; p.w = w; p.y = out;
    p.w_bytes = wbytes(d);
    p.x_bytes = op == 0 ? xbytes(d, b) : ybytes(d, b);
    p.y_bytes = op == 0 ? ybytes(d, b) : xbytes(d, b);
    p.K = op == 0 ? d.C : d.K;
    p.M = op == 0 ? d.K : d.C;
    p.px = d.H * d.W; p.cols = b * p.px;
    p.w_row = op == 0 ? d.C : 1;
    p.w_k = op == 0 ? 1 : d.C;
    p.div_px = FastDiv(p.px);
    return p;
}

hipError_t pointwise_conv(const Dims &d, int op, int b, const void *in, const void *w, void *out, hipStream_t s)
{
    PointwiseParams p = pointwise_params(d, op, b, in, w, out);
    typedef PointwiseTile T;
    const unsigned grid = pointwise_grid(p, T::MT, T::NT);
    if (LaunchLog *log = launch_log()) {
        log->add(pointwise_text(p, "pointwise_kernel", op == 0 ? "forward" : "backward data", T::MT, T::NT));
        return hipSuccess;
    }
    if (p.px % 4 == 0) {
        if (op == 0) pointwise_kernel<true, true><<<grid, T::THREADS, 0, s>>>(p);
        else pointwise_kernel<false, true><<<grid, T::THREADS, 0, s>>>(p);
    } else {
        if (op == 0) pointwise_kernel<true, false><<<grid, T::THREADS, 0, s>>>(p);
        else pointwise_kernel<false, false><<<grid, T::THREADS, 0, s>>>(p);
    }
    return hipGetLastError();
}

hipError_t pointwise_stream(const Dims &d, int op, int b, const void *in, const void *w, void *out, hipStream_t s)
{
    PointwiseParams p = pointwise_params(d, op, b, in, w, out);
    p.m_tiles = (p.M + 127) / 128;
    p.whole = (p.cols + 255) / 256;
    p.splits = 1;
    if (LaunchLog *log = launch_log()) {
        log->add(pointwise_text(p, "pointwise_split_stream_kernel", op == 0 ? "forward" : "backward data", 128, 256));
        return hipSuccess;
    }
    const unsigned grid = (unsigned)((p.whole + 7) / 8 * 8 * p.m_tiles);
    if (op == 0) pointwise_split_stream_kernel<true><<<grid, 768, 0, s>>>(p);
    else pointwise_split_stream_kernel<false><<<grid, 768, 0, s>>>(p);
    return hipGetLastError();
}

template <class T>
static hipError_t launch_bf16(PointwiseParams &p, int op, hipStream_t s)
{
    const unsigned grid = pointwise_grid(p, T::MT, T::NT);
    if (LaunchLog *log = launch_log()) {
        log->add(pointwise_text(p, "pointwise_bf16_kernel", op == 0 ? "forward" : "backward data", T::MT, T::NT));
        return hipSuccess;
    }
    if (op == 0) pointwise_bf16_kernel<T, true><<<grid, T::THREADS, 0, s>>>(p);
    else pointwise_bf16_kernel<T, false><<<grid, T::THREADS, 0, s>>>(p);
    return hipGetLastError();
}

template <int WM>
static hipError_t launch_stream(const PointwiseParams &a, int op, hipStream_t s)
{
    StreamParams p{};
    p.x = a.x; p.w = a.w; p.y = a.y;
    p.w_bytes = a.w_bytes; p.x_bytes = a.x_bytes; p.y_bytes = a.y_bytes;
    p.K = a.K; p.M = a.M; p.px = a.px; p.cols = a.cols;
    p.w_row = a.w_row; p.w_k = a.w_k; p.div_px = a.div_px;
    p.m_tiles = (p.M + 128 * WM - 1) / (128 * WM);
    p.tiles = (p.cols + 255) / 256;
    if (LaunchLog *log = launch_log()) {
        log->add(pointwise_text(a, "pointwise_stream_kernel", op == 0 ? "forward" : "backward data", 128 * WM, 256));
        return hipSuccess;
    }
    const unsigned grid = (unsigned)((p.tiles + 7) / 8 * 8 * p.m_tiles);
    if (op == 0) pointwise_stream_kernel<WM, true><<<grid, 768, 0, s>>>(p);
    else pointwise_stream_kernel<WM, false><<<grid, 768, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t pointwise_bf16(const Dims &d, int op, int b, const void *in, const void *w, void *out, hipStream_t s)
{
    PointwiseParams p = pointwise_params(d, op, b, in, w, out);
    switch (bf16_route(d, op, b)) {
    case Bf16Route::kNarrow: return launch_bf16<PointwiseHalfTile<1>>(p, op, s);
    case Bf16Route::kWide: return launch_bf16<PointwiseHalfTile<2>>(p, op, s);
    // tiles of 256 output channels once those of 128 take more than one round: in one round 128 / 256 take 0.87, in more 1.35
    default: return p.M > 128 && stream_groups(p.M, p.cols) > device_cus() ? launch_stream<2>(p, op, s) : launch_stream<1>(p, op, s);
    }
}

}  // namespace ucd
