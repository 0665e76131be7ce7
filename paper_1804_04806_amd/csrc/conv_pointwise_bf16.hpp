// 1x1 stride-1 convolutions, bf16 tensors (gfx950): the structure of pointwise_kernel (see conv_pointwise.hpp) with operands as
// they are.  The products take a sixth of the fp32 layers' time, so that memory and the start and end of a tile set the pace of
// the tile GEMMs, which read the input once per 128 output channels, and of whose BackwardData the filter gathers; here the input
// is read once, and results of two adjacent pixels are exchanged between lanes and stored as one dword.  256 -> 1024 14x14
// b = 256: Forward 77 -> 46 us (129 MB at 2.8 TB/s, 26 GFLOP at 570 TF), BackwardData of 1024 -> 256 90 -> 50.
#pragma once
#include "conv_pointwise.hpp"

namespace ucd {

// Eight multiplying waves, 2 x 4, of 64 output channels x 32 WN pixels, and four producers; steps of 32 channels
template <int WN_>
struct PointwiseHalfTile {
    static constexpr int WM = 2, WN = WN_, MT = 128, NT = 128 * WN, THREADS = 768, LDS = 162816;
    static constexpr int A_CELLS = (MT + 4) * 16, A_BUF = 4 * A_CELLS;   // four cells of eight channels per row
    static constexpr int B_CELLS = (NT + 4) * 16, B_STEP = 4 * B_CELLS;
    static constexpr int kMaxK = (LDS - 2 * A_BUF) / (2 * B_STEP) * 64;
};

// K % 8 == 0 and images of a multiple of four pixels.  ROWS: the filter is contiguous along the reduction (Forward), not:
// along the rows (BackwardData), M even
template <class T, bool ROWS>
__global__ __launch_bounds__(T::THREADS, 3) void pointwise_bf16_kernel(PointwiseParams p)
{
    constexpr int WM = T::WM, WN = T::WN, MT = T::MT, NT = T::NT;
    __shared__ __attribute__((aligned(16))) char lds[T::LDS];
    char *const lds_b = lds + 2 * T::A_BUF;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave & 1) * (WM * 32), wn0 = (wave >> 1) * (WN * 32);
    int tile = (int)blockIdx.x, mt_begin = 0, mt_end = p.m_tiles;
    if (tile >= p.whole) {
        const int r = tile - p.whole, part = r % p.splits;
        tile = p.whole + r / p.splits;
        mt_begin = p.m_tiles * part / p.splits;
        mt_end = p.m_tiles * (part + 1) / p.splits;
    }
    const int j0 = tile * NT, steps = (p.K + 63) / 64 * 2;   // an even number: the producers' two sets of registers take turns
    const __amdgpu_buffer_rsrc_t rx = make_rsrc_bytes(p.x, 0, p.x_bytes), rw = make_rsrc_bytes(p.w, 0, p.w_bytes),
                                 ry = make_rsrc_bytes(p.y, 0, p.y_bytes);
    const uint32_t plane = 2u * (uint32_t)p.px;

    // producers: ROWS cells (row, eight channels) `cell` and `cell` + 256 of a step, four of a row adjacent; otherwise the same
    // eight channels of two adjacent rows, transposed on their way into LDS
    const bool producer = wave >= 8;
    const int cell = tid & 255, a_k = ROWS ? cell & 3 : cell >> 6, a_row = ROWS ? cell >> 2 : 2 * (cell & 63);
    const uint32_t a_off = ROWS ? 2u * (uint32_t)(a_row * p.w_row + 8 * a_k) : 2u * (uint32_t)(8 * a_k * p.w_k + a_row);
    struct Cells { u32x4 v[2]; };
    auto load_a = [&](int mt, int st, Cells &r) __attribute__((always_inline)) {
        // rows past the last one lie behind the filter, or are the next channel's; channels past the last one are left out
        const bool in = 32 * st + 8 * a_k < p.K;
        if constexpr (ROWS) {
            const uint32_t so = 2u * (uint32_t)(mt * MT * p.w_row + 32 * st);
#pragma unroll
            for (int x = 0; x < 2; ++x)
                r.v[x] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(in ? a_off + 2u * (uint32_t)(64 * x * p.w_row) : kOob), (int)so, 0);
        } else {
            const uint32_t so = 2u * (uint32_t)(mt * MT + 32 * st * p.w_k);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                r.v[i >> 2][i & 3] = __builtin_amdgcn_raw_buffer_load_b32(rw, (int)(in ? a_off : kOob), (int)(so + 2u * (uint32_t)(i * p.w_k)), 0);
        }
    };
    auto put_a = [&](int st, const Cells &r) __attribute__((always_inline)) {
        char *const to = lds + (st & 1) * T::A_BUF + a_k * T::A_CELLS + a_row * 16;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            u32x4 c = r.v[x];
            if constexpr (!ROWS) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    c[j] = __builtin_amdgcn_perm(r.v[j >> 1][2 * (j & 1) + 1], r.v[j >> 1][2 * (j & 1)], x ? 0x07060302u : 0x05040100u);
            }
            *reinterpret_cast<u32x4 *>(to + (ROWS ? 1024 : 16) * x) = c;
        }
    };
    Cells ra0, ra1;
    int lm = mt_begin, ls = 0;   // the step whose filter cells are loaded next
    auto next = [&]() __attribute__((always_inline)) {
        if (++ls == steps) { ls = 0; ++lm; }
    };
    if (producer) {
        load_a(lm, ls, ra0);
        next();
    }
    // all channels of the tile's pixels: eight channels of four adjacent pixels per thread and turn, transposed in registers
    for (int e = tid; e < steps * 4 * (NT / 4); e += T::THREADS) {
        const int q = e % (NT / 4), c8 = e / (NT / 4);
        uint32_t n, px;
        p.div_px.divmod((uint32_t)(j0 + 4 * q), n, px);
        const uint32_t vo = j0 + 4 * q < p.cols && 8 * c8 < p.K ? 2u * (uint32_t)(((int)n * p.K + 8 * c8) * p.px + (int)px) : kOob;
        u32x2 r[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = __builtin_amdgcn_raw_buffer_load_b64(rx, (int)vo, (int)((uint32_t)i * plane), 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            u32x4 c;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                c[j] = __builtin_amdgcn_perm(r[2 * j + 1][i >> 1], r[2 * j][i >> 1], i & 1 ? 0x07060302u : 0x05040100u);
            *reinterpret_cast<u32x4 *>(lds_b + c8 * T::B_CELLS + (4 * q + i) * 16) = c;
        }
    }
    if (producer) {
        put_a(0, ra0);
        load_a(lm, ls, ra1);
        next();
        load_a(lm, ls, ra0);
        next();
        __syncthreads();
        for (int mt = mt_begin; mt < mt_end; ++mt)
            for (int st = 0; st < steps; st += 2) {   // the cells of the step after each, loads of two steps in flight
                put_a(st + 1, ra1);
                load_a(lm, ls, ra1);
                next();
                __syncthreads();
                put_a(st + 2 < steps ? st + 2 : 0, ra0);
                load_a(lm, ls, ra0);
                next();
                __syncthreads();
            }
        return;
    }

    // even lanes store rows 2i of their pixel and the next one, odd lanes rows 2i + 1 of the pixel before and theirs
    const int odd = lane & 1;
    uint32_t out[WN];
#pragma unroll
    for (int j = 0; j < WN; ++j) {
        const int col = j0 + wn0 + 32 * j + l32;
        uint32_t n, px;
        p.div_px.divmod((uint32_t)col, n, px);
        out[j] = col < p.cols ? 2u * (uint32_t)(((int)n * p.M + wm0 + 4 * lhi + odd) * p.px + (int)px - odd) : kOob;
    }
    __syncthreads();

    for (int mt = mt_begin; mt < mt_end; ++mt) {
        f32x16 acc[WM][WN];
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
        for (int st = 0; st < steps; ++st) {
            const char *pa = lds + (st & 1) * T::A_BUF + lhi * T::A_CELLS + (wm0 + l32) * 16;
            const char *pb = lds_b + st * T::B_STEP + lhi * T::B_CELLS + (wn0 + l32) * 16;
            u32x4 va[2][WM], vb[2][WN];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int i = 0; i < WM; ++i) va[h][i] = *reinterpret_cast<const u32x4 *>(pa + 2 * h * T::A_CELLS + i * 512);
#pragma unroll
                for (int j = 0; j < WN; ++j) vb[h][j] = *reinterpret_cast<const u32x4 *>(pb + 2 * h * T::B_CELLS + j * 512);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[h][i]),
                                                                            __builtin_bit_cast(bf16x8, vb[h][j]), acc[i][j], 0, 0, 0);
            __syncthreads();
        }
        const int m0 = mt * MT + wm0;
        auto store = [&](auto wholec) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                uint32_t vo = out[j] == kOob ? kOob : out[j] + (uint32_t)(mt * MT) * plane;
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int e = 0; e < 16; e += 2) {
                        constexpr int kSwap = 0xB1;   // lanes 2i and 2i + 1 exchanged
                        const float a = acc[i][j][e], b = acc[i][j][e + 1];
                        const float give = odd ? a : b;   // what the other lane stores
                        const float got = __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(give), kSwap, 0xf, 0xf, true));
                        const uint32_t d = odd ? pack_bf16(got, b) : pack_bf16(a, got);
                        uint32_t v = vo;
                        if constexpr (!wholec) v = m0 + 32 * i + 8 * (e / 4) + e % 4 + 4 * lhi + odd < p.M ? vo : kOob;
                        __builtin_amdgcn_raw_buffer_store_b32(d, ry, (int)v, 0, 0);
                        vo += e % 4 == 2 ? 6u * plane : 2u * plane;
                        asm("" : "+v"(vo));   // one running address, not one scalar per row
                    }
            }
        };
        if (m0 + 32 * WM <= p.M) store(std::true_type{});
        else store(std::false_type{});
    }
}

// More input channels than fit LDS: input and filter stream through it together, tiles of 128 WM output channels x 256 pixels,
// eight multiplying waves (4 x 2, each 32 WM channels of 128 pixels) and four producers.  Columns of the tile are ordered so
// that a producer's transposed cells go to LDS without bank conflicts and a lane's four columns are adjacent pixels, one store.
// Memory sets the pace (each input element is read once per 256 output channels; a step of 32 channels is 768 cycles of LDS
// reads, 512 of the matrix units): loads of three steps are in flight, so that waves of a CU keep 90 KB outstanding.
// 1024 -> 256 14x14 b = 256: Forward 57 -> 34 us (129 MB at 3.8 TB/s), BackwardData of 256 -> 1024 100 -> 37.
struct StreamParams {
    const void *x, *w;
    void *y;
    uint32_t w_bytes, x_bytes, y_bytes;
    int K, M, px, cols;
    int w_row, w_k;
    int m_tiles, tiles;
    FastDiv div_px;
};

template <int WM, bool ROWS>
__global__ __launch_bounds__(768, 3) void pointwise_stream_kernel(StreamParams p)
{
    constexpr int MT = 128 * WM, NT = 256, RW = MT / 64;
    constexpr int A_CELLS = (MT + 4) * 16, A_BUF = 4 * A_CELLS, B_CELLS = (NT + 4) * 16, B_BUF = 4 * B_CELLS;
    __shared__ __attribute__((aligned(16))) char lds[2 * (A_BUF + B_BUF)];
    char *const lds_b = lds + 2 * A_BUF;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the tile rows of a pixel tile on one XCD
    const int xcd = (int)blockIdx.x % 8, rest = (int)blockIdx.x / 8;
    const int mt = rest % p.m_tiles, tile = rest / p.m_tiles * 8 + xcd;
    if (tile >= p.tiles) return;
    const int j0 = tile * NT, m0 = mt * MT, steps = (p.K + 31) / 32;
    const uint32_t plane = 2u * (uint32_t)p.px;

    if (wave >= 8) {
        const __amdgpu_buffer_rsrc_t rx = make_rsrc_bytes(p.x, 0, p.x_bytes), rw = make_rsrc_bytes(p.w, 0, p.w_bytes);
        const int cell = tid & 255, q = cell & 63, c8 = cell >> 6;
        uint32_t n, px;
        p.div_px.divmod((uint32_t)(j0 + 4 * q), n, px);
        const bool in_x = j0 + 4 * q < p.cols;
        const uint32_t b_off = 2u * (uint32_t)(((int)n * p.K + 8 * c8) * p.px + (int)px);
        // ROWS: eight channels of rows a_row + 64 x; otherwise the same of RW adjacent rows, transposed on their way into LDS
        const int a_k = ROWS ? cell & 3 : c8, a_row = ROWS ? cell >> 2 : RW * q;
        const uint32_t a_off = ROWS ? 2u * (uint32_t)((m0 + a_row) * p.w_row + 8 * a_k) : 2u * (uint32_t)(8 * a_k * p.w_k + m0 + a_row);
        struct Cells {
            u32x2 b[8];
            u32x4 a[RW];
        };
        auto load = [&](int st, Cells &r) __attribute__((always_inline)) {
            const int k0 = 32 * st < p.K ? 32 * st : 0;
            const uint32_t vb = in_x && 32 * st + 8 * c8 < p.K ? b_off : kOob;
            // rows past the last one lie behind the filter, or are the next channel's
            const bool in = 32 * st + 8 * a_k < p.K;
#pragma unroll
            for (int i = 0; i < 8; ++i) r.b[i] = __builtin_amdgcn_raw_buffer_load_b64(rx, (int)vb, (int)((uint32_t)(k0 + i) * plane), 0);
            if constexpr (ROWS) {
#pragma unroll
                for (int x = 0; x < RW; ++x)
                    r.a[x] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(in ? a_off + 2u * (uint32_t)(64 * x * p.w_row) : kOob), 2 * k0, 0);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int so = 2 * (k0 + i) * p.w_k;
                    if constexpr (RW == 4) {
                        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rw, (int)(in ? a_off : kOob), so, 0);
                        r.a[i >> 1][2 * (i & 1)] = v[0];
                        r.a[i >> 1][2 * (i & 1) + 1] = v[1];
                    } else {
                        r.a[i >> 2][i & 3] = __builtin_amdgcn_raw_buffer_load_b32(rw, (int)(in ? a_off : kOob), so, 0);
                    }
                }
            }
        };
        auto put = [&](int st, const Cells &r) __attribute__((always_inline)) {
            char *const to_b = lds_b + (st & 1) * B_BUF + c8 * B_CELLS + q * 16, *const to_a = lds + (st & 1) * A_BUF + a_k * A_CELLS;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                u32x4 c;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    c[j] = __builtin_amdgcn_perm(r.b[2 * j + 1][i >> 1], r.b[2 * j][i >> 1], i & 1 ? 0x07060302u : 0x05040100u);
                *reinterpret_cast<u32x4 *>(to_b + i * 1024) = c;
            }
#pragma unroll
            for (int x = 0; x < RW; ++x) {
                u32x4 c = r.a[x];
                if constexpr (!ROWS) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        constexpr int D = RW / 2;   // dwords per channel
                        const int lo = 2 * j * D + (x >> 1), hi = (2 * j + 1) * D + (x >> 1);
                        c[j] = __builtin_amdgcn_perm(r.a[hi >> 2][hi & 3], r.a[lo >> 2][lo & 3], x & 1 ? 0x07060302u : 0x05040100u);
                    }
                }
                *reinterpret_cast<u32x4 *>(to_a + (ROWS ? a_row * 16 : q * 16) + x * 1024) = c;
            }
        };
        Cells r0, r1, r2;   // loads of three steps in flight
        load(0, r0);
        load(1, r1);
        load(2, r2);
        put(0, r0);
        load(3, r0);
        __syncthreads();
        for (int st = 0;; st += 3) {
            put(st + 1, r1);
            load(st + 4, r1);
            __syncthreads();
            if (st + 1 >= steps) return;
            put(st + 2, r2);
            load(st + 5, r2);
            __syncthreads();
            if (st + 2 >= steps) return;
            put(st + 3, r0);
            load(st + 6, r0);
            __syncthreads();
            if (st + 3 >= steps) return;
        }
    }

    const int wm0 = (wave >> 1) * (32 * WM), wq0 = (wave & 1) * 32;
    f32x16 acc[WM][4];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    __syncthreads();
    for (int st = 0; st < steps; ++st) {
        const char *pa = lds + (st & 1) * A_BUF + lhi * A_CELLS + (wm0 + l32) * 16;
        const char *pb = lds_b + (st & 1) * B_BUF + lhi * B_CELLS + (wq0 + l32) * 16;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 va[WM], vb[4];
#pragma unroll
            for (int i = 0; i < WM; ++i) va[i] = *reinterpret_cast<const u32x4 *>(pa + 2 * h * A_CELLS + i * 512);
#pragma unroll
            for (int j = 0; j < 4; ++j) vb[j] = *reinterpret_cast<const u32x4 *>(pb + 2 * h * B_CELLS + j * 1024);
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[i]),
                                                                        __builtin_bit_cast(bf16x8, vb[j]), acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }

    const __amdgpu_buffer_rsrc_t ry = make_rsrc_bytes(p.y, 0, p.y_bytes);
    const int col = j0 + 4 * (wq0 + l32);
    if (col >= p.cols) return;
    constexpr int RS = ROWS ? 1 : RW;   // output channels between adjacent rows of the tile
    const int mw = m0 + RS * 4 * lhi + (ROWS ? wm0 : RW * (wm0 & 63) + (wm0 >> 6));
    uint32_t n, px;
    p.div_px.divmod((uint32_t)col, n, px);
    uint32_t vo = 2u * (uint32_t)(((int)n * p.M + mw) * p.px + (int)px);
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (mw + RS * (32 * i + 8 * (e / 4) + e % 4) < p.M)
                __builtin_amdgcn_raw_buffer_store_b64(u32x2{pack_bf16(acc[i][0][e], acc[i][1][e]), pack_bf16(acc[i][2][e], acc[i][3][e])},
                                                      ry, (int)vo, 0, 0);
            vo += (uint32_t)(e % 4 == 3 ? 5 * RS : RS) * plane;
            asm("" : "+v"(vo));   // one running address, not one scalar per row
        }
}

}  // namespace ucd
