// Forward and BackwardData of 3x3 stride-1 layers with bf16 tensors over a window kept in LDS, on v_mfma_f32_32x32x16_bf16.
//
// An implicit GEMM fetches and transposes an input element once per tap that reads it (the images are contiguous along
// pixels, an MFMA operand is eight channels of one pixel).  Here a workgroup of eight waves turns the window of its
// output positions into operands once per 16 channels: cells of 16 bytes, eight channels of one pixel, so that a tap is an
// offset of the operand's address.  The filter is turned the same way, from the runs in which it lies in memory: 16 channels of an output channel
// (Forward), all of a workgroup's input channels of one output channel (BackwardData).
//
// A chunk of 16 channels is 9 steps of one MFMA per 32 x 32 tile; its operands are put into LDS while the chunk before it is
// multiplied, in two parts with a barrier behind each: the filter's runs as they are and the window's cells, then the
// filter's cells from the runs.  The two waves of a SIMD do that work at different ends of a part.
//
// Positions run over images, blocks of Wc columns, rows, columns of the block; a tile is NT consecutive ones.  Window rows
// are those of the images with ph zero rows in front of each, which also serve the image before.
//
// 128 x 512, 384 -> 384 13x13 b = 256: 100 us, 1150 TFLOP/s; 46 % of the matrix pipe's cycles are MFMAs, 2.2 other vector instructions each.
// An operand serves two or four MFMAs, so that LDS moves 1 KB per MFMA, and that, with the barriers, is what bounds the kernel.
#pragma once
#include "gemm_core.hpp"

namespace ucd {

constexpr int kWinC = 16;   // channels per chunk

struct WindowParams {
    const void *in, *w;
    void *out;
    uint32_t in_bytes, w_bytes, out_bytes;
    int Ci, Hi, Wi, Co, Ho, Wo;     // as convolved: BackwardData has dy as input
    int ph, pw;
    int Wc, nb, runs, rows, pitch, cells;   // columns per block, blocks; runs of four cells per window row, rows, row pitch and cells in LDS
    int images, cols, tiles_m;      // images * blocks, positions, row tiles
    FastDiv div_wc, div_ho, div_nb, div_runs, div_rows, div_step;   // div_step: window rows from one image to the next
};

// OP 0 Forward, 1 BackwardData; a wave owns WM x WN tiles of 32 x 32, WAVES_N of the eight waves side by side
template <int OP_, int WM_, int WN_, int WAVES_N_>
struct WindowTile {
    static constexpr int OP = OP_, WM = WM_, WN = WN_, WAVES_N = WAVES_N_, WAVES_M = 8 / WAVES_N_;
    static constexpr int MT = 32 * WM * WAVES_M, NT = 32 * WN * WAVES_N;
    static constexpr int A_HALF = MT * 16, A_TAP = 2 * A_HALF, A_BUF = 9 * A_TAP;
    // the filter's runs: of an output channel 16 channels, or of a channel all MT output channels and a few bytes that spread
    // the channels over the banks
    static constexpr int kRow = OP == 0 ? 18 * kWinC : 18 * MT + 32, RAW = OP == 0 ? MT * kRow : kWinC * kRow;
    static constexpr int kPieces = OP == 0 ? kRow / 16 : 18 * MT / 16, NP = (MT * 18 + 511) / 512;   // of 16 bytes: per run, per thread
    static constexpr bool kPair = WM * WN == 1;   // two workgroups share a CU
    static constexpr int LDS = kPair ? 81920 : MT == 128 ? 163840 : 131072;
    static_assert(MT == 128 || MT == 64 || MT == 32, "put_a's rows");
    static constexpr int kMaxCells = (LDS - 2 * A_BUF - RAW) / 64;
};

template <class T>
__global__ __launch_bounds__(512, T::kPair ? 4 : 2) void conv_window_kernel(WindowParams p)
{
    constexpr int WM = T::WM, WN = T::WN, MT = T::MT, NT = T::NT, NP = T::NP;
    __shared__ __attribute__((aligned(16))) char lds[T::LDS];
    char *const raw = lds + 2 * T::A_BUF, *const win = raw + T::RAW;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / T::WAVES_N) * (WM * 32), wn0 = (wave % T::WAVES_N) * (WN * 32);

    const uint32_t id = xcd_order(blockIdx.x, gridDim.x);
    const int m0 = (int)(id % (uint32_t)p.tiles_m) * MT, j0 = (int)(id / (uint32_t)p.tiles_m) * NT;

    const __amdgpu_buffer_rsrc_t rin = make_rsrc_bytes(p.in, 0, p.in_bytes), rw = make_rsrc_bytes(p.w, 0, p.w_bytes),
                                 rout = make_rsrc_bytes(p.out, 0, p.out_bytes);
    const int half_b = p.cells * 16, buf_b = 2 * half_b;
    const int step = p.Hi + p.ph;
    const int g0 = (int)p.div_wc.div((uint32_t)j0), v0 = (int)p.div_ho.div((uint32_t)g0);
    const int rho0 = v0 * step + (g0 - v0 * p.Ho);   // the window's first row

    // the window: a thread takes four adjacent cells of a row for eight channels.  It loads four pixels that lie in
    // the row, and the selectors move them to where the cells' columns are, zeros to where there is no pixel.
    uint32_t b_off = kOob, b_lo = 0x03020100u, b_hi = 0x07060504u;
    int b_dst = -1, b_c = 0;
    {
        uint32_t e1, run, half, lr;
        p.div_runs.divmod((uint32_t)tid, e1, run);
        p.div_rows.divmod(e1, half, lr);
        if (half < 2) {
            b_dst = (int)half * half_b + ((int)lr * p.pitch + 4 * (int)run) * 16;
            b_c = 8 * (int)half;
            uint32_t v, h, n, cb;
            p.div_step.divmod((uint32_t)rho0 + lr, v, h);
            p.div_nb.divmod(v, n, cb);
            const int hi = (int)h - p.ph, col = (int)cb * p.Wc + 4 * (int)run - p.pw;
            const int at = min(max(col, 0), p.Wi - 4), sh = col - at;
            if ((int)v < p.images && hi >= 0 && sh > -4 && sh < 4) {
                b_off = 2u * (uint32_t)((((int)n * p.Ci + b_c) * p.Hi + hi) * p.Wi + at);
                b_lo = b_hi = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int k = i + sh;
                    const uint32_t sel = k >= 0 && k < 4 ? (uint32_t)(2 * k) * 0x0101u + 0x0100u : 0x0c0cu;
                    (i < 2 ? b_lo : b_hi) |= sel << (16 * (i & 1));
                }
            }
        }
    }
    // the filter's pieces of 16 bytes
    uint32_t a_off[NP];
#pragma unroll
    for (int x = 0; x < NP; ++x) {
        const int e = tid + 512 * x, row = e / T::kPieces, piece = e % T::kPieces;
        a_off[x] = e < MT * 18 ? (uint32_t)(T::OP == 0 ? (m0 + row) * p.Ci * 18 : (row * p.Co + m0) * 18) + 16u * piece : kOob;
    }
    // this lane's columns: the cell of tap (0, 0)
    int col_cell[WN];
#pragma unroll
    for (int i = 0; i < WN; ++i) {
        const int j = min(j0 + wn0 + 32 * i + l32, p.cols - 1);
        uint32_t g, u, v, t;
        p.div_wc.divmod((uint32_t)j, g, u);
        p.div_ho.divmod(g, v, t);
        col_cell[i] = lhi * half_b + (((int)v * step + (int)t - rho0) * p.pitch + (int)u) * 16;
    }

    const int chunks = (p.Ci + kWinC - 1) / kWinC;
    const uint32_t in_plane = 2u * (uint32_t)(p.Hi * p.Wi);
    u32x4 ra[NP];
    u32x2 rb[8];
    auto load_a = [&](int c) __attribute__((always_inline)) {
        const uint32_t so = (uint32_t)c * (uint32_t)(T::OP == 0 ? 18 * kWinC : 18 * kWinC * p.Co);
#pragma unroll
        for (int x = 0; x < NP; ++x) ra[x] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)a_off[x], (int)so, 0));
    };
    auto load_b = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            uint32_t vo = b_off;
            if (kWinC * (c + 1) > p.Ci) vo = kWinC * c + b_c + i < p.Ci ? vo : kOob;   // channels past the last one are the next image's
            rb[i] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rin, (int)vo, (int)((uint32_t)(kWinC * c + i) * in_plane), 0));
        }
    };
    constexpr uint32_t kLow = 0x05040100u, kHigh = 0x07060302u;   // the low / high halves of two words
    auto put_raw = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NP; ++x) {
            const int e = tid + 512 * x;
            if (512 * (x + 1) <= MT * 18 || e < MT * 18) {
                const int at = T::OP == 0 ? e * 16 : (e / T::kPieces) * T::kRow + (e % T::kPieces) * 16;
                *reinterpret_cast<u32x4 *>(raw + at) = ra[x];
            }
        }
    };
    auto put_b = [&](int buf) __attribute__((always_inline)) {
        if (b_dst < 0) return;
        char *dst = win + buf * buf_b + b_dst;
        u32x4 cell[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t x0 = __builtin_amdgcn_perm(rb[2 * q][1], rb[2 * q][0], b_lo), x1 = __builtin_amdgcn_perm(rb[2 * q][1], rb[2 * q][0], b_hi);
            const uint32_t y0 = __builtin_amdgcn_perm(rb[2 * q + 1][1], rb[2 * q + 1][0], b_lo);
            const uint32_t y1 = __builtin_amdgcn_perm(rb[2 * q + 1][1], rb[2 * q + 1][0], b_hi);
            cell[0][q] = __builtin_amdgcn_perm(y0, x0, kLow);
            cell[1][q] = __builtin_amdgcn_perm(y0, x0, kHigh);
            cell[2][q] = __builtin_amdgcn_perm(y1, x1, kLow);
            cell[3][q] = __builtin_amdgcn_perm(y1, x1, kHigh);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4 *>(dst + 16 * i) = cell[i];
    };
    // the filter's cells: eight channels of a tap and row; the second half's rows are exchanged by eights, so that both halves'
    // pieces that a wave writes at a time fall on different banks
    auto put_a = [&](int c, int buf) __attribute__((always_inline)) {
        char *dst = lds + buf * T::A_BUF;
        if constexpr (T::OP == 0) {
            const int q = tid & 3, m = tid >> 2;   // four channels of a row
            if (MT == 128 || m < MT) {
                const char *src = raw + m * T::kRow + q * 72;
                uint32_t d[18];
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const u32x2 v = *reinterpret_cast<const u32x2 *>(src + 8 * i);
                    d[2 * i] = v[0]; d[2 * i + 1] = v[1];
                }
                u32x2 keep = {0xFFFFFFFFu, 0xFFFFFFFFu};
                const bool tail = kWinC * (c + 1) > p.Ci;   // behind the last channel the next row begins
                if (tail) {
                    // (channels are even; without the masks of an odd rest the kernel is compiled to be 3 % slower)
                    const int left = p.Ci - kWinC * c - 4 * q;
                    keep[0] = left >= 2 ? 0xFFFFFFFFu : left == 1 ? 0xFFFFu : 0u;
                    keep[1] = left >= 4 ? 0xFFFFFFFFu : left == 3 ? 0xFFFFu : 0u;
                }
                dst += (q >> 1) * T::A_HALF + (m ^ ((q >> 1) << 3)) * 16 + (q & 1) * 8;
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    u32x2 v;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int e0 = 18 * i + t, e1 = e0 + 9;
                        const uint32_t sel = (e0 & 1 ? 0x0302u : 0x0100u) | (e1 & 1 ? 0x07060000u : 0x05040000u);
                        v[i] = __builtin_amdgcn_perm(d[e1 >> 1], d[e0 >> 1], sel);
                    }
                    if (tail) { v[0] &= keep[0]; v[1] &= keep[1]; }
                    *reinterpret_cast<u32x2 *>(dst + t * T::A_TAP) = v;
                }
            }
        } else {
            const int kp = tid & 3, mp = (tid >> 2) % (MT / 2), half = (tid >> 2) / (MT / 2);   // two channels of two rows
            if (half < 2) {
                const char *src = raw + (8 * half + 2 * kp) * T::kRow + mp * 36;
                uint32_t d0[9], d1[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    d0[i] = *reinterpret_cast<const uint32_t *>(src + 4 * i);
                    d1[i] = *reinterpret_cast<const uint32_t *>(src + T::kRow + 4 * i);
                }
                dst += half * T::A_HALF + ((2 * mp) ^ (half << 3)) * 16 + kp * 4;
#pragma unroll
                for (int t = 0; t < 9; ++t)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int e = 9 * i + 8 - t;   // taps reversed
                        *reinterpret_cast<uint32_t *>(dst + t * T::A_TAP + 16 * i) = __builtin_amdgcn_perm(d1[e >> 1], d0[e >> 1], e & 1 ? kHigh : kLow);
                    }
            }
        }
    };

    f32x16 acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    load_a(0);
    load_b(0);
    put_raw();
    put_b(0);
    if (chunks > 1) { load_a(1); load_b(1); }
    __syncthreads();
    put_a(0, 0);
    __syncthreads();

    const bool early = WM * WN < 8 || wave < 4;
    const char *const a_base = lds + lhi * T::A_HALF + ((wm0 + l32) ^ (lhi << 3)) * 16;
    for (int c = 0; c < chunks; ++c) {
        const bool more = c + 1 < chunks;
        const char *pa = a_base + (c & 1) * T::A_BUF;
        const char *pb = win + (c & 1) * buf_b;
        u32x4 va[2][WM], vb[2][WN];
        auto read = [&](int t, int x) __attribute__((always_inline)) {   // operand x of tap t: the rows', then the columns'
            if (x < WM) va[t & 1][x] = *reinterpret_cast<const u32x4 *>(pa + t * T::A_TAP + x * 32 * 16);
            else vb[t & 1][x - WM] = *reinterpret_cast<const u32x4 *>(pb + col_cell[x - WM] + ((t / 3) * p.pitch + t % 3) * 16);
        };
        // The next tap's operands are read in front of the MFMAs; of eight, one behind each (128 x 512: 101 against 99 us for
        // 384 -> 384 13x13 b = 256; of two and four 171 against 163).
        auto tap = [&](int t) __attribute__((always_inline)) {
            constexpr int kReads = WM + WN, kMfmas = WM * WN;
            if (t < 8 && kMfmas < 8)
#pragma unroll
                for (int x = 0; x < kReads; ++x) read(t + 1, x);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < kMfmas; ++m) {
                const int i = m / WN, j = m % WN;
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[t & 1][i]),
                                                                    __builtin_bit_cast(bf16x8, vb[t & 1][j]), acc[i][j], 0, 0, 0);
                if (kMfmas < 8) continue;
                __builtin_amdgcn_sched_barrier(0);
                if (t < 8 && m < kReads) read(t + 1, m);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto first = [&]() __attribute__((always_inline)) {
            if (!more) return;
            put_raw();
            put_b((c + 1) & 1);
            if (c + 2 < chunks) { load_a(c + 2); load_b(c + 2); }
        };
#pragma unroll
        for (int x = 0; x < WM + WN; ++x) read(0, x);
        if (early) first();
#pragma unroll
        for (int t = 0; t < 4; ++t) tap(t);
        if (!early) first();
        __syncthreads();
        if (early && more) put_a(c + 1, (c + 1) & 1);
#pragma unroll
        for (int t = 4; t < 9; ++t) tap(t);
        if (!early && more) put_a(c + 1, (c + 1) & 1);
        __syncthreads();
    }

    const uint32_t plane = 2u * (uint32_t)(p.Ho * p.Wo);
#pragma unroll
    for (int j = 0; j < WN; ++j) {
        const int jo = j0 + wn0 + 32 * j + l32;
        uint32_t g, u, v, t, n, cb;
        p.div_wc.divmod((uint32_t)jo, g, u);
        p.div_ho.divmod(g, v, t);
        p.div_nb.divmod(v, n, cb);
        const int w = (int)cb * p.Wc + (int)u;
        const int k = m0 + wm0 + 4 * lhi;
        const bool in = jo < p.cols && w < p.Wo, whole = m0 + wm0 + 32 * WM <= p.Co;
        uint32_t vo = in ? 2u * (uint32_t)((((int)n * p.Co + k) * p.Ho + (int)t) * p.Wo + w) : kOob;
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                uint32_t h;
                asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(h) : "v"(acc[i][j][e]), "v"(acc[i][j][e + 1]));
                uint32_t v0o = vo, v1o = vo + plane;
                if (!whole) {
                    const int row = k + 32 * i + 8 * (e / 4) + e % 4;
                    v0o = row < p.Co ? v0o : kOob;
                    v1o = row + 1 < p.Co ? v1o : kOob;
                }
                __builtin_amdgcn_raw_buffer_store_b16((short)h, rout, (int)v0o, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b16((short)(h >> 16), rout, (int)v1o, 0, 0);
                vo += e % 4 == 2 ? 6u * plane : 2u * plane;
            }
    }
}

}  // namespace ucd
