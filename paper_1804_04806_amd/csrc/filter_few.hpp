// BackwardFilter of fp32 layers with few input channels (a network's first layer) on the bf16 matrix pipe, with split operands (products, error
// and range as in gemm_split.hpp).
//
// The columns of the GEMM are the filter's elements (c, r, s), the reduction runs over pixels of dy, eight adjacent ones of a row per
// operand.  Tile GEMMs gather x once per element and read dy once per tile of columns; here a workgroup owns all columns (of as many channels as
// fit), so that dy is read and split once, and keeps a window of x, split once too.  Its rows stand by column modulo the stride: the
// eight pixels that a tap meets are neighbours there, and begin on any element: taps that begin on an odd one have tiles of columns of their own, whose
// operands are five words and a shift.  A word's parts stand side by side, so that one address reads an operand.
//
// A tile is G groups of eight pixels (running over images, blocks of gw groups of columns, rows, groups of the block).  Of the eight waves WR
// share the output channels and 8 / WR the groups, two steps of two groups each; a wave multiplies its 32 output channels with all columns, so
// that the filter's sums, the larger part of which are registers, are held once per share of the groups and meet at the end, in LDS and
// then by atomics.  LDS holds two tiles: one is multiplied while the next is split into place and the one after is on its way.
//
// 3 -> 64 7x7/2 224x224 b = 128: 385 us as tile GEMMs, 266 with this; its MFMAs, 8 % on columns that do not exist, would
// take 98, its bytes 93.  What is left is 7.4 vector instructions per MFMA (the splits, and x's addresses) and LDS, where an operand's 32
// columns meet 2.2 times on a bank.  A window row has an odd number of pairs per phase for that: 3 -> 64 7x7 120x120 b = 73 with
// three groups to a block 238 -> 182 us.  Waves that stage at different ends of a tile made it 3 % slower, and x's addresses
// kept in registers, which then spill, 11 %.
#pragma once
#include "gemm_split.hpp"

namespace ucd {

struct FilterFewParams {
    const void *x, *dy;
    float *dw;
    uint32_t x_bytes, dy_bytes;
    int C, H, W, K, P, Q, R, S, CRS, sh, sw, ph, pw;
    int gw, nb, half, rows, pairs;                  // groups per block, blocks; pairs per phase of a window row, rows per channel, pairs
    int images, groups, tiles;                      // images * blocks, groups, tiles
    int CB, c_blocks, k_blocks;                     // channels per block, blocks of channels and of output channels
    int taps[2];                                    // of a filter row, that begin on an even and on an odd element
    FastDiv div_gw, div_p, div_nb, div_len, div_rows, div_half, div_sw, div_r, div_taps[2];
};

// NE and NO tiles of columns for even and odd taps
template <int WR_, int NE_, int NO_>
struct FilterFewTile {
    static constexpr int WR = WR_, WQ = 8 / WR_, NE = NE_, NO = NO_, NJ = NE_ + NO_, MT = 32 * WR, G = 4 * WQ, PARTS = 3;
    static constexpr int PG = G + 1, A_PART = MT * PG * 16, A_BUF = PARTS * A_PART;    // an odd pitch
    static constexpr int NX = 4, kRows = 128;                                           // pairs of x per thread; rows of a window
    static constexpr int LDS = 163840 - 512 - 24 * kRows - 36 * G;
    static constexpr int kFits = (LDS - 2 * A_BUF) / (4 * PARTS) / 8 * 8, kMaxElements = (kFits < 1024 * NX ? kFits : 1024 * NX) - 16;
    static constexpr int B_BUF = 2 * PARTS * (kMaxElements + 16);
    static_assert(MT * G == 1024 && 2 * (A_BUF + B_BUF) <= LDS && 2 * (A_BUF + B_BUF) >= 8 * 4096, "two cells per thread");
};

template <class T>
__global__ __launch_bounds__(512, 2) void filter_few_kernel(FilterFewParams p)
{
    constexpr int WQ = T::WQ, NJ = T::NJ, MT = T::MT, G = T::G, PARTS = T::PARTS, NX = T::NX;
    __shared__ __attribute__((aligned(16))) char lds[T::LDS];
    __shared__ int row_tab[6 * T::kRows], g_cell[3 * G], g_left[3 * G], g_dy[3 * G];   // of three tiles
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wk = wave / WQ, wq = wave % WQ;

    uint32_t id = xcd_order(blockIdx.x, gridDim.x);
    const int k0 = (int)(id % (uint32_t)p.k_blocks) * MT; id /= (uint32_t)p.k_blocks;
    const int c0 = (int)(id % (uint32_t)p.c_blocks) * p.CB; id /= (uint32_t)p.c_blocks;
    const int first = (int)id, stride = (int)(gridDim.x / (uint32_t)(p.k_blocks * p.c_blocks));
    const int rows_w = min(p.CB, p.C - c0) * p.R;   // rows of the filter

    const __amdgpu_buffer_rsrc_t rx = make_rsrc_bytes(p.x, 0, p.x_bytes), rd = make_rsrc_bytes(p.dy, 0, p.dy_bytes);
    const int len = p.sh * (p.P - 1) + p.R, row_cells = 2 * p.half * p.sw;

    // where a tile's groups lie in dy (of output channel 0) and in the window, how many of their pixels exist; where the window's rows lie in x
    // (less their first column) and that column: rows of the first virtual image (images x blocks) from the tile's first group on, then whole ones
    auto tables = [&](int n, int slot) __attribute__((always_inline)) {
        const int j0 = n * G, a0 = (int)p.div_gw.div((uint32_t)j0), v0 = (int)p.div_p.div((uint32_t)a0), t0 = a0 - v0 * p.P, len0 = len - p.sh * t0;
        if (tid < T::kRows) {
            uint32_t cc, lr, img, cb;
            p.div_rows.divmod((uint32_t)tid, cc, lr);
            int v = v0, row = p.sh * t0 + (int)lr;
            if ((int)lr >= len0) {
                const int k = (int)p.div_len.div(lr - (uint32_t)len0);
                v = v0 + 1 + k;
                row = (int)lr - len0 - k * len;
            }
            row -= p.ph;
            p.div_nb.divmod((uint32_t)v, img, cb);
            const bool ok = n < p.tiles && c0 + (int)cc < p.C && v < p.images && (unsigned)row < (unsigned)p.H;
            row_tab[2 * (slot * T::kRows + tid)] = ok ? (((int)img * p.C + c0 + (int)cc) * p.H + row) * p.W : 0;
            row_tab[2 * (slot * T::kRows + tid) + 1] = ok ? 8 * (int)cb * p.gw * p.sw - p.pw : -(1 << 30);
        } else if (tid - T::kRows < G) {
            const int g = tid - T::kRows, j = j0 + g;
            uint32_t a, u, v, t, img, cb;
            p.div_gw.divmod((uint32_t)min(j, p.groups - 1), a, u);
            p.div_p.divmod(a, v, t);
            p.div_nb.divmod(v, img, cb);
            const int q = 8 * ((int)cb * p.gw + (int)u);
            const int row = (int)v == v0 ? p.sh * ((int)t - t0) : len0 + ((int)v - v0 - 1) * len + p.sh * (int)t;
            const int left = j < p.groups && n < p.tiles ? max(0, min(8, p.Q - q)) : 0;
            g_cell[slot * G + g] = n < p.tiles ? PARTS * ((row * row_cells + 8 * (int)u) >> 1) : 0;
            g_left[slot * G + g] = left;
            g_dy[slot * G + g] = left > 0 ? (((int)img * p.K) * p.P + (int)t) * p.Q + q : -1;
        }
    };

    u32x4 qd[2][2];
    float qx[NX][2];
    int left_d;   // pixels of this thread's group
    const int dg = tid % G;
    auto load = [&](int slot) __attribute__((always_inline)) {
        const int at = g_dy[slot * G + dg];
        left_d = g_left[slot * G + dg];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = k0 + (tid + 512 * i) / G;
            const uint32_t vo = at >= 0 && k < p.K ? 4u * (uint32_t)(at + k * p.P * p.Q) : kOob;
#pragma unroll
            for (int h = 0; h < 2; ++h) qd[i][h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rd, (int)vo + 16 * h, 0, 0));
        }
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            if (512 * x >= p.pairs) break;
            int e = tid + 512 * x;
            asm volatile("" : "+v"(e));   // not before the break, nor kept
            uint32_t cp, m, cr, a;
            p.div_half.divmod((uint32_t)min(e, p.pairs - 1), cp, m);
            p.div_sw.divmod(cp, cr, a);
            const int *const rt = row_tab + 2 * (slot * T::kRows + (int)cr);
            const int from = rt[0], col = rt[1] + 2 * (int)m * p.sw + (int)a;
            qx[x][0] = Elem<float>::load(rx, (unsigned)col < (unsigned)p.W ? 4u * (uint32_t)(from + col) : kOob, 0u);
            qx[x][1] = Elem<float>::load(rx, (unsigned)(col + p.sw) < (unsigned)p.W ? 4u * (uint32_t)(from + col + p.sw) : kOob, 0u);
        }
    };
    uint32_t rest = 0;
    const bool ragged = p.Q % 8 != 0;
    auto put = [&](auto fp32c, int buf) __attribute__((always_inline)) {
        constexpr bool FP32 = fp32c;
        char *const da = lds + buf * T::A_BUF, *const db = lds + 2 * T::A_BUF + buf * T::B_BUF;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            char *dst = da + ((tid + 512 * i) / G * T::PG + dg) * 16;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(qd[i][e >> 2][e & 3]);
            if (ragged)
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = e < left_d ? v[e] : 0.f;
            if constexpr (FP32) {
                *reinterpret_cast<f32x4 *>(dst) = f32x4{v[0], v[1], v[2], v[3]};
                *reinterpret_cast<f32x4 *>(dst + T::A_PART) = f32x4{v[4], v[5], v[6], v[7]};
            } else {
                u32x4 c[3];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t h, m, l;
                    split_pair(v[2 * e], v[2 * e + 1], h, m, l, rest);
                    c[0][e] = h; c[1][e] = m; c[2][e] = l;
                }
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4 *>(dst + pl * T::A_PART) = c[pl];
            }
        }
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            if (512 * x >= p.pairs) break;
            const int e = tid + 512 * x;
            if (e >= p.pairs) break;
            uint32_t *const dst = reinterpret_cast<uint32_t *>(db) + PARTS * e;
            if constexpr (FP32) {
                dst[0] = __float_as_uint(qx[x][0]);
                dst[1] = __float_as_uint(qx[x][1]);
            } else {
                uint32_t h, m, l;
                split_pair(qx[x][0], qx[x][1], h, m, l, rest);
                dst[0] = h; dst[1] = m; dst[2] = l;
            }
        }
    };

    // column 32 j + l32 of the even or odd taps: row of the filter and tap
    auto column = [&](int lane32, int j, int &row, int &s) __attribute__((always_inline)) {
        const int odd = j >= T::NE, n = 32 * (odd ? j - T::NE : j) + lane32;
        uint32_t cr, k, i, a;
        p.div_taps[odd].divmod((uint32_t)n, cr, k);
        p.div_sw.divmod(k, i, a);
        row = (int)cr;
        s = (2 * (int)i + odd) * p.sw + (int)a;
        return n < rows_w * p.taps[odd];
    };
    // where its tap lies in the window, from a group's first cell on (words of a part; the word that an odd tap begins in)
    int col[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        int row, s;
        const bool ok = column(l32, j, row, s);
        uint32_t c, r, idx, a;
        p.div_r.divmod((uint32_t)row, c, r);
        p.div_sw.divmod((uint32_t)s, idx, a);
        col[j] = ok ? PARTS * ((((int)c * p.rows + (int)r) * row_cells + (int)a * 2 * p.half + (int)idx) >> 1) : 0;
    }

    f32x16 acc[NJ], low[NJ];
    auto pass = [&](auto fp32c) __attribute__((always_inline)) {
        constexpr bool FP32 = fp32c;   // operands as they are, on the fp32 instructions; pixels that only meet zeros are zeros
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) { acc[j][e] = 0.f; low[j][e] = 0.f; }
        tables(first, 0);
        __syncthreads();
        load(0);
        __syncthreads();
        put(fp32c, 0);
        tables(first + stride, 1);
        __syncthreads();
        load(1);

        int buf = 0, slot = 0;
        for (int n = first; n < p.tiles; n += stride) {
            const int next = slot == 2 ? 0 : slot + 1, after = next == 2 ? 0 : next + 1;
            const char *const pa = lds + buf * T::A_BUF + ((32 * wk + l32) * T::PG + lhi) * 16, *const pb = lds + 2 * T::A_BUF + buf * T::B_BUF;
            auto step = [&](int s) __attribute__((always_inline)) {
                const int cell = g_cell[slot * G + 2 * s + lhi];   // words
                if constexpr (FP32) {
                    const int left = g_left[slot * G + 2 * s + lhi];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const f32x4 va = *reinterpret_cast<const f32x4 *>(pa + 32 * s + h * T::A_PART);
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int i = 4 * h + e + (j >= T::NE);
                                float b = reinterpret_cast<const float *>(pb)[cell + col[j] + PARTS * (i >> 1) + (i & 1)];
                                b = 4 * h + e < left ? b : 0.f;
                                acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[e], b, acc[j], 0, 0, 0);
                            }
                    }
                } else {
                    u32x4 va[PARTS];
#pragma unroll
                    for (int pl = 0; pl < PARTS; ++pl) va[pl] = *reinterpret_cast<const u32x4 *>(pa + 32 * s + pl * T::A_PART);
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        u32x4 vb[PARTS];
                        const uint32_t *const src = reinterpret_cast<const uint32_t *>(pb) + (cell + col[j]);
#pragma unroll
                        for (int pl = 0; pl < PARTS; ++pl) {
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                vb[pl][i] = j < T::NE ? src[PARTS * i + pl] : __builtin_amdgcn_alignbit(src[PARTS * (i + 1) + pl], src[PARTS * i + pl], 16);
                        }
                        constexpr int PL_A[6] = {0, 2, 1, 1, 0, 0}, PL_B[6] = {0, 0, 1, 0, 1, 2};
#pragma unroll
                        for (int m = 0; m < 6; ++m) {
                            f32x16 &d = m == 0 ? acc[j] : low[j];
                            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[PL_A[m]]), __builtin_bit_cast(bf16x8, vb[PL_B[m]]), d,
                                                                        0, 0, 0);
                        }
                    }
                }
            };
            step(2 * wq);
            if (n + stride < p.tiles) put(fp32c, buf ^ 1);
            step(2 * wq + 1);
            tables(n + 2 * stride, after);
            __syncthreads();
            load(after);
            buf ^= 1;
            slot = next;
        }
    };
    pass(std::false_type{});
    float not_finite = 0.f;
    uint32_t least = 0xFFFFFFFFu;
    auto sums = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float v = acc[j][e] + low[j][e];
                acc[j][e] = v;
                not_finite = fmaf(v, 0.f, not_finite);
                least = min(least, (__float_as_uint(v) << 1) - 1u);
            }
    };
    sums();
    // not finite, or below 2^-104 and not zero (see conv_halo.hpp)
    if (__syncthreads_or(!(not_finite == 0.f) || (rest & 0xFFFFu) != 0 || least < ((127u - 104u) << 24) - 1u)) {
        pass(std::true_type{});
        sums();
    }

    // the waves that shared the groups give each other their sums, a tile of columns at a time, and each adds a part of the rows to dw
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        float *const meet = reinterpret_cast<float *>(lds);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16; ++e) meet[(wave * 16 + e) * 64 + lane] = acc[j][e];
        __syncthreads();
        int row, s, again = l32;
        asm volatile("" : "+v"(again));   // not kept from above
        const bool ok = column(again, j, row, s);
#pragma unroll
        for (int i = 0; i < 16 / WQ; ++i) {
            const int e = wq * (16 / WQ) + i, k = k0 + 32 * wk + 8 * (e >> 2) + 4 * lhi + (e & 3);
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < WQ; ++w) v += meet[((wk * WQ + w) * 16 + e) * 64 + lane];
            if (k < p.K && ok) unsafeAtomicAdd(p.dw + (size_t)k * p.CRS + (size_t)(c0 * p.R + row) * p.S + s, v);
        }
    }
}

}  // namespace ucd
