// BackwardData of layers with few input channels (a network's first layer) over a window in LDS, on the bf16 matrix pipe; fp32 tensors as
// split operands (products, error and range as in gemm_split.hpp), bf16 tensors as they are.
//
// The rows of an MFMA tile are the pixels of a block of vsh x vsw of dx (fh x fw strides) times the input channels: with
//     h + ph = vsh*t + a,   p = fh*t + (fh - 1) - u,   r = a - sh*(fh - 1) + sh*u   (no such tap: zero)
// all of them meet the same window of dy, u = 0 .. ceil(R / sh) + fh - 2 (columns likewise).  Merging as many pixels as 32 rows hold leaves fewest of
// a tile's rows empty; how many of the window's taps are real falls with it.
//
// A workgroup keeps the window of 256 positions (blocks) in LDS as operands, split once: a cell of 16 bytes per part holds eight channels of a
// pixel.  The two halves of an MFMA's reduction are two taps of those eight channels, not 16 channels of a tap: that halves the window, which
// is what decides whether it fits twice.  Window columns stand by their remainder modulo fw, so that neighbouring positions read
// neighbouring cells.  Of the eight waves four share the positions and two the taps: a wave multiplies every other pair of taps for
// 64 positions, so that an operand of the filter serves two tiles (with 32 positions and all pairs LDS alone would take as long as the MFMAs), and the
// two sums meet at the end.
//
// 3 -> 64 7x7/2 224x224 b = 128: 818 us as tile GEMMs of merged phases on the fp32 instructions, 432 with this; its MFMAs alone, with three
// quarters of the rows and 61 % of the taps real, would be 180.  39 % of the matrix pipe's cycles are MFMAs, with 5.9 other vector instructions
// each (the split of the window's cells, half of them, and of the filter's); operands read a pair ahead made it 3 % slower.
#pragma once
#include "gemm_split.hpp"

namespace ucd {

constexpr int kFewC = 8;        // channels per chunk
constexpr int kFewN = 256;      // positions per tile
constexpr int kFewPairs = 12;   // pairs of taps whose filter cells are in LDS at a time, at most
constexpr int kFewLds = 162560, kFewTaps = 256;

struct FewParams {
    const void *in, *w;
    void *out;
    uint32_t in_bytes, w_bytes, out_bytes;
    int K, P, Q, C, H, W, R, S, CRS;
    int sh, sw, ph, pw, fh, fw, vsh, vsw, U, V, taps;
    int pairs, groups;                    // pairs of taps per step, steps per chunk
    int Hb, Wc, nb, span, pitch, cells;   // position rows, columns per block, blocks; cells per remainder, window row and part
    int images, cols;                     // images * blocks, positions
    FastDiv div_wc, div_hb, div_nb, div_pitch, div_span, div_v, div_block, div_vsw;
};

template <class E>
__global__ __launch_bounds__(512, 2) void conv_few_kernel(FewParams p)
{
    constexpr bool F32 = std::is_same<E, float>::value;
    constexpr int PARTS = F32 ? 3 : 1, NA = (kFewPairs * 64 + 511) / 512, NB = 3, EB = (int)Elem<E>::kBytes;
    __shared__ __attribute__((aligned(16))) char lds[kFewLds];
    __shared__ int tab[kFewTaps];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn0 = (wave & 3) * 64, wr = wave >> 2;
    const int j0 = (int)xcd_order(blockIdx.x, gridDim.x) * kFewN;

    const __amdgpu_buffer_rsrc_t rin = make_rsrc_bytes(p.in, 0, p.in_bytes), rw = make_rsrc_bytes(p.w, 0, p.w_bytes),
                                 rout = make_rsrc_bytes(p.out, 0, p.out_bytes);
    const int a_part = p.pairs * 64 * 16, a_buf = PARTS * a_part, b_part = p.cells * 16, b_buf = PARTS * b_part;
    char *const lds_b = lds + 2 * a_buf;

    // the cell that tap (u, v) reads less the one of the last tap
    if (tid < kFewTaps) {
        uint32_t u, v;
        p.div_v.divmod((uint32_t)tid, u, v);
        const int dv = p.V - 1 - (int)v;
        tab[tid] = tid < p.taps ? ((p.U - 1 - (int)u) * p.pitch + dv % p.fw * p.span + dv / p.fw) * 16 : 0;
    }

    // the window: rows of the first virtual image (images x column blocks) from its position row t0 on, then whole ones
    const int g0 = (int)p.div_wc.div((uint32_t)j0), v0 = (int)p.div_hb.div((uint32_t)g0), t0 = g0 - v0 * p.Hb;
    const int len = p.fh * p.Hb + p.U - p.fh, len0 = len - p.fh * t0;
    uint32_t b_off[NB];
#pragma unroll
    for (int x = 0; x < NB; ++x) {
        const int e = tid + 512 * x;
        uint32_t lr, at, rem, lc;
        p.div_pitch.divmod((uint32_t)e, lr, at);
        p.div_span.divmod(at, rem, lc);
        lc = lc * p.fw + rem;
        int v = v0, row = p.fh * t0 + (int)lr;
        if ((int)lr >= len0) {
            const int k = ((int)lr - len0) / len;
            v = v0 + 1 + k;
            row = (int)lr - len0 - k * len;
        }
        row += p.fh - p.U;
        uint32_t n, cb;
        p.div_nb.divmod((uint32_t)v, n, cb);
        const int col = p.fw * (int)cb * p.Wc + (int)lc + p.fw - p.V;
        const bool ok = e < p.cells && v < p.images && (unsigned)row < (unsigned)p.P && (unsigned)col < (unsigned)p.Q;
        b_off[x] = ok ? (uint32_t)EB * (uint32_t)(((int)n * p.K * p.P + row) * p.Q + col) : kOob;
    }
    // the filter: a thread takes eight channels of a tap and row
    uint32_t a_off[NA];
    auto place_a = [&](int g) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NA; ++x) {
            const int e = tid + 512 * x, m = e & 31, tap = 2 * (g * p.pairs + (e >> 6)) + (e >> 5 & 1);
            uint32_t u, v, c, a, ah, aw;
            p.div_v.divmod((uint32_t)tap, u, v);
            p.div_block.divmod((uint32_t)m, c, a);
            p.div_vsw.divmod(a, ah, aw);
            const int r = (int)ah + p.sh * ((int)u - p.fh + 1), s = (int)aw + p.sw * ((int)v - p.fw + 1);
            const bool ok = (int)c < p.C && tap < p.taps && (unsigned)r < (unsigned)p.R && (unsigned)s < (unsigned)p.S;
            a_off[x] = ok ? (uint32_t)EB * (uint32_t)(((int)c * p.R + r) * p.S + s) : kOob;
        }
    };
    place_a(0);
    // this lane's positions: the cell of the last tap
    int col_cell[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int j = min(j0 + wn0 + 32 * i + l32, p.cols - 1);
        uint32_t g, u, v, t;
        p.div_wc.divmod((uint32_t)j, g, u);
        p.div_hb.divmod(g, v, t);
        const int row = (int)v == v0 ? p.fh * ((int)t - t0) : len0 + ((int)v - v0 - 1) * len + p.fh * (int)t;
        col_cell[i] = (row * p.pitch + (int)u) * 16;
    }

    f32x16 acc[2], low[2];
    uint32_t rest = 0;
    const int chunks = (p.K + kFewC - 1) / kFewC, steps = chunks * p.groups;
    const uint32_t in_plane = (uint32_t)EB * (uint32_t)(p.P * p.Q);

    auto pass = [&](auto fp32c) __attribute__((always_inline)) {
        constexpr bool FP32 = fp32c;   // operands as they are, on the fp32 instructions: cells of eight floats
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) { acc[j][e] = 0.f; low[j][e] = 0.f; }
        float ra[NA][8], rb[NB][8];
        auto load_a = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < NA; ++x)
#pragma unroll
                for (int i = 0; i < 8; ++i)   // channels past the last one lie behind the filter and read as zero
                    ra[x][i] = Elem<E>::load(rw, a_off[x], (uint32_t)EB * (uint32_t)((kFewC * c + i) * p.CRS));
        };
        auto load_b = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                if (512 * x >= p.cells) break;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    uint32_t vo = b_off[x];
                    if (kFewC * (c + 1) > p.K) vo = kFewC * c + i < p.K ? vo : kOob;   // channels past the last one are the next image's
                    rb[x][i] = Elem<E>::load(rin, vo, (uint32_t)(kFewC * c + i) * in_plane);
                }
            }
        };
        auto put = [&](char *dst, int part, const float (&v)[8]) __attribute__((always_inline)) {
            if constexpr (FP32) {   // two rows of 16 bytes in the first two parts' places
                const f32x4 x = {v[0], v[1], v[2], v[3]}, y = {v[4], v[5], v[6], v[7]};
                *reinterpret_cast<f32x4 *>(dst) = x;
                *reinterpret_cast<f32x4 *>(dst + part) = y;
            } else if constexpr (F32) {
                u32x4 c[3];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t h, m, l;
                    split_pair(v[2 * i], v[2 * i + 1], h, m, l, rest);
                    c[0][i] = h; c[1][i] = m; c[2][i] = l;
                }
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4 *>(dst + pl * part) = c[pl];
            } else {
                u32x4 c;
#pragma unroll
                for (int i = 0; i < 4; ++i)   // widened bf16: the high halves
                    c[i] = __builtin_amdgcn_perm(__float_as_uint(v[2 * i + 1]), __float_as_uint(v[2 * i]), 0x07060302u);
                *reinterpret_cast<u32x4 *>(dst) = c;
            }
        };
        auto put_a = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < NA; ++x) {
                const int e = tid + 512 * x;
                if (e < p.pairs * 64) put(lds + buf * a_buf + e * 16, a_part, ra[x]);
            }
        };
        auto put_b = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                const int e = tid + 512 * x;
                if (e < p.cells) put(lds_b + buf * b_buf + e * 16, b_part, rb[x]);
            }
        };
        // the step whose filter cells are loaded next
        int lc = 0, lg = 0;
        auto next_a = [&]() __attribute__((always_inline)) {
            if (p.groups > 1) place_a(lg);
            load_a(lc);
            if (++lg == p.groups) { lg = 0; ++lc; }
        };
        next_a();
        load_b(0);
        put_a(0);
        put_b(0);
        next_a();
        if (chunks > 1) load_b(1);
        __syncthreads();

        const bool early = wave < 4;   // the two waves of a SIMD stage at different ends of a step
        int c = 0, g = 0;
        for (int s = 0; s < steps; ++s) {
            const bool last = g == p.groups - 1;
            auto stage = [&]() __attribute__((always_inline)) {
                if (s + 1 >= steps) return;
                put_a((s + 1) & 1);
                next_a();
                if (last) {
                    put_b((c + 1) & 1);
                    if (c + 2 < chunks) load_b(c + 2);
                }
            };
            if (early) stage();
            const char *pa = lds + (s & 1) * a_buf + lane * 16, *pb = lds_b + (c & 1) * b_buf;
            const int *pt = tab + 2 * g * p.pairs + lhi;
            for (int i = wr; i < p.pairs; i += 2) {
                const int off = pt[2 * i];
                u32x4 va[PARTS], vb[PARTS][2];
#pragma unroll
                for (int pl = 0; pl < (FP32 ? 2 : PARTS); ++pl) {
                    va[pl] = *reinterpret_cast<const u32x4 *>(pa + i * 1024 + pl * a_part);
#pragma unroll
                    for (int j = 0; j < 2; ++j) vb[pl][j] = *reinterpret_cast<const u32x4 *>(pb + col_cell[j] + off + pl * b_part);
                }
                if constexpr (FP32) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(va[e >> 2][e & 3]), __uint_as_float(vb[e >> 2][j][e & 3]),
                                                                          acc[j], 0, 0, 0);
                } else {
                    constexpr int PL_A[6] = {0, 2, 1, 1, 0, 0}, PL_B[6] = {0, 0, 1, 0, 1, 2};
#pragma unroll
                    for (int m = 0; m < (F32 ? 6 : 1); ++m)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            f32x16 &d = m == 0 ? acc[j] : low[j];
                            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[PL_A[m]]),
                                                                        __builtin_bit_cast(bf16x8, vb[PL_B[m]][j]), d, 0, 0, 0);
                        }
                }
            }
            if (!early) stage();
            if (last) { g = 0; ++c; } else ++g;
            __syncthreads();
        }
    };
    pass(std::false_type{});

    if constexpr (F32) {
        // not finite, or below 2^-104 and not zero (see conv_halo.hpp)
        float not_finite = 0.f;
        uint32_t least = 0xFFFFFFFFu;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float v = acc[j][e] + low[j][e];
                acc[j][e] = v;
                not_finite = fmaf(v, 0.f, not_finite);
                least = min(least, (__float_as_uint(v) << 1) - 1u);
            }
        const bool redo = (rest & 0xFFFFu) != 0 || !(not_finite == 0.f) || least < ((127u - 104u) << 24) - 1u;
        if (__syncthreads_or(redo)) pass(std::true_type{});
    }

    // the waves of a pair give each other one of the two tiles
    float *give = reinterpret_cast<float *>(lds) + wave * 1024 + lane, *take = reinterpret_cast<float *>(lds) + (wave ^ 4) * 1024 + lane;
#pragma unroll
    for (int e = 0; e < 16; ++e) give[64 * e] = wr ? acc[0][e] : acc[1][e];
    __syncthreads();
    float y[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = (wr ? acc[1][e] : acc[0][e]) + take[64 * e];

    const int jo = j0 + wn0 + 32 * wr + l32;
    if (jo >= p.cols) return;
    uint32_t gr, uw, v, t, n, cb;
    p.div_wc.divmod((uint32_t)jo, gr, uw);
    p.div_hb.divmod(gr, v, t);
    p.div_nb.divmod(v, n, cb);
    const int h0 = p.vsh * (int)t - p.ph, w0 = p.vsw * ((int)cb * p.Wc + (int)uw) - p.pw;
    // a position behind the last one of its row belongs to the next block or to none
    if ((int)(cb * p.Wc + uw) * p.vsw >= p.W + p.pw) return;
    // A tap that is not there is a zero in the products above, and one with an infinity is no zero: sums that are not finite are taken
    // again, tap by tap
    bool finite = true;
#pragma unroll
    for (int e = 0; e < 16; ++e) finite &= fabsf(y[e]) < __builtin_inff();
    if (!finite)
#pragma unroll 1
        for (int e = 0; e < 16; ++e) {
            uint32_t c, a, ah, aw;
            p.div_block.divmod((uint32_t)(8 * (e >> 2) + 4 * lhi + (e & 3)), c, a);
            p.div_vsw.divmod(a, ah, aw);
            const int h = h0 + (int)ah + p.ph, w = w0 + (int)aw + p.pw;   // of the padded image
            if ((int)c >= p.C) break;
            float sum = 0.f;
            for (int r = h % p.sh; r < p.R; r += p.sh) {
                if (h < r || (h - r) / p.sh >= p.P) continue;
                for (int s = w % p.sw; s < p.S; s += p.sw) {
                    if (w < s || (w - s) / p.sw >= p.Q) continue;
                    const uint32_t at = (uint32_t)EB * (uint32_t)(((int)n * p.K * p.P + (h - r) / p.sh) * p.Q + (w - s) / p.sw);
                    const uint32_t tap = (uint32_t)EB * (uint32_t)(((int)c * p.R + r) * p.S + s);
                    for (int k = 0; k < p.K; ++k)
                        sum = fmaf(Elem<E>::load(rin, at, (uint32_t)k * in_plane), Elem<E>::load(rw, tap, (uint32_t)EB * (uint32_t)(k * p.CRS)), sum);
                }
            }
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (i == e && !(fabsf(y[i]) < __builtin_inff())) y[i] = sum;
        }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = 8 * q + 4 * lhi;
        if (F32 && p.vsw % 4 == 0) {   // four adjacent pixels
            uint32_t c, a, ah, aw;
            p.div_block.divmod((uint32_t)m, c, a);
            p.div_vsw.divmod(a, ah, aw);
            const int h = h0 + (int)ah, w = w0 + (int)aw;
            if ((int)c >= p.C || (unsigned)h >= (unsigned)p.H) continue;
            const uint32_t off = 4u * (uint32_t)((((int)n * p.C + (int)c) * p.H + h) * p.W + w);
            if (w >= 0 && w + 3 < p.W) {
                const u32x4 d = {__float_as_uint(y[4 * q]), __float_as_uint(y[4 * q + 1]), __float_as_uint(y[4 * q + 2]), __float_as_uint(y[4 * q + 3])};
                __builtin_amdgcn_raw_buffer_store_b128(d, rout, (int)off, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if ((unsigned)(w + e) < (unsigned)p.W) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[4 * q + e]), rout, (int)(off + 4u * e), 0, 0);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t c, a, ah, aw;
                p.div_block.divmod((uint32_t)(m + e), c, a);
                p.div_vsw.divmod(a, ah, aw);
                const int h = h0 + (int)ah, w = w0 + (int)aw;
                if ((int)c < p.C && (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W)
                    Elem<E>::store(p.out, (((long)n * p.C + c) * p.H + h) * p.W + w, y[4 * q + e]);
            }
        }
    }
}

}  // namespace ucd
