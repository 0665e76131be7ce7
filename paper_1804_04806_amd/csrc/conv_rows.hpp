// Forward of layers with few input channels (a network's first layer) over windows of image rows in LDS, on the bf16 matrix pipe; fp32
// tensors as split operands (products, error and range as in gemm_split.hpp), bf16 tensors as they are.
//
// The reduction runs along the rows of the filter: in quads of four adjacent taps, S rounded up, which meet four adjacent pixels.  So the
// window lies in LDS as the image's rows do, every element split and written once, and an operand (eight products of a position) is two
// reads of eight bytes wherever the stride puts them: columns begin on whole words where the stride is even; where it is odd a third word is read
// and the lanes of odd columns shift.  An odd padding is made even by a tap of zeros in front.
//
// A workgroup of eight waves, one per CU, owns MT output channels: it splits their filter once and keeps it in LDS, and goes over tiles of NT
// positions (which run over images, blocks of Wc columns, rows, columns of the block).  Of these it keeps one window with all channels; the
// next one's pixels are on their way to registers while it multiplies, and are split into its place between two barriers.
//
// 3 -> 64 7x7/2 224x224 b = 128: 357 us as tile GEMMs on the fp32 instructions, 223 with this (bf16 170, 107); 42 % of the matrix pipe's cycles are MFMAs.  Its
// memory alone (411 of 488 MB are stores) would take 93 at a copy's rate, its MFMAs, 16 % on zeros, 97.  What is left is that a CU's
// eight waves multiply, split and store together: sums stored while the next tile is multiplied (284 to 249 us against storing
// them at the tile's end, 246 and 258 with twice and four times the stores per step), narrow blocks of columns (249 to 237).  Two
// workgroups of four waves per CU, which stage the filter with every tile, took 285.
#pragma once
#include "gemm_split.hpp"

namespace ucd {

constexpr int kRowsQuads = 128;   // quads of a filter, at most
constexpr int kRowsMost = 256;    // rows of a window, all channels
constexpr int kRowsLds = 163840 - 512 - 4 * kRowsQuads - 8 * kRowsMost;

struct RowsParams {
    const void *in, *w;
    void *out;
    uint32_t in_bytes, w_bytes, out_bytes;
    int C, H, W, K, P, Q, R, S, CRS, sh, sw, ph, pw;
    int delta, SQ, quads, steps;                     // zero taps in front, quads per filter row, of the filter, steps of four quads
    int Wc, nb, pitch, rows, pairs, b_part;          // columns per block, blocks; elements per window row, rows per channel, pairs of elements, bytes per part
    int images, cols, tiles_m, tiles_n;              // images * blocks, positions, tiles
    FastDiv div_wc, div_p, div_nb, div_half, div_rows, div_sq, div_r, div_len;   // div_half: pitch / 2; div_len: rows of a whole virtual image
};

// Eight waves side by side, each with WM tiles of 32 x 32.
template <class E_, int WM_>
struct RowsTile {
    typedef E_ E;
    static constexpr bool F32 = std::is_same<E, float>::value;
    static constexpr int WM = WM_, MT = 32 * WM, NT = 256, PARTS = F32 ? 3 : 1;
    static constexpr int A_PART = 2 * MT * 16, A_STEP = PARTS * A_PART;   // a step's two halves
    static constexpr int NB = 10;                                         // pairs of the window per thread
};

template <class T, bool ODD>
__global__ __launch_bounds__(512, 2) void conv_rows_kernel(RowsParams p)
{
    typedef typename T::E E;
    constexpr bool F32 = T::F32;
    constexpr int WM = T::WM, MT = T::MT, NT = T::NT, PARTS = T::PARTS, NB = T::NB, EB = (int)Elem<E>::kBytes;
    __shared__ __attribute__((aligned(16))) char lds[kRowsLds];
    __shared__ __attribute__((aligned(16))) int b_tab[kRowsQuads], row_tab[2 * kRowsMost];
    __shared__ int again;   // bf16: a sum of the tile is not finite
    char *const win = lds + p.steps * T::A_STEP;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn0 = wave * 32;
    const uint32_t id = xcd_order(blockIdx.x, gridDim.x);
    const int m0 = (int)(id % (uint32_t)p.tiles_m) * MT, first = (int)(id / (uint32_t)p.tiles_m), stride = (int)(gridDim.x / (uint32_t)p.tiles_m);

    const __amdgpu_buffer_rsrc_t rin = make_rsrc_bytes(p.in, 0, p.in_bytes), rw = make_rsrc_bytes(p.w, 0, p.w_bytes),
                                 rout = make_rsrc_bytes(p.out, 0, p.out_bytes);
    const int len = p.sh * (p.P - 1) + p.R;   // window rows of a whole virtual image

    // where the quads of the filter lie in the window (elements)
    if (tid < kRowsQuads) {
        uint32_t cr, sq, cc, r;
        p.div_sq.divmod((uint32_t)tid, cr, sq);
        p.div_r.divmod(cr, cc, r);
        b_tab[tid] = tid < p.quads ? ((int)cc * p.rows + (int)r) * p.pitch + 4 * (int)sq : 0;
    }

    uint32_t rest;
    // eight values into the three (one) parts' cells, or as they are into two of them
    auto put_cell = [&](auto fp32c, char *dst, const float (&v)[8]) __attribute__((always_inline)) {
        constexpr bool FP32 = fp32c;
        if constexpr (FP32) {
            *reinterpret_cast<f32x4 *>(dst) = f32x4{v[0], v[1], v[2], v[3]};
            *reinterpret_cast<f32x4 *>(dst + T::A_PART) = f32x4{v[4], v[5], v[6], v[7]};
        } else if constexpr (F32) {
            u32x4 c[3];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t h, m, l;
                split_pair(v[2 * i], v[2 * i + 1], h, m, l, rest);
                c[0][i] = h; c[1][i] = m; c[2][i] = l;
            }
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4 *>(dst + pl * T::A_PART) = c[pl];
        } else {
            u32x4 c;
#pragma unroll
            for (int i = 0; i < 4; ++i) c[i] = __builtin_amdgcn_perm(__float_as_uint(v[2 * i + 1]), __float_as_uint(v[2 * i]), 0x07060302u);
            *reinterpret_cast<u32x4 *>(dst) = c;
        }
    };
    // the filter's cells, two quads each; taps that do not exist are zeros
    auto put_filter = [&](auto fp32c) __attribute__((always_inline)) {
#pragma unroll 1
        for (int e = tid; e < p.steps * 2 * MT; e += 512) {
            const int row = e % MT, pair = e / MT;
            float v[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t cr, sq;
                p.div_sq.divmod((uint32_t)(2 * pair + h), cr, sq);
                const int s = 4 * (int)sq - p.delta;
                const bool ok = 2 * pair + h < p.quads && m0 + row < p.K;
                const uint32_t at = (uint32_t)EB * (uint32_t)((m0 + row) * p.CRS + (int)cr * p.S + s);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[4 * h + i] = Elem<E>::load(rw, ok && (unsigned)(s + i) < (unsigned)p.S ? at + (uint32_t)EB * i : kOob, 0u);
            }
            put_cell(fp32c, lds + (pair >> 1) * T::A_STEP + ((pair & 1) * MT + row) * 16, v);
        }
    };
    // where the rows of tile n's window begin in the tensor, less their first column, and that column: rows of the first virtual
    // image (images x column blocks) from the tile's first position on, then whole ones
    auto put_rows = [&](int n) __attribute__((always_inline)) {
        if (tid >= kRowsMost) return;
        const int g0 = (int)p.div_wc.div((uint32_t)(n * NT)), v0 = (int)p.div_p.div((uint32_t)g0), t0 = g0 - v0 * p.P, len0 = len - p.sh * t0;
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
        const bool ok = n < p.tiles_n && (int)cc < p.C && v < p.images && (unsigned)row < (unsigned)p.H;
        row_tab[2 * tid] = ok ? (((int)img * p.C + (int)cc) * p.H + row) * p.W : 0;
        row_tab[2 * tid + 1] = ok ? (int)cb * p.Wc * p.sw - p.pw - p.delta : -(1 << 30);
    };
    const bool whole = p.W % 2 == 0;   // no pair of pixels ends behind its row
    auto load_b = [&](uint32_t (&rb)[NB][2]) __attribute__((always_inline)) {   // as they lie in memory
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            if (512 * x >= p.pairs) break;
            int e = tid + 512 * x;
            asm volatile("" : "+v"(e));   // not before the break, nor kept
            uint32_t cr, half;
            p.div_half.divmod((uint32_t)min(e, p.pairs - 1), cr, half);
            const int at = row_tab[2 * cr], col = row_tab[2 * cr + 1] + 2 * (int)half;
            const uint32_t off = (unsigned)col < (unsigned)p.W ? (uint32_t)EB * (uint32_t)(at + col) : kOob;
            if (F32 && whole) {
                const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rin, (int)off, 0, 0));
                rb[x][0] = v[0];
                rb[x][1] = v[1];
            } else {
                const int next = (int)(col + 1 < p.W ? off + EB : kOob);
                if constexpr (F32) {
                    rb[x][0] = __builtin_amdgcn_raw_buffer_load_b32(rin, (int)off, 0, 0);
                    rb[x][1] = __builtin_amdgcn_raw_buffer_load_b32(rin, next, 0, 0);
                } else {
                    rb[x][0] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rin, (int)off, 0, 0);
                    rb[x][1] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rin, next, 0, 0);
                }
            }
        }
    };
    auto put_b = [&](auto fp32c, const uint32_t (&rb)[NB][2]) __attribute__((always_inline)) {
        constexpr bool FP32 = fp32c;
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            if (512 * x >= p.pairs) break;
            const int e = tid + 512 * x;
            if (e >= p.pairs) break;
            if constexpr (FP32) {
                *reinterpret_cast<u32x2 *>(win + 8 * e) = u32x2{rb[x][0], rb[x][1]};
            } else if constexpr (F32) {
                uint32_t h, m, l;
                split_pair(__uint_as_float(rb[x][0]), __uint_as_float(rb[x][1]), h, m, l, rest);
                *reinterpret_cast<uint32_t *>(win + 4 * e) = h;
                *reinterpret_cast<uint32_t *>(win + p.b_part + 4 * e) = m;
                *reinterpret_cast<uint32_t *>(win + 2 * p.b_part + 4 * e) = l;
            } else {
                *reinterpret_cast<uint32_t *>(win + 4 * e) = __builtin_amdgcn_perm(rb[x][1], rb[x][0], 0x05040100u);
            }
        }
    };

    rest = 0;
    if (!F32) again = 0;
    put_filter(std::false_type{});
    put_rows(first);
    const bool plain = F32 && __syncthreads_or((rest & 0xFFFFu) != 0);   // a filter that the parts do not hold
    if (plain) put_filter(std::true_type{});
    if (!F32) __syncthreads();
    uint32_t rb[NB][2];
    load_b(rb);
    __syncthreads();   // row_tab is written again
    rest = 0;
    put_b(std::false_type{}, rb);
    put_rows(first + stride);
    __syncthreads();
    load_b(rb);

    // sums that are stored while the next tile is multiplied, and where
    float done[WM][16];
    uint32_t done_at = kOob;
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) done[i][e] = 0.f;
    const uint32_t plane = (uint32_t)EB * (uint32_t)(p.P * p.Q);
    const int rows_left = p.K - m0 - 4 * lhi;
    auto store = [&](int i, int e) __attribute__((always_inline)) {
        const int row = 32 * i + 8 * (e >> 2) + (e & 3);
        const uint32_t off = row < rows_left ? done_at : kOob, so = (uint32_t)row * plane;
        if constexpr (F32) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(done[i][e]), rout, (int)off, (int)so, 0);
        else __builtin_amdgcn_raw_buffer_store_b16((short)Elem<bf16>::round(done[i][e]), rout, (int)off, (int)so, 0);
    };

    for (int n = first; n < p.tiles_n; n += stride) {
        // this lane's position: where its first tap lies in the window
        uint32_t g, u, v, t, img, cb;
        const int jo = n * NT + wn0 + l32;
        p.div_wc.divmod((uint32_t)min(jo, p.cols - 1), g, u);
        p.div_p.divmod(g, v, t);
        p.div_nb.divmod(v, img, cb);
        int cell;
        {
            const int g0 = (int)p.div_wc.div((uint32_t)(n * NT)), v0 = (int)p.div_p.div((uint32_t)g0), t0 = g0 - v0 * p.P, len0 = len - p.sh * t0;
            const int row = (int)v == v0 ? p.sh * ((int)t - t0) : len0 + ((int)v - v0 - 1) * len + p.sh * (int)t;
            cell = row * p.pitch + (int)u * p.sw;
        }
        const uint32_t shift = ODD ? 16u * (cell & 1) : 0u;
        const int q = (int)cb * p.Wc + (int)u;
        f32x16 acc[WM], low[WM];
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) { acc[i][e] = 0.f; low[i][e] = 0.f; }
        const char *const pa = lds + (lhi * MT + l32) * 16;
        // which of a quad's four taps there are
        auto taps_of = [&](int quad) __attribute__((always_inline)) {
            uint32_t cr, sq, there = 0;
            p.div_sq.divmod((uint32_t)quad, cr, sq);
#pragma unroll
            for (int e = 0; e < 4; ++e) there |= quad < p.quads && (unsigned)(4 * (int)sq - p.delta + e) < (unsigned)p.S ? 1u << e : 0u;
            return there;
        };
        auto step = [&](auto exact, int s) __attribute__((always_inline)) {
            constexpr bool EXACT = exact;   // pixels under taps that are not there, which meet a zero, are zeros too
            const int o0 = b_tab[4 * s + 2 * lhi], o1 = b_tab[4 * s + 2 * lhi + 1];
            u32x4 va[WM][PARTS], vb[PARTS];
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int pl = 0; pl < PARTS; ++pl) va[i][pl] = *reinterpret_cast<const u32x4 *>(pa + s * T::A_STEP + i * 512 + pl * T::A_PART);
#pragma unroll
            for (int pl = 0; pl < PARTS; ++pl)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t *src = reinterpret_cast<const uint32_t *>(win + pl * p.b_part) + ((cell >> 1) + ((h ? o1 : o0) >> 1));
                    uint32_t d0 = src[0], d1 = src[1];
                    if (ODD) {
                        const uint32_t d2 = src[2];
                        d0 = __builtin_amdgcn_alignbit(d1, d0, shift);
                        d1 = __builtin_amdgcn_alignbit(d2, d1, shift);
                    }
                    if constexpr (EXACT) {
                        const uint32_t there = taps_of(4 * s + 2 * lhi + h);
                        d0 &= (there & 1 ? 0xFFFFu : 0u) | (there & 2 ? 0xFFFF0000u : 0u);
                        d1 &= (there & 4 ? 0xFFFFu : 0u) | (there & 8 ? 0xFFFF0000u : 0u);
                    }
                    vb[pl][2 * h] = d0;
                    vb[pl][2 * h + 1] = d1;
                }
            constexpr int PL_A[6] = {0, 2, 1, 1, 0, 0}, PL_B[6] = {0, 0, 1, 0, 1, 2};
#pragma unroll
            for (int m = 0; m < (F32 ? 6 : 1); ++m)
#pragma unroll
                for (int i = 0; i < WM; ++i) {
                    f32x16 &d = m == 0 ? acc[i] : low[i];
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[i][PL_A[m]]), __builtin_bit_cast(bf16x8, vb[PL_B[m]]), d, 0, 0, 0);
                }
        };
#pragma unroll
        for (int s = 0; s < 4 * WM; ++s) {
            if (s < p.steps) step(std::false_type{}, s);
#pragma unroll
            for (int e = 0; e < 4; ++e) store(s >> 2, 4 * (s & 3) + e);
        }
#pragma unroll 1
        for (int s = 4 * WM; s < p.steps; ++s) step(std::false_type{}, s);
        if constexpr (F32) {
            // not finite, or below 2^-104 and not zero (see conv_halo.hpp)
            float not_finite = 0.f;
            uint32_t least = 0xFFFFFFFFu;
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float y = acc[i][e] + low[i][e];
                    acc[i][e] = y;
                    not_finite = fmaf(y, 0.f, not_finite);
                    least = min(least, (__float_as_uint(y) << 1) - 1u);
                }
            const bool redo = __syncthreads_or(plain || (rest & 0xFFFFu) != 0 || !(not_finite == 0.f) || least < ((127u - 104u) << 24) - 1u);
            if (redo) {   // the tile once more, on the fp32 instructions, operands as they are
                uint32_t once_more[NB][2];
                if (!plain) put_filter(std::true_type{});
                put_rows(n);
                __syncthreads();
                load_b(once_more);
                put_b(std::true_type{}, once_more);
                __syncthreads();
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
#pragma unroll 1
                for (int s = 0; s < p.steps; ++s) {
                    const int o0 = b_tab[4 * s + 2 * lhi], o1 = b_tab[4 * s + 2 * lhi + 1];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t there = taps_of(4 * s + 2 * lhi + h);
                        f32x4 va[WM];
#pragma unroll
                        for (int i = 0; i < WM; ++i) va[i] = *reinterpret_cast<const f32x4 *>(pa + s * T::A_STEP + i * 512 + h * T::A_PART);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float b = *reinterpret_cast<const float *>(win + 4 * (cell + (h ? o1 : o0) + e));
                            b = there >> e & 1 ? b : 0.f;
#pragma unroll
                            for (int i = 0; i < WM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i][e], b, acc[i], 0, 0, 0);
                        }
                    }
                }
                __syncthreads();
                if (!plain) put_filter(std::false_type{});
            }
        } else {
            float sums[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) sums[e & 3] = fmaf(acc[i][e], 0.f, sums[e & 3]);
            if (!(sums[0] + sums[1] + (sums[2] + sums[3]) == 0.f)) again = 1;
            __syncthreads();
            if (again) {   // the tile once more
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
#pragma unroll 1
                for (int s = 0; s < p.steps; ++s) step(std::true_type{}, s);
                __syncthreads();
                again = 0;
            }
        }
        rest = 0;
        if (n + stride < p.tiles_n) put_b(std::false_type{}, rb);
        put_rows(n + 2 * stride);
        __syncthreads();
        load_b(rb);

        const bool in = jo < p.cols && q < p.Q;
        done_at = in ? (uint32_t)EB * (uint32_t)((((int)img * p.K + m0 + 4 * lhi) * p.P + (int)t) * p.Q + q) : kOob;
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) done[i][e] = acc[i][e];
    }
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) store(i, e);
}

}  // namespace ucd
