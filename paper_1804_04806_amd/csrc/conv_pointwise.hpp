// 1x1 stride-1 convolutions with more output than input channels, fp32 tensors on the bf16 matrix pipe (gfx950); products,
// error and range as in gemm_split.hpp.
//
// A tile GEMM of such a layer has few reduction steps, so that a tile's start and end cost as much as its steps, and
// loads and splits the activations once per tile row.  Here a workgroup keeps all input channels of its NT pixels
// in LDS as MFMA operands, split once, and walks over the output channels: the filter streams through two LDS
// buffers without a break from one tile row to the next, and a row's results are stored while the next one is multiplied.
// Workgroups of the last, partly filled round take only a range of the tile rows.
#pragma once
#include "gemm_split.hpp"

namespace ucd {

struct PointwiseParams {
    const void *x, *w;
    void *y;
    uint32_t x_bytes, w_bytes, y_bytes;
    int K, M, px, cols;          // reduction (input) channels, output channels, pixels of an image, pixels of the micro-batch
    int w_row, w_k;              // element (m, k) of the filter: w[m * w_row + k * w_k]
    int m_tiles, whole, splits;  // tile rows; pixel tiles that take them all; workgroups per later tile
    FastDiv div_px;
};

// Eight waves, 2 x 4, multiply and store, 64 output channels x 32 pixels each.  Four more load and split the filter: loads and
// stores of a wave are counted together and in order, so one that waits for filter cells would wait for the results it
// stored before them (128 -> 512 channels 28x28 b = 128: 103 us with eight waves doing both, 94 so; two workgroups of half
// the pixels per CU 106, the tile GEMM 131).
struct PointwiseTile {
    static constexpr int WM = 2, WN = 1, MT = 128, NT = 128, THREADS = 768;
    static constexpr int LDS = 162816;
    static constexpr int A_HALF = (MT + 4) * 16, A_PART = 2 * A_HALF, A_BUF = 3 * A_PART;
    static constexpr int B_HALF = (NT + 4) * 16, B_PART = 2 * B_HALF, B_STEP = 3 * B_PART;
    static constexpr int kMaxK = (LDS - 2 * A_BUF) / (2 * B_STEP) * 32;
};

// A wave's tile on the fp32 instructions, operands straight from memory: `row` is the lane's filter row, load_b(k, b) its
// pixels' values of input channel k (zero behind the last one).  Eight channels at a time, of which lanes 0-31 hold the first
// four, in two sets of registers, so that the loads of one have the time of the other's products.  A launch of which
// everything is computed again takes 1.6 to 2.7 times as long (160 -> 1024 channels 14x14 b = 168: 75 / 190 us; with two
// channels at a time, one after another, 380).
template <bool ROWS, int WM, int WN, class LoadB>
__device__ __forceinline__ void pointwise_fp32(const PointwiseParams &p, __amdgpu_buffer_rsrc_t rw, int row, int lhi, LoadB load_b,
                                               f32x16 (&acc)[WM][WN])
{
    constexpr int kAhead = 2;
    asm volatile("" : "+v"(row), "+v"(lhi));   // addresses are computed here, not ahead of the caller's loops
    struct Set { float a[WM][4], b[4][WN]; } set[kAhead];
    auto load = [&](int k0, Set &s) __attribute__((always_inline)) {
        const int k = k0 + 4 * lhi;
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const int r = row + 32 * i;
            const uint32_t vo = r < p.M && k < p.K ? 4u * (uint32_t)(r * p.w_row + k * p.w_k) : kOob;
            if constexpr (ROWS) {
                const f32x4 v = buf_load4(rw, vo);
                s.a[i][0] = v.x; s.a[i][1] = v.y; s.a[i][2] = v.z; s.a[i][3] = v.w;
            } else {   // channels past the last one lie behind the filter
#pragma unroll
                for (int e = 0; e < 4; ++e) s.a[i][e] = Elem<float>::load(rw, vo, 4u * (uint32_t)(e * p.w_k));
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) load_b(k + e, s.b[e]);
    };
    auto multiply = [&](int k0, Set &s) __attribute__((always_inline)) {
        if (ROWS && k0 + 8 > p.K) {   // what follows a row's last channel is the next one's first
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) s.a[i][e] = k0 + 4 * lhi + e < p.K ? s.a[i][e] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(s.a[i][e], s.b[e][j], acc[i][j], 0, 0, 0);
    };
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) load(8 * i, set[i]);
#pragma unroll 1
    for (int k0 = 0; k0 < p.K; k0 += 8 * kAhead) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            multiply(k0 + 8 * i, set[i]);
            load(k0 + 8 * (i + kAhead), set[i]);
        }
    }
}

// ROWS: the filter is contiguous along the reduction (Forward); otherwise along the output channels (BackwardData).
// VEC: images of a multiple of four pixels
template <bool ROWS, bool VEC>
__global__ __launch_bounds__(PointwiseTile::THREADS, 3) void pointwise_kernel(PointwiseParams p)
{
    typedef PointwiseTile T;
    constexpr int WM = T::WM, WN = T::WN, MT = T::MT, NT = T::NT;
    __shared__ __attribute__((aligned(16))) char lds[T::LDS];
    // Some operand was not split exactly: an input element, or a filter element of tile row mt, which leaves mt + 1 in the
    // word of its parity.  The multiplying waves look behind a row's last barrier, where the producers are at the next
    // row's cells already; they come to the row after that, which has the same word again, behind another barrier.
    __shared__ uint32_t inexact_x, inexact_w[2];
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
    const int j0 = tile * NT, steps = (p.K + 31) / 32 * 2;   // an even number: the producers' two sets of registers take turns
    const __amdgpu_buffer_rsrc_t rx = make_rsrc_bytes(p.x, 0, p.x_bytes), rw = make_rsrc_bytes(p.w, 0, p.w_bytes),
                                 ry = make_rsrc_bytes(p.y, 0, p.y_bytes);
    const uint32_t plane = 4u * (uint32_t)p.px;
    uint32_t rest = 0;

    auto split_cell = [&](char *dst, int part, const float (&v)[8]) __attribute__((always_inline)) {
        u32x4 c[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t h, m, l;
            split_pair(v[2 * i], v[2 * i + 1], h, m, l, rest);
            c[0][i] = h; c[1][i] = m; c[2][i] = l;
        }
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4 *>(dst + pl * part) = c[pl];
    };

    // the producers' filter cells.  A tile row's and a step's parts of the address are scalar; rows past the last one lie
    // behind the filter or, along the output channels, read what is not stored.
    const bool producer = wave >= 8;
    const int cell = tid & 255, a_hi = ROWS ? cell & 1 : cell >> 7, a_row = ROWS ? cell >> 1 : cell & 127;
    const uint32_t a_off = 4u * (uint32_t)(a_row * p.w_row + 8 * a_hi * p.w_k);
    auto load_a = [&](int mt, int st, float (&ra)[8]) __attribute__((always_inline)) {
        const uint32_t so = 4u * (uint32_t)(mt * MT * p.w_row + 16 * st * p.w_k);
        if constexpr (ROWS) {
            const f32x4 u = buf_load4(rw, a_off, so), v = buf_load4(rw, a_off + 16u, so);
            ra[0] = u.x; ra[1] = u.y; ra[2] = u.z; ra[3] = u.w;
            ra[4] = v.x; ra[5] = v.y; ra[6] = v.z; ra[7] = v.w;
        } else {   // channels past the last one lie behind the filter
#pragma unroll
            for (int i = 0; i < 8; ++i) ra[i] = Elem<float>::load(rw, a_off, so + 4u * (uint32_t)(i * p.w_k));
        }
    };
    auto put_a = [&](int mt, int st, float (&ra)[8]) __attribute__((always_inline)) {
        rest = 0;
        if (ROWS && 16 * st + 16 > p.K) {   // what follows a row's last channel is the next one's first
#pragma unroll
            for (int i = 0; i < 8; ++i) ra[i] = 16 * st + 8 * a_hi + i < p.K ? ra[i] : 0.f;
        }
        split_cell(lds + (st & 1) * T::A_BUF + a_hi * T::A_HALF + a_row * 16, T::A_PART, ra);
        if ((rest & 0xFFFFu) != 0) inexact_w[mt & 1] = (uint32_t)mt + 1u;
    };

    float ra0[8], ra1[8];
    int lm = mt_begin, ls = 0;   // the step whose filter cells are loaded next
    auto next = [&]() __attribute__((always_inline)) {
        if (++ls == steps) { ls = 0; ++lm; }
    };
    if (tid == 0) inexact_x = inexact_w[0] = inexact_w[1] = 0;
    if (producer) {
        load_a(lm, ls, ra0);
        next();
    }
    __syncthreads();
    // all channels of the tile's pixels: eight channels of one or four adjacent pixels per thread and turn
    constexpr int PX = VEC ? 4 : 1;
    for (int e = tid; e < steps * 2 * (NT / PX); e += T::THREADS) {
        const int q = e % (NT / PX), hi = e / (NT / PX) & 1, st = e / (2 * (NT / PX)), c = 16 * st + 8 * hi;
        uint32_t n, px;
        p.div_px.divmod((uint32_t)(j0 + PX * q), n, px);
        const uint32_t vo = j0 + PX * q < p.cols ? 4u * (uint32_t)(((int)n * p.K + c) * p.px + (int)px) : kOob;
        float v[PX][8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t o = c + i < p.K ? vo : kOob;   // channels past the last one are the next image's
            if constexpr (VEC) {
                const f32x4 u = buf_load4(rx, o, (uint32_t)i * plane);
                v[0][i] = u.x; v[1][i] = u.y; v[2][i] = u.z; v[3][i] = u.w;
            } else {
                v[0][i] = Elem<float>::load(rx, o, (uint32_t)i * plane);
            }
        }
#pragma unroll
        for (int i = 0; i < PX; ++i) split_cell(lds_b + st * T::B_STEP + hi * T::B_HALF + (PX * q + i) * 16, T::B_PART, v[i]);
    }
    if ((rest & 0xFFFFu) != 0) inexact_x = 1;
    if (producer) {
        put_a(mt_begin, 0, ra0);
        load_a(lm, ls, ra1);
        next();
        load_a(lm, ls, ra0);
        next();
        __syncthreads();
        for (int mt = mt_begin; mt < mt_end; ++mt)
            for (int st = 0; st < steps; st += 2) {   // the cells of the step after each, loads of two steps in flight
                put_a(mt, st + 1, ra1);
                load_a(lm, ls, ra1);
                next();
                __syncthreads();
                const bool more = st + 2 < steps;
                put_a(more ? mt : mt + 1, more ? st + 2 : 0, ra0);
                load_a(lm, ls, ra0);
                next();
                __syncthreads();
            }
        return;
    }

    uint32_t out[WN];   // this lane's pixels in y, at its first row of tile row 0
#pragma unroll
    for (int j = 0; j < WN; ++j) {
        const int col = j0 + wn0 + 32 * j + l32;
        uint32_t n, px;
        p.div_px.divmod((uint32_t)col, n, px);
        out[j] = col < p.cols ? 4u * (uint32_t)(((int)n * p.M + wm0 + 4 * lhi) * p.px + (int)px) : kOob;
    }
    __syncthreads();

    u32x4 vn[3][WN];   // pixels' operands of the next step
    auto read_b = [&](int st) __attribute__((always_inline)) {
        const char *pb = lds_b + st * T::B_STEP + lhi * T::B_HALF + (wn0 + l32) * 16;
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll
            for (int j = 0; j < WN; ++j) vn[pl][j] = *reinterpret_cast<const u32x4 *>(pb + pl * T::B_PART + j * 512);
    };
    read_b(0);
    for (int mt = mt_begin; mt < mt_end; ++mt) {
        f32x16 acc[WM][WN], low[WM][WN];
        auto step = [&](int st, auto oddc, auto firstc) __attribute__((always_inline)) {
            constexpr bool FIRST = firstc;   // sums start from zero
            constexpr int odd = oddc;
            // the pixels' operands are read a step ahead, the filter's only behind the barrier
            const char *pa = lds + odd * T::A_BUF + lhi * T::A_HALF + (wm0 + l32) * 16;
            u32x4 va[3][WM], vb[3][WN];
#pragma unroll
            for (int pl = 2; pl >= 0; --pl)
#pragma unroll
                for (int i = 0; i < WM; ++i) va[pl][i] = *reinterpret_cast<const u32x4 *>(pa + pl * T::A_PART + i * 512);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int j = 0; j < WN; ++j) vb[pl][j] = vn[pl][j];
            __builtin_amdgcn_sched_barrier(0);
            constexpr int PL_A[6] = {2, 1, 1, 0, 0, 0}, PL_B[6] = {0, 1, 0, 0, 1, 2};
            auto group = [&](auto gc) __attribute__((always_inline)) {
                constexpr int g = gc;
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) {
                        constexpr f32x16 kZero = {};
                        f32x16 &d = g == 3 ? acc[i][j] : low[i][j];
                        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[PL_A[g]][i]),
                                                                    __builtin_bit_cast(bf16x8, vb[PL_B[g]][j]),
                                                                    FIRST && (g == 0 || g == 3) ? kZero : d, 0, 0, 0);
                    }
                if (g == 0) read_b(st + 1 < steps ? st + 1 : 0);
                __builtin_amdgcn_sched_barrier(0);
            };
            static_for<6>(group);
            __syncthreads();
        };
        typedef std::integral_constant<int, 0> Even;
        typedef std::integral_constant<int, 1> Odd;
        step(0, Even{}, std::true_type{});
        step(1, Odd{}, std::false_type{});
        for (int st = 2; st < steps; st += 2) {
            step(st, Even{}, std::false_type{});
            step(st + 1, Odd{}, std::false_type{});
        }
        // range check as in conv_halo_kernel; a wave computes its part again by itself
        float not_finite = 0.f;
        uint32_t least = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float v = acc[i][j][e] + low[i][j][e];
                    acc[i][j][e] = v;
                    not_finite = fmaf(v, 0.f, not_finite);
                    least = min(least, (__float_as_uint(v) << 1) - 1u);
                }
        const bool redo = !(not_finite == 0.f) || least < ((127u - 104u) << 24) - 1u;
        const int m0 = mt * MT + wm0;
        const bool inexact = __builtin_amdgcn_readfirstlane(*(volatile uint32_t *)&inexact_x) != 0 ||
                             __builtin_amdgcn_readfirstlane(*(volatile uint32_t *)&inexact_w[mt & 1]) == (uint32_t)mt + 1u;
        if (__builtin_expect(inexact || __builtin_amdgcn_ballot_w64(redo), 0)) {
            uint32_t vo_b[WN];
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                int col = j0 + wn0 + 32 * j + l32;
                asm volatile("" : "+v"(col));   // as there
                uint32_t n, px;
                p.div_px.divmod((uint32_t)col, n, px);
                vo_b[j] = col < p.cols ? 4u * (uint32_t)((int)n * p.K * p.px + (int)px) : kOob;
            }
            pointwise_fp32<ROWS>(p, rw, m0 + l32, lhi, [&](int k, float (&b)[WN]) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < WN; ++j) b[j] = Elem<float>::load(rx, k < p.K && vo_b[j] != kOob ? vo_b[j] + (uint32_t)k * plane : kOob, 0);
            }, acc);
        }
        auto store = [&](auto wholec) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                uint32_t vo = out[j] == kOob ? kOob : out[j] + (uint32_t)(mt * MT) * plane;
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        uint32_t v = vo;
                        if constexpr (!wholec) v = m0 + 32 * i + 8 * (e / 4) + e % 4 + 4 * lhi < p.M ? vo : kOob;
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][e]), ry, (int)v, 0, 0);
                        vo += e % 4 == 3 ? 5u * plane : plane;
                        asm("" : "+v"(vo));   // one running address, not one scalar per row
                    }
            }
        };
        if (m0 + 32 * WM <= p.M) store(std::true_type{});
        else store(std::false_type{});
    }
}

}  // namespace ucd
