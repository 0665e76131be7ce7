// Direct convolution over a window kept in LDS, fp32 tensors on the bf16 matrix pipe (gfx950); products, error and range as
// in gemm_split.hpp.
//
// An implicit GEMM loads and splits an input element once per filter tap that reads it.  Here a workgroup keeps the
// window of its output positions in LDS as MFMA operands, split once: one cell of 16 bytes per part holds eight channels
// of one pixel, so that a tap is an offset of the operand's address and nothing else.  The reduction runs over 16
// channels at a time, within them over filter rows, within them over the taps of a row.
//
// BackwardData with column stride NPH.  Pixel h = sh*t + a is reached through the filter rows r = (a + ph) % sh + sh*i, from
// row t + (a + ph) / sh - i of dy, and columns likewise.  The row phases a are workgroups of their own (a filter row belongs
// to one of them); the column phases b of a position are accumulated side by side, so that the taps of a filter
// row share the window and no tap is multiplied that is not there.
// Positions (t, u) run over images, then blocks of Wc columns, rows, columns of the block; a tile is NT consecutive ones.
#pragma once
#include "gemm_split.hpp"

namespace ucd {

constexpr int kHaloC = 16;          // channels per chunk

struct HaloParams {
    const void *in, *w;
    void *out;
    uint32_t in_bytes, w_bytes, out_bytes;
    int K, P, Q;                    // the gathered tensor (dy): channels, rows, columns
    int C, H, W;                    // the output (dx)
    int R, RS, CRS;
    int sh, ph, dc;                 // strides and padding; dc: column of dy under a position less its window's first
    int Gh, Wc, nb, pitch, cells;   // position grid: rows, columns per block, blocks; window row in LDS; cells per half and part
    int images, cols, tiles_m;      // images * blocks, positions, row tiles
    FastDiv div_wc, div_gh, div_nb, div_pitch;
};

// NPH column phases, S filter columns, PAR = the column padding modulo NPH; a wave owns WM x WN tiles of 32 x 32 per phase.  Four waves share half of a CU's LDS
// with another workgroup, eight have all of it.
template <int NPH_, int S_, int PAR_, int WM_, int WAVES_M_, int WN_, int WAVES_N_>
struct HaloTile {
    static constexpr int NPH = NPH_, S = S_, PAR = PAR_, WM = WM_, WN = WN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
    static constexpr int THREADS = 64 * WAVES_M * WAVES_N, LDS = THREADS == 256 ? 81408 : 162816;
    static constexpr int MT = 32 * WM * WAVES_M, NT = 32 * WN * WAVES_N;
    // column phase of tap s, and the column it reads less the position's (and less pw / NPH)
    static constexpr int phase(int s) { return (s + PAR) % NPH; }
    static constexpr int column(int s) { return (NPH == 2 && phase(s) == 1 ? PAR : 0) - s / NPH; }
    static constexpr int kFirst = S == 1 ? 0 : column(S - 1) < column(S - 2) ? column(S - 1) : column(S - 2);
    static constexpr int kLast = S == 1 || column(0) > column(1) ? column(0) : column(1);
    static constexpr int kSpan = kLast - kFirst;   // a window row is that much wider than its positions
    static constexpr int A_HALF = (MT + 4) * 16, A_PART = 2 * A_HALF, A_TAP = 3 * A_PART, A_BUF = S * A_TAP;
    static constexpr int NA = MT * 8 / THREADS;           // pairs of channels of a filter row per thread and step
    static constexpr int NB = 2;                          // window cells per thread and chunk
    static constexpr int kMaxCells = (LDS / 2 - A_BUF) / 96 < THREADS ? (LDS / 2 - A_BUF) / 96 : THREADS;
};

typedef float f32x2 __attribute__((ext_vector_type(2)));

// N adjacent dwords, as few loads as they take
template <int N>
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so, float (&d)[N])
{
    int i = 0;
    if constexpr (N >= 4) {
        const f32x4 v = buf_load4(r, vo, so);
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
        i = 4;
    }
    constexpr int M = N % 4;
    if constexpr (M == 3) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b96(r, (int)(vo + 4u * i), (int)so, 0);
        d[i] = __uint_as_float(v[0]); d[i + 1] = __uint_as_float(v[1]); d[i + 2] = __uint_as_float(v[2]);
    } else if constexpr (M == 1) {
        d[i] = Elem<float>::load(r, vo + 4u * i, so);
    }
}

template <class T>
__global__ __launch_bounds__(T::THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv_halo_kernel(HaloParams p)
{
    constexpr int NPH = T::NPH, S = T::S, WM = T::WM, WN = T::WN, MT = T::MT, NT = T::NT;
    __shared__ __attribute__((aligned(16))) char lds[T::LDS];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave % T::WAVES_M) * (WM * 32), wn0 = (wave / T::WAVES_M) * (WN * 32);

    const int a = (int)blockIdx.y;                       // row phase
    const int r0 = (a + p.ph) % p.sh, dr = (a + p.ph) / p.sh;
    const int Ra = (p.R - r0 + p.sh - 1) / p.sh;         // its filter rows r0, r0 + sh, ...
    const uint32_t id = xcd_order(blockIdx.x, gridDim.x);
    const int m0 = (int)(id % (uint32_t)p.tiles_m) * MT, j0 = (int)(id / (uint32_t)p.tiles_m) * NT;

    const __amdgpu_buffer_rsrc_t rin = make_rsrc_bytes(p.in, 0, p.in_bytes), rw = make_rsrc_bytes(p.w, 0, p.w_bytes),
                                 rout = make_rsrc_bytes(p.out, 0, p.out_bytes);
    const int half_b = p.cells * 16, part_b = 2 * half_b, buf_b = 3 * part_b;
    char *const lds_b = lds + 2 * T::A_BUF;

    // the window: rows of the first virtual image (images x column blocks) from its row t0 - (Ra - 1) on, then whole ones
    const int g0 = (int)p.div_wc.div((uint32_t)j0);
    const int v0 = (int)p.div_gh.div((uint32_t)g0), t0 = g0 - v0 * p.Gh, len0 = p.Gh - t0 + Ra - 1, len = p.Gh + Ra - 1;
    uint32_t b_off[T::NB];
    int b_dst[T::NB];
    bool b_hi[T::NB];
#pragma unroll
    for (int x = 0; x < T::NB; ++x) {
        const int e = tid + T::THREADS * x, hi = e >= p.cells ? 1 : 0, q = e - hi * p.cells;
        uint32_t lr, lc;
        p.div_pitch.divmod((uint32_t)q, lr, lc);
        int v = v0, row = t0 + (int)lr - (Ra - 1) + dr;
        if ((int)lr >= len0) {
            const int k = ((int)lr - len0) / len;
            v = v0 + 1 + k;
            row = (int)lr - len0 - k * len - (Ra - 1) + dr;
        }
        uint32_t n, cb;
        p.div_nb.divmod((uint32_t)v, n, cb);
        const int col = (int)cb * p.Wc + (int)lc + p.dc;
        const bool ok = e < 2 * p.cells && v < p.images && (unsigned)row < (unsigned)p.P && (unsigned)col < (unsigned)p.Q;
        b_off[x] = ok ? 4u * (uint32_t)((((int)n * p.K + 8 * hi) * p.P + row) * p.Q + col) : kOob;
        b_dst[x] = e < 2 * p.cells ? hi * half_b + q * 16 : -1;
        b_hi[x] = hi;
    }
    // the filter: a thread takes a row of taps of one output channel for two channels of the chunk.  (One tap of all eight
    // channels of a cell per thread costs the cache three times the accesses, which is then what bounds the kernel.)
    uint32_t a_off[T::NA];
    int a_dst[T::NA];
#pragma unroll
    for (int x = 0; x < T::NA; ++x) {
        const int e = tid + T::THREADS * x, m = e % MT, pair = e / MT;
        a_off[x] = m0 + m < p.C ? 4u * (uint32_t)((m0 + m) * p.RS + 2 * pair * p.CRS) : kOob;
        a_dst[x] = (pair >> 2) * T::A_HALF + m * 16;
    }
    // this lane's columns: the cell of tap (0, 0) of the first filter row
    int col_cell[WN];
#pragma unroll
    for (int i = 0; i < WN; ++i) {
        const int j = min(j0 + wn0 + 32 * i + l32, p.cols - 1);
        uint32_t g, u, v, t;
        p.div_wc.divmod((uint32_t)j, g, u);
        p.div_gh.divmod(g, v, t);
        const int row = (int)v == v0 ? (int)t - t0 : len0 + ((int)v - v0 - 1) * len + (int)t;
        col_cell[i] = (lhi * p.cells + (row + Ra - 1) * p.pitch + (int)u) * 16;
    }

    f32x16 acc[NPH][WM][WN], low[NPH][WM][WN];
    uint32_t rest = 0;
    const int chunks = (p.K + kHaloC - 1) / kHaloC;
    const uint32_t in_plane = 4u * (uint32_t)(p.P * p.Q);

    auto pass = [&](auto fp32c) __attribute__((always_inline)) {
        constexpr bool FP32 = fp32c;   // operands as they are, on the fp32 instructions: cells of eight floats
#pragma unroll
        for (int b = 0; b < NPH; ++b)
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) { acc[b][i][j][e] = 0.f; if (!FP32) low[b][i][j][e] = 0.f; }
        float ra[T::NA][2][S], rb[T::NB][8];
        auto load_a = [&](int c, int gi) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < T::NA; ++x)
#pragma unroll
                for (int i = 0; i < 2; ++i)   // channels past the last one lie behind the filter and read as zero
                    load_row<S>(rw, a_off[x], 4u * (uint32_t)((kHaloC * c + i) * p.CRS + (r0 + p.sh * gi) * S), ra[x][i]);
        };
        auto load_b = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < T::NB; ++x)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    uint32_t vo = b_off[x];
                    // channels past the last one are the next image's
                    if (kHaloC * (c + 1) > p.K) vo = kHaloC * c + (b_hi[x] ? 8 : 0) + i < p.K ? vo : kOob;
                    rb[x][i] = Elem<float>::load(rin, vo, (uint32_t)(kHaloC * c + i) * in_plane);
                }
        };
        auto put = [&](char *dst, int part, const float (&v)[8]) __attribute__((always_inline)) {
            if constexpr (FP32) {   // two rows of 16 bytes in the first two parts' places
                const f32x4 x = {v[0], v[1], v[2], v[3]}, y = {v[4], v[5], v[6], v[7]};
                *reinterpret_cast<f32x4 *>(dst) = x;
                *reinterpret_cast<f32x4 *>(dst + part) = y;
            } else {
                u32x4 c[3];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t h, m, l;
                    split_pair(v[2 * i], v[2 * i + 1], h, m, l, rest);
                    c[0][i] = h; c[1][i] = m; c[2][i] = l;
                }
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4 *>(dst + pl * part) = c[pl];
            }
        };
        auto put_a = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < T::NA; ++x) {
                const int pair = ((tid + T::THREADS * x) / MT) & 3;
                char *dst = lds + buf * T::A_BUF + a_dst[x];
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    if constexpr (FP32) {
                        const f32x2 v = {ra[x][0][s], ra[x][1][s]};
                        *reinterpret_cast<f32x2 *>(dst + s * T::A_TAP + (pair >> 1) * T::A_PART + (pair & 1) * 8) = v;
                    } else {
                        uint32_t h, m, l;
                        split_pair(ra[x][0][s], ra[x][1][s], h, m, l, rest);
                        uint32_t *at = reinterpret_cast<uint32_t *>(dst + s * T::A_TAP + pair * 4);
                        at[0] = h;
                        at[T::A_PART / 4] = m;
                        at[2 * T::A_PART / 4] = l;
                    }
                }
            }
        };
        auto put_b = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < T::NB; ++x)
                if (b_dst[x] >= 0) put(lds_b + buf * buf_b + b_dst[x], part_b, rb[x]);
        };
        // the step after (c, gi)
        auto next = [&](int &c, int &gi) __attribute__((always_inline)) {
            if (++gi == Ra) { gi = 0; ++c; }
        };
        int lc = 0, lg = 0;       // the step whose filter cells are loaded next
        load_a(lc, lg);
        load_b(0);
        next(lc, lg);
        put_a(0);
        put_b(0);
        load_a(lc, lg);
        next(lc, lg);
        if (chunks > 1) load_b(1);
        __syncthreads();

        const bool early = T::THREADS == 256 || wave < 4;   // in a workgroup of eight the two waves of a SIMD stage at different ends
        int buf_a = 0;
        for (int c = 0; c < chunks; ++c) {
            for (int gi = 0; gi < Ra; ++gi) {
                const bool last = gi == Ra - 1;
                auto stage = [&]() __attribute__((always_inline)) {
                    put_a(buf_a ^ 1);
                    load_a(lc, lg);
                    if (last && c + 1 < chunks) {
                        put_b((c + 1) & 1);
                        if (c + 2 < chunks) load_b(c + 2);
                    }
                };
                if (early) stage();
                const char *pa = lds + buf_a * T::A_BUF + lhi * T::A_HALF + (wm0 + l32) * 16;
                const char *pb = lds_b + (c & 1) * buf_b - gi * p.pitch * 16;
                u32x4 va[3][WM], vb[3][WN];   // one tap's operands; a column phase reuses the window's from the phase before it
                auto read_a = [&](int s, int pl) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < WM; ++i)
                        va[pl][i] = *reinterpret_cast<const u32x4 *>(pa + s * T::A_TAP + pl * T::A_PART + i * 32 * 16);
                };
                auto read_b = [&](int s, int pl) __attribute__((always_inline)) {
#pragma unroll
                    for (int j = 0; j < WN; ++j)
                        vb[pl][j] = *reinterpret_cast<const u32x4 *>(pb + col_cell[j] + pl * part_b + (T::column(s) - T::kFirst) * 16);
                };
                if constexpr (FP32) {
#pragma unroll
                    for (int s = 0; s < S; ++s) {
#pragma unroll
                        for (int pl = 0; pl < 2; ++pl) {
                            read_a(s, pl);
                            read_b(s, pl);
                        }
#pragma unroll
                        for (int e = 0; e < 8; ++e)
#pragma unroll
                            for (int i = 0; i < WM; ++i)
#pragma unroll
                                for (int j = 0; j < WN; ++j)
                                    acc[T::phase(s)][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                                        __uint_as_float(va[e >> 2][i][e & 3]), __uint_as_float(vb[e >> 2][j][e & 3]), acc[T::phase(s)][i][j], 0, 0, 0);
                    }
                } else {
                    // Six groups of products per tap: lh', mm', mh', hh' (its own accumulator), hm', hl'.  In this order every
                    // part's registers are free, and read again for the next tap, two groups or more before it uses them.
#pragma unroll
                    for (int pl = 2; pl >= 0; --pl) {
                        read_a(0, pl);
                        read_b(0, 2 - pl);
                    }
                    auto tap = [&](auto sc) __attribute__((always_inline)) {
                        constexpr int s = sc;
                        constexpr bool more = s + 1 < S, more_b = more && T::column(s + 1 < S ? s + 1 : s) != T::column(s);
                        constexpr int PL_A[6] = {2, 1, 1, 0, 0, 0}, PL_B[6] = {0, 1, 0, 0, 1, 2};
                        auto group = [&](auto gc) __attribute__((always_inline)) {
                            constexpr int g = gc;
#pragma unroll
                            for (int i = 0; i < WM; ++i)
#pragma unroll
                                for (int j = 0; j < WN; ++j) {
                                    f32x16 &d = g == 3 ? acc[T::phase(s)][i][j] : low[T::phase(s)][i][j];
                                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[PL_A[g]][i]),
                                                                                __builtin_bit_cast(bf16x8, vb[PL_B[g]][j]), d, 0, 0, 0);
                                }
                            if (more && g == 0) read_a(s + 1, 2);
                            if (more && g == 2) read_a(s + 1, 1);
                            if (more_b && g == 3) read_b(s + 1, 0);
                            if (more_b && g == 4) read_b(s + 1, 1);
                            if (more && g == 5) read_a(s + 1, 0);
                            if (more_b && g == 5) read_b(s + 1, 2);
                            __builtin_amdgcn_sched_barrier(0);
                        };
                        static_for<6>(group);
                    };
                    static_for<S>(tap);
                }
                if (!early) stage();
                next(lc, lg);
                buf_a ^= 1;
                __syncthreads();
            }
        }
    };
    pass(std::false_type{});

    // not finite, or below 2^-104 and not zero (see gemm_split.hpp), in few instructions per sum: a product with zero
    // keeps what is not finite, and zero less one in the bits without the sign is the largest of all
    float not_finite = 0.f;
    uint32_t least = 0xFFFFFFFFu;
#pragma unroll
    for (int b = 0; b < NPH; ++b)
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float v = acc[b][i][j][e] + low[b][i][j][e];
                    acc[b][i][j][e] = v;
                    not_finite = fmaf(v, 0.f, not_finite);
                    least = min(least, (__float_as_uint(v) << 1) - 1u);
                }
    const bool redo = (rest & 0xFFFFu) != 0 || !(not_finite == 0.f) || least < ((127u - 104u) << 24) - 1u;
    if (__syncthreads_or(redo)) pass(std::true_type{});

#pragma unroll
    for (int j = 0; j < WN; ++j) {
        const int jo = j0 + wn0 + 32 * j + l32;
        if (jo >= p.cols) continue;
        uint32_t g, u, v, t, n, cb;
        p.div_wc.divmod((uint32_t)jo, g, u);
        p.div_gh.divmod(g, v, t);
        p.div_nb.divmod(v, n, cb);
        const int h = p.sh * (int)t + a, w = NPH * ((int)cb * p.Wc + (int)u);
        if (h >= p.H) continue;
        const uint32_t off = 4u * (uint32_t)((((int)n * p.C + m0 + wm0 + 4 * lhi) * p.H + h) * p.W + w);
        const bool in0 = w < p.W, in1 = NPH == 2 && w + 1 < p.W;
        const bool whole = m0 + wm0 + 32 * WM <= p.C;
        const uint32_t plane = 4u * (uint32_t)(p.H * p.W);
        auto store = [&](auto kind, uint32_t vo) __attribute__((always_inline)) {   // 0: first column phase, 2: both
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    uint32_t v = vo;
                    if (!whole) v = m0 + wm0 + 32 * i + 8 * (e / 4) + e % 4 + 4 * lhi < p.C ? vo : kOob;
                    if constexpr (kind == 2) {
                        const u32x2 d = {__float_as_uint(acc[0][i][j][e]), __float_as_uint(acc[NPH - 1][i][j][e])};
                        __builtin_amdgcn_raw_buffer_store_b64(d, rout, (int)v, 0, 0);
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[0][i][j][e]), rout, (int)v, 0, 0);
                    }
                    vo += e % 4 == 3 ? 5u * plane : plane;
                    asm("" : "+v"(vo));   // one running address, not one scalar per row
                }
        };
        if constexpr (NPH == 1) {
            store(std::integral_constant<int, 0>{}, in0 ? off : kOob);
        } else {
            store(std::integral_constant<int, 2>{}, in0 && in1 ? off : kOob);
            if (__builtin_amdgcn_ballot_w64(in0 && !in1)) store(std::integral_constant<int, 0>{}, in0 && !in1 ? off : kOob);
        }
    }
}

}  // namespace ucd
