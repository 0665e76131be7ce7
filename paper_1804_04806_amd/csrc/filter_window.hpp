// BackwardFilter of 3x3 stride-1 layers with bf16 tensors on v_mfma_f32_32x32x16_bf16, all nine taps of a block of channels at once.
//
// The reduction runs over pixels, which is how both tensors lie in memory: an MFMA operand is eight pixels of a row of one
// channel.  An image is cut into strips of eight columns; a step of 16 pixels is one row of two strips, one per half of the
// wave.  A wave owns 32 output x 32 input channels of every tap.  It walks down the rows of x: a row (ten pixels, from which
// the three column taps' operands are made in registers) meets the three rows of dy that its row taps pair it with, of which one is new, so
// that two operands serve nine MFMAs.
//
// A workgroup multiplies RB rows of a pair of strips (a unit) while it turns the rows of the next into operands in the other half of LDS
// and loads those of the one after.  A thread takes a row of a strip of a channel in loads of four pixels from inside
// the row, moved to where they belong; what lies outside the image is zero.  Cells stand [channel][row][strip] at an odd
// pitch: neighbouring threads write neighbouring cells, and reads of 32 channels fall on all banks.
//
// The units are dealt to several workgroups per block of channels, which add their sums into dw by atomics, by way of LDS so that a wave
// adds to adjacent elements.  75 MB of sums, what the registers of the chip hold, take 40 us to add (6 to store), which is why two waves
// share a block of sums and halve it between them before that (256 channels 14x14 b = 256: 105 -> 101 us, 128 28x28 b = 32 43 -> 37),
// though four rows per unit are then all that the registers leave room for (384 channels 13x13 162 -> 167).
// 384 channels 13x13 b = 256: 276 us with the element-wise tiles, 167 with this, 150 of them without the atomics; its MFMAs, a fifth of them
// padding, would take 85.
#pragma once
#include "gemm_core.hpp"

namespace ucd {

struct FilterWindowParams {
    const void *x, *dy;
    float *dw;
    uint32_t x_bytes, dy_bytes;
    int b, C, H, W, K, P, Q, ph, pw;
    int k_blocks, c_blocks, units, per_wg;
    int down;                         // units follow each other down an image's rows, or along them
    FastDiv div_strips, div_chunks;   // strips per row, units per strip
};

// RB rows of dy per unit, WK x WC waves on a unit, WR units at a time
template <int RB_, int WK_, int WC_, int WR_>
struct FilterWindowTile {
    static constexpr int RB = RB_, WK = WK_, WC = WC_, WR = WR_, KT = 32 * WK, CT = 32 * WC;
    static constexpr int PD = 2 * RB + 1, PX = 2 * (RB + 2) + 1;                        // cells per channel
    static constexpr int DY = KT * PD * 16 + 128, X = CT * PX * 16, UNIT = DY + X + CT * PX * 4, BUF = WR * UNIT;
    static constexpr int kThreads = 512 / (2 * WR);                                     // on a strip
    static constexpr int ND = (KT * RB + kThreads - 1) / kThreads, NX = (CT * (RB + 2) + kThreads - 1) / kThreads;   // rows of a strip per thread
    static constexpr int kOutRow = 292, OUT = 8 * 8 * kOutRow * 4;                      // floats of an output channel, padded
    static constexpr int MEET = 8 * 72 * 64 * 4;                                        // half of every wave's sums
    static constexpr int LDS = 2 * BUF > OUT ? (2 * BUF > MEET ? 2 * BUF : MEET) : OUT > MEET ? OUT : MEET;
    static_assert(WK * WC * WR == 8 && WR == 2 && UNIT % 16 == 0 && LDS <= 163840, "eight waves, LDS");
};

template <class T>
__global__ __launch_bounds__(512, 2) void filter_window_kernel(FilterWindowParams p)
{
    constexpr int RB = T::RB, ND = T::ND, NX = T::NX, WR = T::WR;
    __shared__ __attribute__((aligned(16))) char lds[T::LDS];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk0 = 32 * (wave % T::WK), wc0 = 32 * (wave / T::WK % T::WC), wr = wave / (T::WK * T::WC);

    uint32_t id = xcd_order(blockIdx.x, gridDim.x);
    const int k0 = (int)(id % (uint32_t)p.k_blocks) * T::KT; id /= (uint32_t)p.k_blocks;
    const int c0 = (int)(id % (uint32_t)p.c_blocks) * T::CT; id /= (uint32_t)p.c_blocks;
    const int u0 = (int)id * p.per_wg, u1 = min(p.units, u0 + p.per_wg);

    const __amdgpu_buffer_rsrc_t rx = make_rsrc_bytes(p.x, 0, p.x_bytes), rd = make_rsrc_bytes(p.dy, 0, p.dy_bytes);

    // a thread's rows of strips: all of the strip tid % 2 of the pair and of one of the WR units
    const int half = tid & 1, tr = (tid >> 1) % WR, tq = tid / (2 * WR);
    constexpr int kNoRow = (1 << 15) - 1;
    uint32_t d_off[ND], x_off[NX], d_at[ND], x_at[NX];   // from the strip's first pixel; row << 16 | cell
#pragma unroll
    for (int i = 0; i < ND; ++i) {
        const int e = tq + T::kThreads * i, k = e / RB, row = e % RB;
        d_off[i] = 2u * (uint32_t)(((k0 + k) * p.P + row) * p.Q);
        d_at[i] = (uint32_t)(k0 + k < p.K && k < T::KT ? row : kNoRow) << 16 | (uint32_t)(k * T::PD + 2 * row + half);
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int e = tq + T::kThreads * i, c = e / (RB + 2), row = e % (RB + 2);
        x_off[i] = 2u * (uint32_t)(((c0 + c) * p.H + row) * p.W);
        x_at[i] = (uint32_t)(c0 + c < p.C && c < T::CT ? row : kNoRow) << 16 | (uint32_t)(c * T::PX + 2 * row + half);
    }
    auto in_block = [&](int i, int total) __attribute__((always_inline)) {
        return T::kThreads * (i + 1) <= total || tq < total - T::kThreads * i;
    };
    // the unit in the registers, and how many bits the loads of four pixels have to be moved down (x's first also up)
    u32x2 qd[ND][2], qx[NX][3];
    int sd[2], sx[3], sx_up;
    auto place = [&](int u, int hf, uint32_t &n, uint32_t &strip, uint32_t &rc) __attribute__((always_inline)) {
        uint32_t rest;
        if (p.down) {
            p.div_chunks.divmod((uint32_t)u, rest, rc);
            p.div_strips.divmod(2 * rest + (uint32_t)hf, n, strip);
        } else {
            p.div_strips.divmod(2 * (uint32_t)u + (uint32_t)hf, rest, strip);
            p.div_chunks.divmod(rest, n, rc);
        }
    };
    auto load = [&](int u) __attribute__((always_inline)) {
        uint32_t rc, n, strip;
        place(u + tr, half, n, strip, rc);
        const int p0 = (int)rc * RB, h0 = p0 - p.ph;
        const bool live = (int)n < p.b && u + tr < u1;
        uint32_t at_d[2], at_x[3];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = 8 * (int)strip + 4 * j, at = min(col, p.Q - 4);
            sd[j] = 16 * (col - at);
            at_d[j] = live && col - at < 4 ? 2u * (uint32_t)(((int)n * p.K * p.P + p0) * p.Q + at) : kOob;
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int col = 8 * (int)strip + 4 * j - p.pw, at = min(max(col, 0), p.W - 4);
            sx[j] = 16 * max(col - at, 0);
            if (j == 0) sx_up = 16 * max(at - col, 0);
            at_x[j] = live && col - at < 4 ? 2u * (uint32_t)(((int)n * p.C * p.H + h0) * p.W + at) : kOob;
        }
#pragma unroll
        for (int i = 0; i < ND; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t vo = p0 + (int)(d_at[i] >> 16) < p.P && at_d[j] != kOob ? d_off[i] + at_d[j] : kOob;
                qd[i][j] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rd, (int)vo, 0, 0));
            }
#pragma unroll
        for (int i = 0; i < NX; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const uint32_t vo = (unsigned)(h0 + (int)(x_at[i] >> 16)) < (unsigned)p.H && at_x[j] != kOob ? x_off[i] + at_x[j] : kOob;
                qx[i][j] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rx, (int)vo, 0, 0));
            }
    };
    auto down = [](u32x2 q, int bits) __attribute__((always_inline)) { return __builtin_bit_cast(u32x2, __builtin_bit_cast(uint64_t, q) >> (bits & 63)); };
    auto up = [](u32x2 q, int bits) __attribute__((always_inline)) { return __builtin_bit_cast(u32x2, __builtin_bit_cast(uint64_t, q) << (bits & 63)); };
    auto put = [&](int buf) __attribute__((always_inline)) {
        char *dst = lds + buf * T::BUF + tr * T::UNIT;
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            const u32x2 a = down(qd[i][0], sd[0]), b = down(qd[i][1], sd[1]);
            const u32x4 cell = {a[0], a[1], b[0], b[1]};
            if (in_block(i, T::KT * RB)) *reinterpret_cast<u32x4 *>(dst + (d_at[i] & 0xFFFFu) * 16) = cell;
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const u32x2 a = up(down(qx[i][0], sx[0]), sx_up), b = down(qx[i][1], sx[1]), c = down(qx[i][2], sx[2]);
            const u32x4 cell = {a[0], a[1], b[0], b[1]};
            if (in_block(i, T::CT * (RB + 2))) {
                *reinterpret_cast<u32x4 *>(dst + T::DY + (x_at[i] & 0xFFFFu) * 16) = cell;
                *reinterpret_cast<uint32_t *>(dst + T::DY + T::X + (x_at[i] & 0xFFFFu) * 4) = c[0];
            }
        }
    };

    f32x16 acc[9];
    // EXACT: x that only meets the zeros which fill a unit up (columns behind a row's end, rows behind the last one) is zero too
    auto pass = [&](auto exact) __attribute__((always_inline)) {
        constexpr bool EXACT = exact;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;

        load(u0);
        put(0);
        if (u0 + WR < u1) load(u0 + WR);
        __syncthreads();

        int buf = 0;
        for (int u = u0; u < u1; u += WR) {
            const char *base = lds + buf * T::BUF + wr * T::UNIT;
            const char *pd = base + ((wk0 + l32) * T::PD + lhi) * 16;
            const char *px = base + T::DY + ((wc0 + l32) * T::PX + lhi) * 16;
            const char *pt = base + T::DY + T::X + ((wc0 + l32) * T::PX + lhi) * 4;
            u32x4 a[4], b[2];   // dy rows j - 2 .. j + 1; x rows j, j + 1
            uint32_t bt[2];
            auto read_a = [&](int j) __attribute__((always_inline)) { a[j & 3] = *reinterpret_cast<const u32x4 *>(pd + j * 32); };
            auto read_b = [&](int j) __attribute__((always_inline)) {
                b[j & 1] = *reinterpret_cast<const u32x4 *>(px + j * 32);
                bt[j & 1] = *reinterpret_cast<const uint32_t *>(pt + j * 8);
            };
            u32x4 cols;
            int rows = RB;
            if constexpr (EXACT) {
                uint32_t n, strip, rc;
                place(u + wr, lhi, n, strip, rc);
                rows = p.P - (int)rc * RB;
                const int left = p.Q - 8 * (int)strip;
#pragma unroll
                for (int i = 0; i < 4; ++i) cols[i] = left >= 2 * i + 2 ? 0xFFFFFFFFu : left == 2 * i + 1 ? 0xFFFFu : 0u;
            }
            read_a(0);
            read_b(0);
            auto row = [&](auto jc) __attribute__((always_inline)) {
                constexpr int j = jc;
                if constexpr (j + 1 < RB) read_a(j + 1);
                if constexpr (j + 1 < RB + 2) read_b(j + 1);
                __builtin_amdgcn_sched_barrier(0);
                const u32x4 x = b[j & 1];
                const uint32_t t = bt[j & 1];
                u32x4 o[3];
                o[0] = x;
                o[1] = u32x4{__builtin_amdgcn_alignbit(x[1], x[0], 16), __builtin_amdgcn_alignbit(x[2], x[1], 16),
                             __builtin_amdgcn_alignbit(x[3], x[2], 16), __builtin_amdgcn_alignbit(t, x[3], 16)};
                o[2] = u32x4{x[1], x[2], x[3], t};
                if constexpr (EXACT)
#pragma unroll
                    for (int s = 0; s < 3; ++s) o[s] &= cols;
#pragma unroll
                for (int s = 0; s < 3; ++s)
#pragma unroll
                    for (int r = 0; r < 3; ++r)
                        if (j - r >= 0 && j - r < RB) {
                            u32x4 y = o[s];
                            if (EXACT && j - r >= rows) y = u32x4{0, 0, 0, 0};
                            acc[3 * r + s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[(j - r) & 3]),
                                                                                     __builtin_bit_cast(bf16x8, y), acc[3 * r + s], 0, 0, 0);
                        }
                __builtin_amdgcn_sched_barrier(0);
            };
            const bool more = u + WR < u1, early = wave < 4;
            auto stage = [&]() __attribute__((always_inline)) {
                if (!more) return;
                put(buf ^ 1);
                if (u + 2 * WR < u1) load(u + 2 * WR);
            };
            if (early) stage();
            static_for<RB + 2>(row);
            if (!early) stage();
            __syncthreads();
            buf ^= 1;
        }
    };
    pass(std::false_type{});
    float not_finite = 0.f;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) not_finite = fmaf(acc[t][e], 0.f, not_finite);
    if (__syncthreads_or(!(not_finite == 0.f))) pass(std::true_type{});

    // two waves that shared a block: each gives the other the half of its rows that the other adds to dw
    {
        float *mine = reinterpret_cast<float *>(lds) + wave * 72 * 64 + lane, *other = reinterpret_cast<float *>(lds) + (wave ^ 4) * 72 * 64 + lane;
        auto give = [&](auto first) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int e = 0; e < 8; ++e) mine[(8 * t + e) * 64] = acc[t][first + e];
        };
        auto take = [&](auto first) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[t][first + e] += other[(8 * t + e) * 64];
        };
        typedef std::integral_constant<int, 0> Low;
        typedef std::integral_constant<int, 8> High;
        if (wr) give(Low{});
        else give(High{});
        __syncthreads();
        if (wr) take(High{});
        else take(Low{});
        __syncthreads();
    }
    // eight output channels of the wave at a time
    float *out = reinterpret_cast<float *>(lds) + wave * 8 * T::kOutRow;
    const int left = min(32, p.C - c0 - wc0) * 9;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if (g / 2 != wr) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < 9; ++t) out[(4 * lhi + e) * T::kOutRow + 9 * l32 + t] = acc[t][4 * g + e];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int r = 0; r < 8; ++r) {
            const int k = k0 + wk0 + 8 * g + r;
            if (k >= p.K) break;
            float *dst = p.dw + ((size_t)k * p.C + c0 + wc0) * 9;
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                const int at = lane + 64 * i;
                if (at < left) unsafeAtomicAdd(dst + at, out[r * T::kOutRow + at]);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

}  // namespace ucd
