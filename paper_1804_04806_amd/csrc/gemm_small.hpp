// Implicit GEMMs of small layers (gfx950): a few microseconds of work, where what counts is the chain of waits that one
// workgroup goes through, not the rate of any unit.
//
// The tile kernels give such a launch a handful of workgroups, each walking the whole reduction step by step through LDS
// (32x128 tiles: 16 workgroups of 18 steps for 16 <- 32 channels 3x3 16x16 b = 8, a barrier and a round trip to memory
// each), or split it over workgroups that add into an output which another launch has to clear first.  Here a tile is one
// MFMA of 16x16, so that the chip gets a workgroup per CU, and the waves of a workgroup divide the reduction: each
// loads its operands straight from memory into MFMA order, two batches of kBatch steps in flight, with no barrier until the
// partial sums meet in LDS, in a fixed order.  Forward and BackwardData (all stride phases) are one launch without atomics or
// a zero fill; a BackwardFilter of 512 reduction rows and more adds chunks of its sums to a cleared dw with atomics.
//
// Addresses.  An element's offset is a part that depends on the tile position (one register per lane) plus one that
// depends on the reduction row; the latter, and which taps it stands for, are computed once per workgroup into an LDS
// table that all lanes read four rows at a time.
#pragma once
#include "gemm_core.hpp"

namespace ucd {

constexpr int kSmallRows = 2560;    // reduction rows per filling of the table
constexpr int kSmallPhases = 16;

typedef double f64x4 __attribute__((ext_vector_type(4)));

enum SmallKind { kSmallFwd, kSmallBwdData, kSmallBwdFilter };

// One GEMM: rows m (A), columns j (B), Kd reduction rows.
struct SmallPhase {
    FastDiv grid_hw, grid_w;      // columns (Forward, BackwardData) or reduction rows (BackwardFilter) -> (n, a, b)
    FastDiv taps, taps_w;         // reduction rows or columns -> (channel, tap), tap -> (r, s)
    int N, Kd;
    int mul_h, add_h, mul_w, add_w;   // window origin of (a, b) in the gathered tensor
    int tap_add_h, tap_add_w;         // BackwardData: first filter row / column of the phase
    int h0, w0;                       // BackwardData: pixel (h0 + hs*a, w0 + ws*b) of dx
};
struct SmallHead {
    const void *a, *b;
    void *out;
    uint32_t a_bytes, b_bytes;
    int M, tiles_m;
    int Ct, Ht, Wt, dir;          // the gathered tensor (x or dy)
    int RS, S, CRS;               // of the filter
    int hs, ws;                   // BackwardData: strides
    int HWo, Wo;                  // plane and row of the output; BackwardFilter: plane of dy, row of dw
    int a_n_stride;               // BackwardFilter: elements of an image of dy
    int k_chunk;                  // BackwardFilter: reduction rows per workgroup; several chunks meet through atomics
    bool vec_a, vec_b;            // BackwardFilter: a lane's rows are adjacent in dy (in x) as well
    float beta;
};
template <int PHASES>
struct SmallParamsT : SmallHead {
    SmallPhase ph[PHASES];
};

// (a single phase where there is but one: the arguments are written anew for every launch)
template <int KIND> using SmallParams = SmallParamsT<KIND == kSmallBwdData ? kSmallPhases : 1>;

// FEW: few reduction rows of fp32.  The fp32 instructions round every product, which among so few is the larger part of
// the error (2 to 16 products spread over four accumulators: up to 1.3 times that of the tile kernels that add them in one
// chain; 65 to 128 up to 1.08 times that of those that split them); 64-bit products and sums leave the rounding of the result:
// 0.2 to 0.9 times, in the same time up to 64 rows, one step of a wave (310 layers, 1.00; 65 to 128 rows 1.02).
constexpr int kSmallFew = 64;

template <class E, int KIND, bool BIG, bool FEW = false>
__global__ __launch_bounds__(1024) void gemm_kernel_small(SmallParams<KIND> p)
{
    constexpr bool F32 = std::is_same<E, float>::value;
    constexpr uint32_t EB = Elem<E>::kBytes;
    // consecutive reduction rows of a lane: four feed four v_mfma_f32_16x16x4_f32, eight one v_mfma_f32_16x16x32_bf16
    constexpr int PL = F32 ? 4 : 8, STEP = 4 * PL;
    constexpr int kBatch = F32 ? 4 : 2;
    constexpr int LDP = 18;   // row stride of the partial tiles: the four lane groups of a store on different banks
    // A from memory four (eight) rows at a time; otherwise it has a table column of its own
    constexpr bool VEC_A = KIND == kSmallFwd;
    constexpr bool TAB_MASK = KIND == kSmallBwdFilter;   // the mask is the row's, the tap the lane's
    __shared__ __attribute__((aligned(16))) uint32_t tab_b[kSmallRows], tab_t[kSmallRows];
    __shared__ __attribute__((aligned(16))) uint32_t tab_a[VEC_A ? 4 : kSmallRows];
    __shared__ __attribute__((aligned(16))) uint32_t tab_w[TAB_MASK && BIG ? kSmallRows : 4];
    __shared__ __attribute__((aligned(16))) double part[16][16 * LDP];

    const SmallPhase &q = p.ph[KIND == kSmallBwdData ? blockIdx.y : 0];
    const int lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;
    const int waves = (int)blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m0 = ((int)blockIdx.x % p.tiles_m) * 16, j0 = ((int)blockIdx.x / p.tiles_m) * 16;
    if (j0 >= q.N) return;
    const __amdgpu_buffer_rsrc_t ra = make_rsrc_bytes(p.a, 0, p.a_bytes), rb = make_rsrc_bytes(p.b, 0, p.b_bytes);

    // this lane's part of the addresses; what lies outside the GEMM reads as zero
    uint32_t a_off = kOob, b_off = 0, mask = 0xFFFFFFFFu, mask_w = 0xFFFFFFFFu, tap = 31, tap_s = 31;
    const int m = m0 + l16, j = j0 + l16;
    if (m < p.M) a_off = EB * (uint32_t)(KIND == kSmallFwd ? m * p.CRS : KIND == kSmallBwdData ? m * p.RS : m * p.HWo);
    if (KIND == kSmallBwdFilter) {
        if (j < q.N) {
            uint32_t c, t, r, s;
            q.taps.divmod((uint32_t)j, c, t);
            q.taps_w.divmod(t, r, s);
            b_off = EB * (uint32_t)(((int)c * p.Ht + (int)r) * p.Wt + (int)s);
            tap = BIG ? r : t;
            tap_s = s;
        }
    } else if (j < q.N) {
        uint32_t n, rest, a, b;
        q.grid_hw.divmod((uint32_t)j, n, rest);
        q.grid_w.divmod(rest, a, b);
        const int hb = (int)a * q.mul_h + q.add_h, wb = (int)b * q.mul_w + q.add_w;
        b_off = EB * (uint32_t)(((int)n * p.Ct * p.Ht + hb) * p.Wt + wb);
        const int nr = (int)(q.taps.d / q.taps_w.d), ns = (int)q.taps_w.d;
        uint32_t okh = 0, okw = 0;
        for (int r = 0; r < nr; ++r) okh |= (uint32_t)((unsigned)(hb + p.dir * r) < (unsigned)p.Ht) << r;
        for (int s = 0; s < ns; ++s) okw |= (uint32_t)((unsigned)(wb + p.dir * s) < (unsigned)p.Wt) << s;
        if (BIG) {
            mask = ~okh | 0x80000000u;
            mask_w = ~okw | 0x80000000u;
        } else {
            uint32_t ok = 0;
            for (int r = 0; r < nr; ++r) ok |= ((okh >> r) & 1u) ? okw << (r * ns) : 0u;
            mask = ~ok | 0x80000000u;
        }
    }

    f32x4 acc[4];   // one per MFMA of a step: shorter sums, and no MFMA waits for its predecessor
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    f64x4 few = {0., 0., 0., 0.};
    const int k_begin = KIND == kSmallBwdFilter ? (int)blockIdx.z * p.k_chunk : 0;
    const int k_end = KIND == kSmallBwdFilter ? min(q.Kd, k_begin + p.k_chunk) : q.Kd;
    for (int base = k_begin; base < k_end; base += kSmallRows) {
        const int rows_up = (min(kSmallRows, k_end - base) + STEP - 1) / STEP * STEP;
        if (base != k_begin) __syncthreads();
        for (int e = threadIdx.x; e < rows_up; e += (int)blockDim.x) {
            const int kk = base + e;
            const bool live = kk < k_end;
            if constexpr (KIND == kSmallBwdFilter) {
                uint32_t n, rest, a, b;
                q.grid_hw.divmod((uint32_t)kk, n, rest);
                q.grid_w.divmod(rest, a, b);
                const int hb = (int)a * q.mul_h + q.add_h, wb = (int)b * q.mul_w + q.add_w;
                tab_a[e] = live ? EB * (uint32_t)((int)n * p.a_n_stride + (int)rest) : kOob;
                tab_b[e] = EB * (uint32_t)(((int)n * p.Ct * p.Ht + hb) * p.Wt + wb);
                const int nr = (int)(q.taps.d / q.taps_w.d), ns = (int)q.taps_w.d;
                uint32_t okh = 0, okw = 0;
                for (int s = 0; s < ns; ++s) okw |= (uint32_t)((unsigned)(wb + s) < (unsigned)p.Wt) << s;
                for (int r = 0; r < nr; ++r) {
                    const bool in = (unsigned)(hb + r) < (unsigned)p.Ht;
                    okh |= BIG ? (uint32_t)in << r : in ? okw << (r * ns) : 0u;
                }
                tab_t[e] = live ? ~okh : 0xFFFFFFFFu;
                if constexpr (BIG) tab_w[e] = ~okw;
            } else {
                uint32_t c, t, r, s;
                q.taps.divmod((uint32_t)kk, c, t);
                q.taps_w.divmod(t, r, s);
                tab_b[e] = EB * (uint32_t)(((int)c * p.Ht + p.dir * (int)r) * p.Wt + p.dir * (int)s);
                tab_t[e] = live ? (BIG ? r | s << 8 : t) : 31u;
                if constexpr (!VEC_A)
                    tab_a[e] = live ? EB * (uint32_t)((int)c * p.CRS + (q.tap_add_h + p.hs * (int)r) * p.S + q.tap_add_w + p.ws * (int)s) : kOob;
            }
        }
        __syncthreads();

        const int steps = rows_up / STEP;
        const int s_begin = steps * wave / waves, s_end = steps * (wave + 1) / waves;
        struct Regs { uint32_t a[4], b[4]; };   // a lane's operands of one step
        auto load_run = [&](__amdgpu_buffer_rsrc_t r, uint32_t off, int h, uint32_t (&d)[4]) __attribute__((always_inline)) {
            if constexpr (F32) {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
#pragma unroll
                for (int i = 0; i < 4; ++i) d[i] = v[i];
            } else {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
                d[2 * h] = v[0];
                d[2 * h + 1] = v[1];
            }
        };
        auto load = [&](int st, Regs &g) __attribute__((always_inline)) {
            const int e0 = st * STEP + PL * grp;
#pragma unroll
            for (int h = 0; h < PL / 4; ++h) {
                const u32x4 tb = *reinterpret_cast<const u32x4 *>(tab_b + e0 + 4 * h);
                const u32x4 tt = *reinterpret_cast<const u32x4 *>(tab_t + e0 + 4 * h);
                u32x4 ta, tw;
                if constexpr (!VEC_A) ta = *reinterpret_cast<const u32x4 *>(tab_a + e0 + 4 * h);
                if constexpr (TAB_MASK && BIG) tw = *reinterpret_cast<const u32x4 *>(tab_w + e0 + 4 * h);
                uint32_t bo[4], ao[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t outside;
                    if constexpr (TAB_MASK && BIG) outside = (tt[i] >> tap) | (tw[i] >> tap_s);
                    else if constexpr (TAB_MASK) outside = tt[i] >> tap;
                    else if constexpr (BIG) outside = (mask >> (tt[i] & 31u)) | (mask_w >> (tt[i] >> 8));
                    else outside = mask >> tt[i];
                    bo[i] = (outside << 31) | (b_off + tb[i]);
                    // a part that is out of range stays so in the sum: both are below 2^31 or kOob
                    if constexpr (!VEC_A) ao[i] = (a_off + ta[i]) | ((a_off | ta[i]) & kOob);
                }
                if constexpr (KIND == kSmallBwdFilter) {
                    // four rows of one image: the first one's offset serves them all, and so does its out-of-range bit (the
                    // reduction is a multiple of four rows); x only where no tap can fall outside the image
                    if (p.vec_a) load_run(ra, ao[0], h, g.a);
                    if (p.vec_b) load_run(rb, bo[0], h, g.b);
                }
                const bool one_a = !VEC_A && !(KIND == kSmallBwdFilter && p.vec_a), one_b = !(KIND == kSmallBwdFilter && p.vec_b);
                if constexpr (F32) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (one_b) g.b[i] = __builtin_amdgcn_raw_buffer_load_b32(rb, (int)bo[i], 0, 0);
                        if (one_a) g.a[i] = __builtin_amdgcn_raw_buffer_load_b32(ra, (int)ao[i], 0, 0);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 4; i += 2) {
                        if (one_b) {
                            const uint32_t lo = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rb, (int)bo[i], 0, 0);
                            const uint32_t hi = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rb, (int)bo[i + 1], 0, 0);
                            g.b[2 * h + i / 2] = lo | hi << 16;
                        }
                        if (one_a) {
                            const uint32_t la = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(ra, (int)ao[i], 0, 0);
                            const uint32_t ha = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(ra, (int)ao[i + 1], 0, 0);
                            g.a[2 * h + i / 2] = la | ha << 16;
                        }
                    }
                }
            }
            if constexpr (VEC_A) {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(a_off + EB * (uint32_t)(base + e0)), 0, 0);
#pragma unroll
                for (int i = 0; i < 4; ++i) g.a[i] = v[i];
            }
        };
        auto multiply = [&](int st, int n, Regs &g) __attribute__((always_inline)) {
            if constexpr (VEC_A) {
                // rows past the end of the filter row are the next one's, which need not be finite: none of them counts
                const int left = k_end - base - st * STEP - PL * grp;
                if (st * STEP + STEP > k_end - base) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (F32) g.a[i] = i < left ? g.a[i] : 0u;
                        else g.a[i] = 2 * i + 1 < left ? g.a[i] : 2 * i < left ? g.a[i] & 0xFFFFu : 0u;
                    }
                }
            }
            if constexpr (FEW) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    few = __builtin_amdgcn_mfma_f64_16x16x4f64((double)__uint_as_float(g.a[i]), (double)__uint_as_float(g.b[i]), few, 0, 0, 0);
            } else if constexpr (F32) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(g.a[i]), __uint_as_float(g.b[i]), acc[i], 0, 0, 0);
            } else {
                const u32x4 va = {g.a[0], g.a[1], g.a[2], g.a[3]}, vb = {g.b[0], g.b[1], g.b[2], g.b[3]};
                acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, va), __builtin_bit_cast(bf16x8, vb), acc[n], 0, 0, 0);
            }
        };
        Regs g0[kBatch], g1[kBatch];
        auto load_batch = [&](int st, Regs (&g)[kBatch]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
                if (st + i < s_end) load(st + i, g[i]);
        };
        auto multiply_batch = [&](int st, int n, Regs (&g)[kBatch]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
                if (st + i < s_end) multiply(st + i, (n + i) % 4, g[i]);
        };
        load_batch(s_begin, g0);
        for (int st = s_begin; st < s_end; st += 2 * kBatch) {
            load_batch(st + kBatch, g1);
            multiply_batch(st, 0, g0);
            load_batch(st + 2 * kBatch, g0);
            multiply_batch(st + kBatch, kBatch, g1);
        }
    }

#pragma unroll
    for (int i = 0; i < 4; ++i) {   // a lane's four rows are adjacent, those of a 64-bit MFMA four apart
        if constexpr (FEW) part[wave][(4 * i + grp) * LDP + l16] = few[i];
        else part[wave][(4 * grp + i) * LDP + l16] = ((double)acc[0][i] + (double)acc[1][i]) + ((double)acc[2][i] + (double)acc[3][i]);
    }
    __syncthreads();
    if (threadIdx.x >= 256) return;
    const int row = (int)threadIdx.x >> 4, col = (int)threadIdx.x & 15;
    double all = 0;   // one rounding for the 16 to 64 partial sums
    for (int w = 0; w < waves; ++w) all += part[w][row * LDP + col];
    const float sum = (float)all;
    const int mo = m0 + row, jo = j0 + col;
    if (mo >= p.M || jo >= q.N) return;
    if constexpr (KIND == kSmallBwdFilter) {
        float *dst = (float *)p.out + (size_t)mo * p.Wo + jo;
        if (gridDim.z > 1) unsafeAtomicAdd(dst, sum);
        else *dst = p.beta == 0.f ? sum : *dst + sum;
    } else {
        uint32_t n, rest, a, b;
        q.grid_hw.divmod((uint32_t)jo, n, rest);
        q.grid_w.divmod(rest, a, b);
        Elem<E>::store(p.out, ((long)n * p.M + mo) * p.HWo + (long)(q.h0 + p.hs * (int)a) * p.Wo + q.w0 + p.ws * (int)b, sum);
    }
}

}  // namespace ucd
