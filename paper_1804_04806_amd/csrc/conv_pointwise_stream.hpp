// 1x1 stride-1 convolutions with more input channels than output channels or LDS hold, fp32 tensors on the bf16 matrix pipe
// (gfx950); products, error and range as in gemm_split.hpp.
//
// Input and filter stream through tiles of 128 output channels x 256 pixels.  Eight waves, 2 x 4, multiply 64 channels x 64
// pixels each (24 MFMAs for 12 KB of LDS reads per step of 16 channels); four load and split, with three steps of loads in
// flight, so that neither the splitting nor the wait for memory stands between two MFMAs of a wave.  Adjacent pixels of a pair
// lie in different halves of the tile's columns: cells go to LDS without bank conflicts, a lane's two results are one store.
// 512 -> 128 28x28 b = 128 in BackwardData: 142 us on the fp32 pipe -> 94 (392 tiles, the second round half empty); Forward of
// 256 -> 128 20x20 b = 100 in one round of 16 steps of 1536 MFMA cycles: 33 -> 26.
#pragma once
#include "conv_pointwise.hpp"

namespace ucd {

// Images of an even number of pixels.  ROWS: the filter is contiguous along the reduction (Forward); otherwise along the
// output channels (BackwardData).
template <bool ROWS>
__global__ __launch_bounds__(768, 3) void pointwise_split_stream_kernel(PointwiseParams p)
{
    constexpr int MT = 128, NT = 256;
    constexpr int A_HALF = (MT + 4) * 16, A_PART = 2 * A_HALF, A_BUF = 3 * A_PART;
    constexpr int B_HALF = (NT + 4) * 16, B_PART = 2 * B_HALF, B_BUF = 3 * B_PART;
    __shared__ __attribute__((aligned(16))) char lds[2 * (A_BUF + B_BUF)];
    __shared__ uint32_t inexact;   // some operand was not split exactly
    char *const lds_b = lds + 2 * A_BUF;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the tile rows of a pixel tile on one XCD
    const int xcd = (int)blockIdx.x % 8, rank = (int)blockIdx.x / 8;
    const int tile = rank / p.m_tiles * 8 + xcd, j0 = tile * NT, m0 = rank % p.m_tiles * MT, steps = (p.K + 15) / 16;
    if (tile >= p.whole) return;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc_bytes(p.x, 0, p.x_bytes), rw = make_rsrc_bytes(p.w, 0, p.w_bytes);
    const uint32_t plane = 4u * (uint32_t)p.px;
    if (tid == 0) inexact = 0;
    __syncthreads();

    if (wave >= 8) {
        const int cell = tid & 255, q = cell & 127, c_hi = cell >> 7;
        uint32_t n, px, rest = 0;
        p.div_px.divmod((uint32_t)(j0 + 2 * q), n, px);
        const uint32_t b_off = j0 + 2 * q < p.cols ? 4u * (uint32_t)(((int)n * p.K + 8 * c_hi) * p.px + (int)px) : kOob;
        const int a_hi = ROWS ? cell & 1 : c_hi, a_row = ROWS ? cell >> 1 : q;
        const uint32_t a_off = 4u * (uint32_t)((m0 + a_row) * p.w_row + 8 * a_hi * p.w_k);
        struct Cells {
            u32x2 b[8];
            float a[8];
        };
        auto load = [&](int st, Cells &r) __attribute__((always_inline)) {
            // rows past the last one lie behind the filter, or are the next channel's and not stored; channels past the last
            // one, which are the next image's or row's, are left out
            const int k0 = 16 * st < p.K ? 16 * st : 0, left = p.K - 16 * st;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                r.b[i] = __builtin_amdgcn_raw_buffer_load_b64(rx, (int)(8 * c_hi + i < left ? b_off : kOob), (int)((uint32_t)(k0 + i) * plane), 0);
            if constexpr (ROWS) {
                const uint32_t o = 8 * a_hi < left ? a_off : kOob;
                const f32x4 u = buf_load4(rw, o, 4u * (uint32_t)k0), v = buf_load4(rw, o, 4u * (uint32_t)k0 + 16u);
                r.a[0] = u.x; r.a[1] = u.y; r.a[2] = u.z; r.a[3] = u.w;
                r.a[4] = v.x; r.a[5] = v.y; r.a[6] = v.z; r.a[7] = v.w;
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    r.a[i] = Elem<float>::load(rw, 8 * a_hi + i < left ? a_off : kOob, 4u * (uint32_t)((k0 + i) * p.w_k));
            }
        };
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
        auto put = [&](int st, Cells &r) __attribute__((always_inline)) {
            if (ROWS && 16 * st + 16 > p.K) {
#pragma unroll
                for (int i = 0; i < 8; ++i) r.a[i] = 16 * st + 8 * a_hi + i < p.K ? r.a[i] : 0.f;
            }
            split_cell(lds + (st & 1) * A_BUF + a_hi * A_HALF + a_row * 16, A_PART, r.a);
            char *const to = lds_b + (st & 1) * B_BUF + c_hi * B_HALF + q * 16;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = __uint_as_float(r.b[j][i]);
                split_cell(to + i * 2048, B_PART, v);
            }
            if ((rest & 0xFFFFu) != 0) inexact = 1;
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

    const int wm0 = (wave & 1) * 64, wq0 = (wave >> 1) * 32;
    f32x16 acc[2][2], low[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = low[i][j][e] = 0.f;
    __syncthreads();
    for (int st = 0; st < steps; ++st) {
        const char *pa = lds + (st & 1) * A_BUF + lhi * A_HALF + (wm0 + l32) * 16;
        const char *pb = lds_b + (st & 1) * B_BUF + lhi * B_HALF + (wq0 + l32) * 16;
        u32x4 va[3][2], vb[3][2];
        auto read_a = [&](int pl) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2; ++i) va[pl][i] = *reinterpret_cast<const u32x4 *>(pa + pl * A_PART + i * 512);
        };
        auto read_b = [&](int pl) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 2; ++j) vb[pl][j] = *reinterpret_cast<const u32x4 *>(pb + pl * B_PART + j * 2048);
        };
        auto group = [&](int ga, int gb, f32x16 (&d)[2][2]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    d[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[ga][i]),
                                                                      __builtin_bit_cast(bf16x8, vb[gb][j]), d[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        // a part's reads one group ahead of its products: at most four parts are live
        read_a(2);
        read_b(0);
        read_a(1);
        __builtin_amdgcn_sched_barrier(0);
        group(2, 0, low);
        read_b(1);
        group(1, 0, low);
        read_a(0);
        group(1, 1, low);
        read_b(2);
        group(0, 0, acc);
        group(0, 1, low);
        group(0, 2, low);
        __syncthreads();
    }

    // range check as in conv_halo_kernel; a wave computes its part again by itself
    float not_finite = 0.f;
    uint32_t least = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float v = acc[i][j][e] + low[i][j][e];
                acc[i][j][e] = v;
                not_finite = fmaf(v, 0.f, not_finite);
                least = min(least, (__float_as_uint(v) << 1) - 1u);
            }
    const bool redo = !(not_finite == 0.f) || least < ((127u - 104u) << 24) - 1u;
    const int col = j0 + 2 * (wq0 + l32);
    uint32_t n, px;
    p.div_px.divmod((uint32_t)col, n, px);
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(*(volatile uint32_t *)&inexact) || __builtin_amdgcn_ballot_w64(redo), 0)) {
        const uint32_t vo_b = 4u * (uint32_t)((int)n * p.K * p.px + (int)px);
        pointwise_fp32<ROWS>(p, rw, m0 + wm0 + l32, lhi, [&](int k, float (&b)[2]) __attribute__((always_inline)) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rx, (int)(k < p.K && col < p.cols ? vo_b + (uint32_t)k * plane : kOob), 0, 0);
            b[0] = __uint_as_float(v[0]);
            b[1] = __uint_as_float(v[1]);
        }, acc);
    }
    if (col >= p.cols) return;
    const __amdgpu_buffer_rsrc_t ry = make_rsrc_bytes(p.y, 0, p.y_bytes);
    const int mw = m0 + wm0 + 4 * lhi;
    uint32_t vo = 4u * (uint32_t)(((int)n * p.M + mw) * p.px + (int)px);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (mw + 32 * i + 8 * (e / 4) + e % 4 < p.M)
                __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(acc[i][0][e]), __float_as_uint(acc[i][1][e])}, ry, (int)vo, 0, 0);
            vo += e % 4 == 3 ? 5u * plane : plane;
            asm("" : "+v"(vo));   // one running address, not one scalar per row
        }
}

}  // namespace ucd
