// Fused Winograd F(2x2,3x3), fp32 tensors, on the bf16 matrix pipe (see gemm_split.hpp for the three-way split and
// its error).  Included by conv_winograd.hip behind WinoGeom and FusedParams.
//
// A workgroup owns 64 output channels x 64 tiles for all 16 transform points, as wino_fused_kernel does, but its eight
// waves share the points instead of the block: wave w multiplies points 2w and 2w+1 for the whole block (2 x 2
// MFMA tiles each, 128 accumulator registers, two waves per SIMD).  Every transformed value then has one reader, so
// it crosses LDS as one fp32 word and is split in the reader's registers, once; U is read by its one wave straight
// from the workspace in operand order (blocks of 8 input channels, [point][Ci / 8][Mo4][8]) and never enters LDS.
// With the 32 x 32 quarter blocks of wino_fused_kernel each value would be split, or its three parts read from LDS,
// by two waves.  A step is 16 input channels: 48 MFMAs, about 530 other vector instructions (two patches of 32
// additions, 64 splits of 6), 64 KB of LDS written and read.  The points of a tile meet after the last step, in
// LDS, for the output transform.
//
// One accumulator per point serves all six products: the reduction is over input channels only, 16 of them per
// addition instead of two.  Relative L2 error against fp64, ReLU activations, this kernel / fp32 instructions: 64
// channels 2.2e-7 / 2.3e-7, 256 3.9e-7 / 4.3e-7, 384 4.6e-7 / 5.1e-7, 512 5.4e-7 / 5.9e-7 (16 channels: 1.56e-7 /
// 1.45e-7, which is why layers of fewer than 32 keep wino_fused_kernel, see the launch for the line; it is the faster one there too, 14.2 / 16.2 us
// for 16 -> 32 channels of 16x16 at b = 8).
// Measured at b = 256, us, wino_fused_kernel / this: 384 -> 384 13x13 527 / 410, 256 -> 256 14x14 302 / 230, 64 -> 64 56x56
// 337 / 307, 512 -> 512 7x7 (b = 64) 148 / 99, phases of 11x11 stride 4 509 / 435.  Of the matrix pipe's cycles in the
// first, 39 % are MFMAs (counters; 11 other vector instructions per MFMA), and the pipe hides those only in part (a
// register loop with 8 of them per MFMA runs at 43 cycles per MFMA instead of 32); LDS bank conflicts take twice the
// cycles of its active LDS instructions.
#pragma once

namespace ucd {

constexpr int kWsC = 16;   // input channels per step

// One lane's MFMA operand in three parts, and a quarter of its making: values 2i and 2i + 1 of eight
struct SplitCell {
    u32x4 part[3];
    __device__ __forceinline__ void pair(int i, const float (&v)[8], uint32_t &rest)
    {
        uint32_t h, m, l;
        split_pair(v[2 * i], v[2 * i + 1], h, m, l, rest);
        part[0][i] = h; part[1][i] = m; part[2][i] = l;
    }
    __device__ __forceinline__ bf16x8 operand(int pl) const { return __builtin_bit_cast(bf16x8, part[pl]); }
};

// The four 2x2 output tiles o[i] of output channels kq .. kq+3 at tile (th, tw) of image n (see wino_fused_kernel)
template <bool PHASED>
__device__ __forceinline__ void wino_store4(const FusedParams &p, uint32_t n, int h0, int w0, int kq,
                                            const float (&o)[4][2][2])
{
    const WinoGeom &g = p.g;
    float *out = (float *)p.out;
    if constexpr (PHASED) {
        typedef float f32x4_dw __attribute__((ext_vector_type(4), aligned(4)));
        if (g.sw == 4) {  // the four channels are four adjacent pixels of dx
            if (kq >= g.Co) return;
            const int c = kq / (4 * g.sh), pr = kq / 4 % g.sh;
#pragma unroll
            for (int dr = 0; dr < 2; ++dr)
#pragma unroll
                for (int dc = 0; dc < 2; ++dc) {
                    const int h = g.sh * (h0 + dr) + pr - g.oph, w = 4 * (w0 + dc) - g.opw;
                    if ((unsigned)h >= (unsigned)g.oh) continue;
                    float *dst = out + (((long)n * g.oc + c) * g.oh + h) * g.ow + w;
                    if (w >= 0 && w + 3 < g.ow) {
                        f32x4_dw v4;
                        v4.x = o[0][dr][dc]; v4.y = o[1][dr][dc]; v4.z = o[2][dr][dc]; v4.w = o[3][dr][dc];
                        *reinterpret_cast<f32x4_dw *>(dst) = v4;
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if ((unsigned)(w + i) < (unsigned)g.ow) dst[i] = o[i][dr][dc];
                    }
                }
            return;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = kq + i;
            if (k >= g.Co) continue;
            const int c = k / (g.sh * g.sw), pr = k / g.sw % g.sh, pc = k % g.sw;
#pragma unroll
            for (int dr = 0; dr < 2; ++dr)
#pragma unroll
                for (int dc = 0; dc < 2; ++dc) {
                    const int h = g.sh * (h0 + dr) + pr - g.oph, w = g.sw * (w0 + dc) + pc - g.opw;
                    if ((unsigned)h < (unsigned)g.oh && (unsigned)w < (unsigned)g.ow)
                        out[(((long)n * g.oc + c) * g.oh + h) * g.ow + w] = o[i][dr][dc];
                }
        }
    } else {
        const bool h1 = h0 + 1 < g.Ho, w1 = w0 + 1 < g.Wo;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (kq + i >= g.Co) continue;
            float *dst = out + (((long)n * g.Co + kq + i) * g.Ho + h0) * g.Wo + w0;
            dst[0] = o[i][0][0];
            if (w1) dst[1] = o[i][0][1];
            if (h1) {
                dst[g.Wo] = o[i][1][0];
                if (w1) dst[g.Wo + 1] = o[i][1][1];
            }
        }
    }
}

// PW, ODD_W, PHASED as in wino_fused_kernel (row loads only).
template <int PW, bool ODD_W, bool PHASED>
__global__ __launch_bounds__(512, 2) void wino_fused_split_kernel(FusedParams p)
{
    // V of a step, [point][tile][channel], the four-channel groups of a tile's row exchanged by (tile / 4) % 4 so that
    // neither the writes nor the 16-byte reads pile up on a bank; after the last step the half points' partial outputs
    __shared__ __attribute__((aligned(16))) float Vs[2][16][64][kWsC];
    const WinoGeom &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;

    const uint32_t v = xcd_order(blockIdx.x, gridDim.x);
    const int kb = (int)(v % (uint32_t)p.k_blocks), tb = (int)(v / (uint32_t)p.k_blocks);
    const int k0 = kb * 64, t0 = tb * 64;

    const __amdgpu_buffer_rsrc_t rin = make_rsrc_bytes(p.in, 0, p.in_bytes);
    const __amdgpu_buffer_rsrc_t ru = make_rsrc_bytes(p.U, 0, p.u_bytes);

    // producer role: the patches of tile `lane` for channels 2*wave and 2*wave + 1 of the step, one after the other.
    // Row windows and their completion are wino_fused_kernel's.
    uint32_t voff[4], xoff[4];
    bool first_col, ok0, ok1, ok2, ok3, okm1, okm2, live;
    uint32_t n_img = 0, th = 0, tw = 0;
    {
        const int j = t0 + lane;
        uint32_t t;
        live = j < p.n_tiles;
        if (live) {
            p.divT.divmod((uint32_t)j, n_img, t);
            p.divTW.divmod(t, th, tw);
        }
        const int h0 = 2 * (int)th - g.pad_h, ws = 2 * (int)tw;
        first_col = tw == 0;
        ok1 = ws + 1 < g.Wi; ok2 = ws + 2 < g.Wi; ok3 = ws + 3 < g.Wi;
        ok0 = ws < g.Wi; okm1 = ws - 1 < g.Wi; okm2 = ws - 2 < g.Wi;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int h = h0 + r;
            const bool ok = live && (unsigned)h < (unsigned)g.Hi;
            const uint32_t row = 4u * (uint32_t)(((int)n_img * g.Ci * g.Hi + h) * g.Wi + ws);
            voff[r] = ok ? row : kOob;
            xoff[r] = ok && PW >= 1 && lane == 0 && tw > 0 ? row - PW * 4u : kOob;
        }
    }
    float d[16], dx[PW == 2 ? 8 : 4];
    auto fetch_row = [&](int c0, int h, int r) __attribute__((always_inline)) {
        const int c = c0 + 2 * wave + h;
        const uint32_t so = c < g.Ci ? 4u * (uint32_t)(c * g.Hi * g.Wi) : kOob;  // a channel past the last one reads as 0
        {
            if constexpr (PW == 0) {
                const f32x4 q = buf_load4(rin, voff[r], so);
                d[4 * r] = q.x; d[4 * r + 1] = q.y; d[4 * r + 2] = q.z; d[4 * r + 3] = q.w;
            } else if constexpr (PW == 2) {
                const auto q = __builtin_amdgcn_raw_buffer_load_b64(rin, (int)voff[r], (int)so, 0);
                d[4 * r + 2] = __uint_as_float(q[0]); d[4 * r + 3] = __uint_as_float(q[1]);
                const auto e = __builtin_amdgcn_raw_buffer_load_b64(rin, (int)xoff[r], (int)so, 0);
                dx[2 * r] = __uint_as_float(e[0]); dx[2 * r + 1] = __uint_as_float(e[1]);
            } else {
                const auto q = __builtin_amdgcn_raw_buffer_load_b96(rin, (int)voff[r], (int)so, 0);
#pragma unroll
                for (int c3 = 0; c3 < 3; ++c3) d[4 * r + 1 + c3] = __uint_as_float(q[c3]);
                dx[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rin, (int)xoff[r], (int)so, 0));
            }
        }
    };
    auto fetch_patch = [&](int c0, int h) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) fetch_row(c0, h, r);
    };
    // this lane's word of (point 0, its tile, channel 2*wave): points are 1024 words apart, channel 2*wave + 1 one
    const int v_put = lane * kWsC + ((((wave >> 1) ^ (lane >> 2)) & 3) << 2) + 2 * (wave & 1);
    float tr[16];
    auto finish_patch = [&]() __attribute__((always_inline)) {
        constexpr int kShr = 0x138;  // wave_shr:1
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (PW == 1) {
                if constexpr (ODD_W) d[4 * r + 2] = ok1 ? d[4 * r + 2] : 0.f;
                d[4 * r + 3] = ok2 ? d[4 * r + 3] : 0.f;
                const int left = __builtin_amdgcn_update_dpp((int)__float_as_uint(dx[r]), (int)__float_as_uint(d[4 * r + 2]),
                                                             kShr, 0xf, 0xf, false);
                d[4 * r] = ODD_W ? __uint_as_float((uint32_t)left) : first_col ? 0.f : __uint_as_float((uint32_t)left);
            } else if constexpr (PW == 2) {
                d[4 * r + 2] = ok0 ? d[4 * r + 2] : 0.f;
                d[4 * r + 3] = ok1 ? d[4 * r + 3] : 0.f;
                const float own0 = okm2 ? dx[2 * r] : 0.f, own1 = okm1 ? dx[2 * r + 1] : 0.f;
                const int l0 = __builtin_amdgcn_update_dpp((int)__float_as_uint(own0), (int)__float_as_uint(d[4 * r + 2]),
                                                           kShr, 0xf, 0xf, false);
                const int l1 = __builtin_amdgcn_update_dpp((int)__float_as_uint(own1), (int)__float_as_uint(d[4 * r + 3]),
                                                           kShr, 0xf, 0xf, false);
                d[4 * r] = first_col ? 0.f : __uint_as_float((uint32_t)l0);
                d[4 * r + 1] = first_col ? 0.f : __uint_as_float((uint32_t)l1);
            } else {
                d[4 * r + 1] = ok1 ? d[4 * r + 1] : 0.f;
                d[4 * r + 2] = ok2 ? d[4 * r + 2] : 0.f;
                d[4 * r + 3] = ok3 ? d[4 * r + 3] : 0.f;
            }
        }
    };
    auto column_transform = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float a0 = d[c], a1 = d[4 + c], a2 = d[8 + c], a3 = d[12 + c];
            tr[c] = a0 - a2; tr[4 + c] = a1 + a2; tr[8 + c] = a2 - a1; tr[12 + c] = a1 - a3;
        }
    };
    auto put_row = [&](float *vs, int h, int r) __attribute__((always_inline)) {
        float *dst = vs + v_put + h;
        {
            const float a0 = tr[4 * r], a1 = tr[4 * r + 1], a2 = tr[4 * r + 2], a3 = tr[4 * r + 3];
            dst[(4 * r + 0) * 64 * kWsC] = a0 - a2;
            dst[(4 * r + 1) * 64 * kWsC] = a1 + a2;
            dst[(4 * r + 2) * 64 * kWsC] = a2 - a1;
            dst[(4 * r + 3) * 64 * kWsC] = a1 - a3;
        }
    };
    auto store_v = [&](float *vs, int h) __attribute__((always_inline)) {
        finish_patch();
        column_transform();
#pragma unroll
        for (int r = 0; r < 4; ++r) put_row(vs, h, r);
    };

    // consumer role: point 2*wave + q.  U: 8 channels of output channel 32*ct + l32 in 32 adjacent bytes; the upper
    // half of the wave takes the next block of 8 channels (behind the last block of a plane it reads the next
    // plane's first, whose products with V's zeros vanish)
    const uint32_t u_plane = 4u * (uint32_t)(p.ci_pad * g.Mo4);
    uint32_t uoff[2];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        const int k = k0 + 32 * ct + l32;
        uoff[ct] = k < g.Mo4 ? 32u * (uint32_t)(lhi * g.Mo4 + k) : kOob;
    }
    float ur[2][8];   // [0]: of the point after the one being multiplied, [1]: of that point itself until it is split
    auto fetch_u = [&](int c0, int q, int ct) __attribute__((always_inline)) {
        const uint32_t so = (uint32_t)(2 * wave + q) * u_plane + 4u * (uint32_t)(c0 * g.Mo4);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const f32x4 t = buf_load4(ru, uoff[ct] + 16u * e, so);
            ur[ct][4 * e] = t.x; ur[ct][4 * e + 1] = t.y; ur[ct][4 * e + 2] = t.z; ur[ct][4 * e + 3] = t.w;
        }
    };
    // words of (point 2*wave, tile l32): channel groups 2*lhi and 2*lhi + 1
    const int v_sw = (l32 >> 2) & 3;
    const int v_get0 = (2 * wave * 64 + l32) * kWsC + (((2 * lhi) ^ v_sw) << 2);
    const int v_get1 = (2 * wave * 64 + l32) * kWsC + (((2 * lhi + 1) ^ v_sw) << 2);

    f32x16 acc[2][2][2];  // [point][32 output channels][32 tiles]
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[q][i][j][e] = 0.f;

    float *vbuf = &Vs[0][0][0][0];
    constexpr int kBufWords = 16 * 64 * kWsC;
    // A half step multiplies one point in four groups of six MFMAs, one group per 32 x 32 tile.  Each group's vector
    // work stands between its MFMAs: the operand that the next group, or the next half step's first, needs is split
    // as soon as the registers of its predecessor are free, and a patch of the next step is transformed into the other
    // LDS buffer.  (All splits in front of all MFMAs: both waves of a SIMD leave the barrier together, compute
    // together and then wait for the matrix pipe together; it measured 1-2 % slower with long reductions and 4 %
    // faster on 64 channels.)
    SplitCell a0, a1, b0, b1;
    uint32_t rest = 0;
    float vv[8];
    auto read_v = [&](const float *vr, int q, int tt) __attribute__((always_inline)) {
        const f32x4 x = *reinterpret_cast<const f32x4 *>(vr + v_get0 + (64 * q + 32 * tt) * kWsC);
        const f32x4 y = *reinterpret_cast<const f32x4 *>(vr + v_get1 + (64 * q + 32 * tt) * kWsC);
        vv[0] = x.x; vv[1] = x.y; vv[2] = x.z; vv[3] = x.w; vv[4] = y.x; vv[5] = y.y; vv[6] = y.z; vv[7] = y.w;
    };
    fetch_u(0, 0, 0);
    fetch_u(0, 0, 1);
    {
        float d0[16], dx0[PW == 2 ? 8 : 4];   // both patches in flight at once
        fetch_patch(0, 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) d0[i] = d[i];
#pragma unroll
        for (int i = 0; i < (PW == 2 ? 8 : 4); ++i) dx0[i] = dx[i];
        fetch_patch(0, 1);
        float d1[16], dx1[PW == 2 ? 8 : 4];
#pragma unroll
        for (int i = 0; i < 16; ++i) { d1[i] = d[i]; d[i] = d0[i]; }
#pragma unroll
        for (int i = 0; i < (PW == 2 ? 8 : 4); ++i) { dx1[i] = dx[i]; dx[i] = dx0[i]; }
        store_v(vbuf, 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) d[i] = d1[i];
#pragma unroll
        for (int i = 0; i < (PW == 2 ? 8 : 4); ++i) dx[i] = dx1[i];
        store_v(vbuf, 1);
    }
    fetch_patch(kWsC, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) a0.pair(i, ur[0], rest);
    fetch_u(0, 1, 0);
    __syncthreads();
    read_v(vbuf, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) b0.pair(i, vv, rest);

    int cur = 0;
    for (int c0 = 0; c0 < g.Ci; c0 += kWsC) {
        const float *vr = vbuf + cur * kBufWords;
        float *vw = vbuf + (cur ^ 1) * kBufWords;
        auto half = [&](auto qc) __attribute__((always_inline)) {
            constexpr int q = qc;
            const int c_next = q == 0 ? c0 : c0 + kWsC;   // the next half step: its channels (its point: q ^ 1)
            // group G = 2*ct + tt; work(m) stands behind MFMA m
            auto group = [&](f32x16 &d, const SplitCell &a, const SplitCell &b, auto work) __attribute__((always_inline)) {
                auto one = [&](auto mc) __attribute__((always_inline)) {
                    constexpr int m = mc;
                    constexpr int PL_A[6] = {0, 0, 1, 1, 0, 2}, PL_B[6] = {0, 1, 0, 1, 2, 0};
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.operand(PL_A[m]), b.operand(PL_B[m]), d, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    work(m);
                    __builtin_amdgcn_sched_barrier(0);
                };
                static_for<6>(one);
            };
            // The patch that the half step before loaded is transformed first, so that the next one's loads, into the
            // same registers, are in flight for 18 of the 24 MFMAs (with the loads in the last group, behind the
            // transform's own registers, they had 5: 384 -> 384 13x13 b = 256 423 us against 412 now, 64 -> 64 56x56 322
            // against 312, phases of 11x11 stride 4 433 against 405).
            read_v(vr, q, 1);
            group(acc[q][0][0], a0, b0, [&](int m) __attribute__((always_inline)) {
                if (m == 0) finish_patch();
                if (m == 1) column_transform();
                if (m >= 2) b1.pair(m - 2, vv, rest);
                if (m >= 2) put_row(vw, q, m - 2);
            });
            group(acc[q][0][1], a0, b1, [&](int m) __attribute__((always_inline)) {
                if (m < 4) fetch_row(q == 0 ? c0 + kWsC : c0 + 2 * kWsC, q ^ 1, m);
                if (m < 4) a1.pair(m, ur[1], rest);
                if (m == 4) fetch_u(c_next, q ^ 1, 1);
            });
            group(acc[q][1][0], a1, b0, [&](int m) __attribute__((always_inline)) {
                if (m >= 2) a0.pair(m - 2, ur[0], rest);
                if (m == 5) fetch_u(c0 + kWsC, q, 0);
            });
            if (q == 1) __syncthreads();   // the next step's V is complete, and this step's has been read
            read_v(q == 0 ? vr : vw, q ^ 1, 0);
            group(acc[q][1][1], a1, b1, [&](int m) __attribute__((always_inline)) {
                if (m >= 2) b0.pair(m - 2, vv, rest);
            });
        };
        half(std::integral_constant<int, 0>{});
        half(std::integral_constant<int, 1>{});
        cur ^= 1;
    }

    // range check as in gemm_kernel_split
    bool redo = (rest & 0xFFFFu) != 0;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    redo |= __builtin_amdgcn_classf(acc[q][i][j][e], 0x297) |
                            __builtin_amdgcn_classf(acc[q][i][j][e] * 0x1p-22f, 0x090);
    if (__syncthreads_or(redo)) {
        // the same sums with the fp32 instructions, one step after the other: MFMA e takes channel e of the lower half
        // wave's eight and of the upper half's (every block recomputed, 384 -> 384 13x13 b = 256: 1000 us, against 410
        // without and 525 of wino_fused_kernel)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[q][i][j][e] = 0.f;
#pragma unroll 1
        for (int c0 = 0; c0 < g.Ci; c0 += kWsC) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                fetch_patch(c0, h);
                store_v(vbuf, h);
            }
            __syncthreads();
            const bool in_plane = c0 + 8 * lhi < p.ci_pad;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) {
                    fetch_u(c0, q, ct);
#pragma unroll
                    for (int e = 0; e < 8; ++e) ur[ct][e] = in_plane ? ur[ct][e] : 0.f;
                }
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    read_v(vbuf, q, tt);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
#pragma unroll
                        for (int ct = 0; ct < 2; ++ct)
                            acc[q][ct][tt] = __builtin_amdgcn_mfma_f32_32x32x2f32(ur[ct][e], vv[e], acc[q][ct][tt], 0, 0, 0);
                }
            }
            __syncthreads();
        }
    }

    // Output transform.  Along the columns a wave has two of its row's four points: wave 2i the terms m0 + m1 and
    // m1 of the two output columns, wave 2i + 1 m2 and -m2 - m3.  They meet in LDS, 32 output channels at a time:
    // [wave][output column][output channel][tile].
    float *ex = vbuf;
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
        if (ct) __syncthreads();
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = 8 * (e / 4) + 4 * lhi + e % 4;
                const float ma = acc[0][ct][tt][e], mb = acc[1][ct][tt][e];
                float *dst = ex + ((wave * 2) * 32 + row) * 64 + 32 * tt + l32;
                dst[0] = wave & 1 ? ma : ma + mb;
                dst[32 * 64] = wave & 1 ? -ma - mb : mb;
            }
        __syncthreads();
        float o[4][2][2];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                float t[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float *src = ex + ((4 * r + c) * 32 + 4 * wave + i) * 64 + lane;
                    t[r] = src[0] + src[2 * 32 * 64];
                }
                o[i][0][c] = t[0] + t[1] + t[2];
                o[i][1][c] = t[1] - t[2] - t[3];
            }
        if (live) wino_store4<PHASED>(p, n_img, 2 * (int)th, 2 * (int)tw, k0 + 32 * ct + 4 * wave, o);
    }
}

}  // namespace ucd
