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
// 3 -> 64 7x7/2 224x224 b = 128: 807 us as tile GEMMs of merged phases on the fp32 instructions, 413 with this (bf16 482, 225); its MFMAs
// alone, with three quarters of the rows and 61 % of the taps real, would be 180.  37 % of the matrix pipe's cycles are MFMAs, with 6.0 other vector
// instructions each (the split of the window's cells, half of them, and of the filter's); operands read a pair ahead made it 3 % slower.
// A tile of which not all sums are finite or in range is begun anew, with parameters read again, so that nothing of it is live in the loop
// of the others, whose scalar registers are all in use (3 to 13 % of the time when they were spilled there).
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

// The tile from position j0 on; AGAIN: whose sums the split operands do not hold.  True: it has to be done again.
template <class E, bool AGAIN>
__device__ __forceinline__ bool few_tile(const FewParams &p, int j0, char *lds, int *tab)
{
    constexpr bool F32 = std::is_same<E, float>::value;
    constexpr int PARTS = F32 ? 3 : 1, NA = (kFewPairs * 64 + 511) / 512, NB = 3, EB = (int)Elem<E>::kBytes;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn0 = (wave & 3) * 64, wr = wave >> 2;

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
    int r0, s0, a_row;   // of its row: the filter's element under tap (0, 0), and where it lies; negative: no such row
    {
        uint32_t c, a, ah, aw;
        p.div_block.divmod((uint32_t)(tid & 31), c, a);
        p.div_vsw.divmod(a, ah, aw);
        r0 = (int)c < p.C ? (int)ah - p.sh * (p.fh - 1) : -(1 << 20);
        s0 = (int)aw - p.sw * (p.fw - 1);
        a_row = (int)c * p.R * p.S;
    }
    auto place_a = [&](int g) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NA; ++x) {
            const int e = tid + 512 * x, tap = 2 * (g * p.pairs + (e >> 6)) + (e >> 5 & 1);
            uint32_t u, v;
            p.div_v.divmod((uint32_t)tap, u, v);
            const int r = r0 + p.sh * (int)u, s = s0 + p.sw * (int)v;
            const bool ok = tap < p.taps && (unsigned)r < (unsigned)p.R && (unsigned)s < (unsigned)p.S;
            a_off[x] = ok ? (uint32_t)EB * (uint32_t)(a_row + r * p.S + s) : kOob;
        }
    };
    place_a(0);
    // this lane's positions: the cell of the last tap; of the one that it stores, image and first pixel
    int col_cell[2], n = -1, h0 = 0, w0 = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int j = j0 + wn0 + 32 * i + l32;
        uint32_t g, u, v, t, img, cb;
        p.div_wc.divmod((uint32_t)min(j, p.cols - 1), g, u);
        p.div_hb.divmod(g, v, t);
        p.div_nb.divmod(v, img, cb);
        const int row = (int)v == v0 ? p.fh * ((int)t - t0) : len0 + ((int)v - v0 - 1) * len + p.fh * (int)t;
        col_cell[i] = (row * p.pitch + (int)u) * 16;
        const int w = p.vsw * ((int)cb * p.Wc + (int)u);
        if (i == wr) {
            // a position behind the last one of its row belongs to the next block or to none
            n = j < p.cols && w < p.W + p.pw ? (int)img : -1;
            h0 = p.vsh * (int)t - p.ph;
            w0 = w - p.pw;
        }
    }

    f32x16 acc[2], low[2];
    uint32_t rest = 0;
    const int chunks = (p.K + kFewC - 1) / kFewC, steps = chunks * p.groups;
    const uint32_t in_plane = (uint32_t)EB * (uint32_t)(p.P * p.Q);

    // How the sums are made.  kSplit: as above.  kPlain: fp32 operands as they are, on the fp32 instructions, in cells of eight floats.
    // A tap that is not there is a zero in a tile's rows, and that times an infinity is no zero.  So when sums are not finite, elements of dy that
    // are not either count as 1 or -1 in the second time (bf16: kFinite), and two more passes find the sums that they belong to, on bf16
    // instructions: kSigns adds up the signs of their products with the filter (0 if a product is NaN), kNumber their number, over the taps that
    // there are.  The sum is infinite if all signs are equal, else NaN; where there are none it stands.
    enum { kSplit, kPlain, kFinite, kSigns, kNumber };
    int mode = kSplit;
    bool odd = false;  // dy is not finite
    auto load_bits = [](__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) __attribute__((always_inline)) -> uint32_t {
        if constexpr (F32) return __builtin_amdgcn_raw_buffer_load_b32(r, (int)vo, (int)so, 0);
        else return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)vo, (int)so, 0);
    };
    auto pass = [&](auto first) __attribute__((always_inline)) {   // first: kSplit or kPlain, or as mode says
        constexpr int FIRST = first;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) { acc[j][e] = 0.f; low[j][e] = 0.f; }
        uint32_t ra[NA][8], rb[NB][8];   // as they lie in memory
        auto value = [](uint32_t v) __attribute__((always_inline)) { return __uint_as_float(F32 ? v : v << 16); };
        auto load_a = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < NA; ++x)
#pragma unroll
                for (int i = 0; i < 8; ++i)   // channels past the last one lie behind the filter and read as zero
                    ra[x][i] = load_bits(rw, a_off[x], (uint32_t)EB * (uint32_t)((kFewC * c + i) * p.CRS));
        };
        auto load_b = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                if (512 * x >= p.cells) break;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    // channels past the last one are the next image's: an offset behind the tensor, also if added to kOob
                    const int k = kFewC * c + i;
                    rb[x][i] = load_bits(rin, b_off[x], k < p.K ? (uint32_t)k * in_plane : 0x7FFFFFF0u);
                }
            }
        };
        auto put = [&](char *dst, int part, const uint32_t (&d)[8]) __attribute__((always_inline)) {
            if constexpr (F32 && FIRST == kSplit) {
                u32x4 c[3];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t h, m, l;
                    split_pair(__uint_as_float(d[2 * i]), __uint_as_float(d[2 * i + 1]), h, m, l, rest);
                    c[0][i] = h; c[1][i] = m; c[2][i] = l;
                }
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4 *>(dst + pl * part) = c[pl];
            } else if constexpr (F32 && FIRST == kPlain) {   // two rows of 16 bytes in the first two parts' places
                *reinterpret_cast<u32x4 *>(dst) = u32x4{d[0], d[1], d[2], d[3]};
                *reinterpret_cast<u32x4 *>(dst + part) = u32x4{d[4], d[5], d[6], d[7]};
            } else {
                u32x4 c;
#pragma unroll
                for (int i = 0; i < 4; ++i)   // bf16: the low halves; fp32 signs and numbers: the high ones
                    c[i] = __builtin_amdgcn_perm(d[2 * i + 1], d[2 * i], F32 ? 0x07060302u : 0x05040100u);
                *reinterpret_cast<u32x4 *>(dst) = c;
            }
        };
        auto bits = [](float v) __attribute__((always_inline)) { return F32 ? __float_as_uint(v) : __float_as_uint(v) >> 16; };   // of values that bf16 holds
        auto put_a = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < NA; ++x) {
                const int e = tid + 512 * x;
                if constexpr (FIRST > kPlain) if (mode >= kSigns)
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float v = value(ra[x][i]);
                        ra[x][i] = bits(mode == kNumber ? a_off[x] != kOob : v > 0.f ? 1.f : v < 0.f ? -1.f : 0.f);
                    }
                if (e < p.pairs * 64) put(lds + buf * a_buf + e * 16, a_part, ra[x]);
            }
        };
        auto put_b = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                const int e = tid + 512 * x;
                if constexpr (FIRST != kSplit)
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float v = value(rb[x][i]), one = copysignf(1.f, v);
                        const bool finite = fabsf(v) < __builtin_inff();
                        if (e < p.cells) odd |= !finite;
                        if (mode < kSigns) rb[x][i] = finite ? rb[x][i] : bits(one);
                        else rb[x][i] = bits(finite ? 0.f : mode == kNumber ? 1.f : v != v ? 0.f : one);
                    }
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
            auto read = [&](int i, int pl, u32x4 (&va)[PARTS], u32x4 (&vb)[PARTS][2]) __attribute__((always_inline)) {
                const int off = pt[2 * i];
                va[pl] = *reinterpret_cast<const u32x4 *>(pa + i * 1024 + pl * a_part);
#pragma unroll
                for (int j = 0; j < 2; ++j) vb[pl][j] = *reinterpret_cast<const u32x4 *>(pb + col_cell[j] + off + pl * b_part);
            };
            auto product = [&](u32x4 a, u32x4 b, f32x16 &d) __attribute__((always_inline)) {
                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), d, 0, 0, 0);
            };
            if constexpr (F32 && FIRST == kSplit) {
                for (int i = wr; i < p.pairs; i += 2) {
                    u32x4 va[PARTS], vb[PARTS][2];
#pragma unroll
                    for (int pl = 0; pl < PARTS; ++pl) read(i, pl, va, vb);
                    constexpr int PL_A[6] = {0, 2, 1, 1, 0, 0}, PL_B[6] = {0, 0, 1, 0, 1, 2};
#pragma unroll
                    for (int m = 0; m < 6; ++m)
#pragma unroll
                        for (int j = 0; j < 2; ++j) product(va[PL_A[m] % PARTS], vb[PL_B[m] % PARTS][j], m == 0 ? acc[j] : low[j]);
                }
            } else if constexpr (F32 && FIRST == kPlain) {
#pragma unroll 1
                for (int i = wr; i < p.pairs; i += 2) {
                    u32x4 va[PARTS], vb[PARTS][2];
#pragma unroll
                    for (int pl = 0; pl < 2; ++pl) read(i, pl % PARTS, va, vb);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(va[(e >> 2) % PARTS][e & 3]),
                                                                          __uint_as_float(vb[(e >> 2) % PARTS][j][e & 3]), acc[j], 0, 0, 0);
                }
            } else {
                for (int i = wr; i < p.pairs; i += 2) {
                    u32x4 va[PARTS], vb[PARTS][2];
                    read(i, 0, va, vb);
#pragma unroll
                    for (int j = 0; j < 2; ++j) product(va[0], vb[0][j], acc[j]);
                }
            }
            if (!early) stage();
            if (last) { g = 0; ++c; } else ++g;
            __syncthreads();
        }
    };
    // the waves of a pair give each other one of the two tiles
    auto halves = [&](float (&y)[16]) __attribute__((always_inline)) {
        float *give = reinterpret_cast<float *>(lds) + wave * 1024 + lane, *take = reinterpret_cast<float *>(lds) + (wave ^ 4) * 1024 + lane;
#pragma unroll
        for (int e = 0; e < 16; ++e) give[64 * e] = wr ? acc[0][e] : acc[1][e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16; ++e) y[e] = (wr ? acc[1][e] : acc[0][e]) + take[64 * e];
    };
    typedef std::integral_constant<int, kSplit> Split;
    typedef std::integral_constant<int, kPlain> Plain;
    typedef std::integral_constant<int, kFinite> Other;
    float y[16];
    // (Only split operands reach so far.  A word for each of the two ways: a wave may begin the second while others read the first's.)
    int &flag = *reinterpret_cast<int *>(lds + kFewLds - (AGAIN ? 12 : 16));
    if constexpr (!AGAIN) {
        if (!F32) flag = 0;
        pass(Split{});
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
            if (__builtin_expect(__syncthreads_or((rest & 0xFFFFu) != 0 || !(not_finite == 0.f) || least < ((127u - 104u) << 24) - 1u), 0)) return true;
        } else {
            float sums[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) sums[e & 3] = fmaf(acc[j][e], 0.f, sums[e & 3]);
            if (!(sums[0] + sums[1] + (sums[2] + sums[3]) == 0.f)) flag = 1;
            __syncthreads();
            if (__builtin_expect(flag, 0)) return true;
        }
        halves(y);
    } else {
        mode = F32 ? kPlain : kFinite;
        flag = 0;
        if constexpr (F32) {
            pass(Plain{});
            halves(y);
            mode = kSigns;
        }
        float sign[16];
#pragma unroll 1
        for (; mode <= kNumber; ++mode) {
            if (mode == kSigns) {
                if (odd) flag = 1;
                __syncthreads();
                if (!__builtin_amdgcn_readfirstlane(flag)) break;
            }
            __syncthreads();
            pass(Other{});
            float z[16];
            halves(z);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if (mode == kFinite) y[e] = z[e];
                else if (mode == kSigns) sign[e] = z[e];
                else if (z[e] != 0.f) y[e] = fabsf(sign[e]) == z[e] ? y[e] + copysignf(__builtin_inff(), sign[e]) : __builtin_nanf("");
            }
        }
    }

    if (n < 0) return false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = 8 * q + 4 * lhi;
        if (F32 && p.vsw % 4 == 0) {   // four adjacent pixels
            uint32_t c, a, ah, aw;
            p.div_block.divmod((uint32_t)m, c, a);
            p.div_vsw.divmod(a, ah, aw);
            const int h = h0 + (int)ah, w = w0 + (int)aw;
            if ((int)c >= p.C || (unsigned)h >= (unsigned)p.H) continue;
            const uint32_t off = 4u * (uint32_t)(((n * p.C + (int)c) * p.H + h) * p.W + w);
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
    return false;
}

struct FewWords { uint32_t w[sizeof(FewParams) / 4]; };
// The kernel's parameters, read again
__device__ __forceinline__ FewParams few_args()
{
    typedef const __attribute__((address_space(4))) uint32_t *Words;
    Words from = (Words)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(from));
    FewWords t;
#pragma unroll
    for (size_t i = 0; i < sizeof(FewParams) / 4; ++i) t.w[i] = from[i];
    return __builtin_bit_cast(FewParams, t);
}

template <class E>
__global__ __launch_bounds__(512, 2) void conv_few_kernel(FewParams p)
{
    __shared__ __attribute__((aligned(16))) char lds[kFewLds];
    __shared__ int tab[kFewTaps];
    const int j0 = (int)xcd_order(blockIdx.x, gridDim.x) * kFewN;
    // The parameters in registers one by one: as they are loaded, sixteen at a time, they are also kept and spilled sixteen at a time.
    FewWords t = __builtin_bit_cast(FewWords, p);
#pragma unroll
    for (uint32_t &w : t.w) {
        uint32_t own;
        asm volatile("s_mov_b32 %0, %1" : "=s"(own) : "s"(w));
        w = own;
    }
    FewParams q = __builtin_bit_cast(FewParams, t);
    q.in = p.in; q.w = p.w; q.out = p.out;
    if (__builtin_expect(!few_tile<E, false>(q, j0, lds, tab), 1)) return;
    int again = j0;
    asm volatile("" : "+s"(again));
    few_tile<E, true>(few_args(), again, lds, tab);
}

}  // namespace ucd
