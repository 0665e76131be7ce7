// BackwardFilter with bf16 tensors: both operands in runs of four pixels.
//
// The reduction runs over output pixels, along which dy, and x of a layer of column stride 1, are contiguous in
// memory.  The element-wise loaders of gemm_kernel_bf16 spend a load, its address and mask arithmetic and a 2-byte LDS
// write on every element and synchronise every 16 rows.  Here a thread fetches four pixels of one tile position with
// one 8-byte load (16 threads together read 128 contiguous bytes), masks border taps on the packed pairs and writes
// half an LDS cell; a step is 64 rows, 16 MFMAs per 2 x 2 tile wave.  Where the four pixels of some thread of a wave are
// not evenly spaced in memory or a window touches the tensor's ends, the wave loads element by element.  What depends on
// the pixel alone comes from an LDS table, refilled every kTabRows rows.
// Measured (us, gemm_kernel_bf16 / this; b = 256 unless said): 256 channels 3x3 14x14 158 / 128 (461 TFLOP/s), 64
// channels 3x3 56x56 225 / 190, 1x1 1024 -> 256 14x14 109 / 67, 1x1/2 256 -> 512 56x56 b = 128 169 / 107, 1x1
// 128 -> 512 28x28 b = 128 68 / 52, 1x1 352 -> 128 32x32 b = 64 57 / 38, 7x7/2 3 -> 64 224x224 b = 128 224 / 202.  Bound
// by the vector work beside the MFMAs (masks, table reads) and by the LDS writes.  dw's error against 64 bits is smaller
// on all of them (256 channels: 2.3e-7 / 2.0e-7).
#pragma once
#include "gemm_core.hpp"

namespace ucd {

constexpr int kQuadBK = 64;

struct PixelQuadTable {
    static constexpr int kTabRows = 256, kCap = kTabRows + 2 * kQuadBK;  // the pipeline looks two steps ahead
    uint32_t dy_off[kCap];  // byte offset of (n, a, b) in dy, kOob past the end
    uint32_t x_off[kCap];   // byte offset (signed) of the window origin in x
    uint32_t ok_a[kCap];    // MODE 1: bit r*S+s set = tap inside the image; MODE 2: bit r, of the window's rows
    uint32_t ok_b[kCap];    // MODE 2: bit s, of the window's columns
};

template <class T>
struct QuadTile {
    // plane stride = 8 dwords modulo the 64 banks: the 16 half cells of a tile position fall into different ones
    static constexpr int PA = (T::BM + 15) / 16 * 16 + 2, PB = (T::BN + 15) / 16 * 16 + 2;
    static constexpr int A_BYTES = (kQuadBK / 8) * PA * 16, B_BYTES = (kQuadBK / 8) * PB * 16;
};

template <int TD_>
struct QuadHalf {
    static constexpr bool kBf16 = true, kQuads = true, kCellStore = false;
    static constexpr int TD = TD_, NP = TD / 16;   // positions per thread
    const KLaneParams *p;
    __amdgpu_buffer_rsrc_t rsrc;
    int q, c0;   // the thread's rows 4q .. 4q+3 of the step, its first position

    __device__ __forceinline__ void init_quad(const KLaneParams &prm)
    {
        p = &prm;
        rsrc = make_rsrc_bytes(prm.t, 0, prm.bytes);
        q = threadIdx.x & 15;
        c0 = threadIdx.x >> 4;
    }
    static __device__ __forceinline__ bool apart(const uint32_t (&o)[4], uint32_t bytes)
    {
        return (((o[1] - o[0]) ^ bytes) | ((o[2] - o[1]) ^ bytes) | ((o[3] - o[2]) ^ bytes)) == 0;
    }
    static __device__ __forceinline__ void read4(uint32_t (&d)[4], const uint32_t *src)
    {
        const u32x4 v = *reinterpret_cast<const u32x4 *>(src);
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = v[e];
    }
    __device__ __forceinline__ uint32_t load1(uint32_t vo, uint32_t so) const
    {
        return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsrc, (int)vo, (int)so, 0);
    }
    template <int P>
    __device__ __forceinline__ void put(char *tile, int i, u32x2 v) const
    {
        *reinterpret_cast<u32x2 *>(tile + ((q >> 1) * P + c0 + 16 * i) * 16 + (q & 1) * 8) = v;
    }
};

// MODE: 0 no padding, 1 at most 31 taps, 2 more.  STEP: column stride 1 or 2 (others go element by element).
template <int TD, int MODE, int STEP>
struct QuadHalfX : QuadHalf<TD> {
    typedef QuadHalf<TD> Base;
    typedef PixelQuadTable Shared;
    static constexpr int NP = Base::NP;
    static std::string name()
    {
        return std::string("PixelTab<x,quads") + (MODE == 0 ? ",no padding" : MODE == 2 ? ",taps>31" : "") +
               (STEP == 2 ? ",stride 2>" : ">") + "/bf16";
    }
    struct Regs { u32x2 d[NP]; uint32_t oka[MODE ? 4 : 1], okb[MODE == 2 ? 4 : 1]; };
    const PixelQuadTable *tab;
    int k_begin_;
    uint32_t coff[NP], tap[NP];   // tap: MODE 1 bit r*S+s, MODE 2 r | s << 8

    __device__ __forceinline__ void init(const KLaneParams &prm, int origin, int extent)
    {
        this->init_quad(prm);
        tab = nullptr;
        k_begin_ = 0;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int j = origin + this->c0 + 16 * i;
            uint32_t c = 0, t = 0, r = 0, s = 0;
            if (j < extent) {
                prm.col_taps.divmod((uint32_t)j, c, t);
                prm.col_taps_w.divmod(t, r, s);
            }
            coff[i] = 2u * (uint32_t)(((int)c * prm.Ht + (int)r) * prm.Wt + (int)s);
            tap[i] = MODE == 1 ? t : r | (s << 8);
        }
    }
    template <class Peer>
    __device__ __forceinline__ void setup(PixelQuadTable &sh, int k_begin, int k_end, const Peer &peer)
    {
        tab = &sh;
        k_begin_ = k_begin;
        const KLaneParams &g = *this->p;
#pragma unroll 1
        for (int e = threadIdx.x; e < PixelQuadTable::kCap; e += kThreads) {
            const int kk = k_begin + e;
            if (kk >= k_end) {
                sh.dy_off[e] = sh.x_off[e] = kOob;
                if constexpr (MODE != 0) sh.ok_a[e] = 0u;
                if constexpr (MODE == 2) sh.ok_b[e] = 0u;
                continue;
            }
            uint32_t n, rest, a, b;
            g.grid_hw.divmod((uint32_t)kk, n, rest);
            g.grid_w.divmod(rest, a, b);
            const int hb = (int)a * g.mul_h + g.add_h, wb = (int)b * g.mul_w + g.add_w;
            sh.dy_off[e] = 2u * (uint32_t)((int)n * peer.p->n_stride + (int)rest);
            sh.x_off[e] = 2u * (uint32_t)((int)n * g.n_stride + hb * g.Wt + wb);
            if constexpr (MODE != 0) {
                uint32_t okh = 0, okw = 0;
#pragma unroll 1
                for (int s = 0; s < g.n_tap_w; ++s)
                    if ((unsigned)(wb + s) < (unsigned)g.Wt) okw |= 1u << s;
#pragma unroll 1
                for (int r = 0; r < g.n_tap_h; ++r)
                    if ((unsigned)(hb + r) < (unsigned)g.Ht) okh |= MODE == 1 ? okw << (r * g.n_tap_w) : 1u << r;
                sh.ok_a[e] = okh;
                if constexpr (MODE == 2) sh.ok_b[e] = okw;
            }
        }
    }
    // all ones where element e of position i lies inside the image
    __device__ __forceinline__ uint32_t inside(int e, int i, const Regs &r) const
    {
        if constexpr (MODE == 1) return (uint32_t)__builtin_amdgcn_sbfe((int)r.oka[e], tap[i], 1);
        if constexpr (MODE == 2)
            return (uint32_t)(__builtin_amdgcn_sbfe((int)r.oka[e], tap[i] & 0xffu, 1) &
                              __builtin_amdgcn_sbfe((int)r.okb[e], tap[i] >> 8, 1));
        return 0xFFFFFFFFu;
    }
    template <class Peer>
    __device__ __forceinline__ void fetch(int k0, Regs &r, const Peer &) const
    {
        const int row = k0 - k_begin_ + 4 * this->q;
        uint32_t xo[4];
        Base::read4(xo, tab->x_off + row);
        if constexpr (MODE != 0) Base::read4(r.oka, tab->ok_a + row);
        if constexpr (MODE == 2) Base::read4(r.okb, tab->ok_b + row);
        bool whole = Base::apart(xo, 2u * (uint32_t)STEP);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const uint32_t start = xo[0] + coff[i];
            whole = whole && start < 0x7FFFFF00u && start + 8u * STEP <= this->p->bytes;
        }
        if (__builtin_amdgcn_ballot_w64(!whole) == 0) {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int start = (int)(xo[0] + coff[i]);
                r.d[i] = __builtin_amdgcn_raw_buffer_load_b64(this->rsrc, start, 0, 0);
                if constexpr (STEP == 2) {  // every other of eight
                    const u32x2 hi = __builtin_amdgcn_raw_buffer_load_b64(this->rsrc, start + 8, 0, 0);
                    r.d[i] = u32x2{__builtin_amdgcn_perm(r.d[i].y, r.d[i].x, 0x05040100u),
                                   __builtin_amdgcn_perm(hi.y, hi.x, 0x05040100u)};
                }
            }
        } else {  // only elements inside the image are dereferenced
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                uint32_t h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] = this->load1(inside(e, i, r) ? xo[e] + coff[i] : kOob, 0);
                r.d[i] = u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
            }
        }
    }
    template <int P>
    __device__ __forceinline__ void stage(char *tile, const Regs &r) const
    {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            u32x2 v = r.d[i];
            if constexpr (MODE != 0) {
                v.x &= (inside(0, i, r) & 0xFFFFu) | (inside(1, i, r) & 0xFFFF0000u);
                v.y &= (inside(2, i, r) & 0xFFFFu) | (inside(3, i, r) & 0xFFFF0000u);
            }
            this->template put<P>(tile, i, v);
        }
    }
};

// dy beside QuadHalfX, whose table it uses
template <int TD>
struct QuadHalfDy : QuadHalf<TD> {
    typedef QuadHalf<TD> Base;
    typedef NoShared Shared;
    static constexpr int NP = Base::NP;
    static std::string name() { return "PixelTab<dy,quads>/bf16"; }
    struct Regs { u32x2 d[NP]; };
    uint32_t coff0;

    __device__ __forceinline__ void init(const KLaneParams &prm, int origin, int)
    {
        this->init_quad(prm);
        coff0 = 2u * (uint32_t)((origin + this->c0) * prm.Ht * prm.Wt);
    }
    template <class Peer>
    __device__ __forceinline__ void fetch(int k0, Regs &r, const Peer &peer) const
    {
        uint32_t o[4];
        Base::read4(o, peer.tab->dy_off + (k0 - peer.k_begin_ + 4 * this->q));
        const bool whole = __builtin_amdgcn_ballot_w64(!Base::apart(o, 2u)) == 0;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const uint32_t so = 2u * (uint32_t)(16 * i * this->p->Ht * this->p->Wt);
            if (whole) {
                r.d[i] = __builtin_amdgcn_raw_buffer_load_b64(this->rsrc, (int)(o[0] + coff0), (int)so, 0);
            } else {
                uint32_t h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] = this->load1(o[e] + coff0, so);
                r.d[i] = u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
            }
        }
    }
    template <int P>
    __device__ __forceinline__ void stage(char *tile, const Regs &r) const
    {
#pragma unroll
        for (int i = 0; i < NP; ++i) this->template put<P>(tile, i, r.d[i]);
    }
};
template <int TD> using QuadHalfXFree = QuadHalfX<TD, 0, 1>;
template <int TD> using QuadHalfXFree2 = QuadHalfX<TD, 0, 2>;
template <int TD> using QuadHalfXTab = QuadHalfX<TD, 1, 1>;
template <int TD> using QuadHalfXBig = QuadHalfX<TD, 2, 1>;
template <int TD> using QuadHalfXBig2 = QuadHalfX<TD, 2, 2>;

template <class L>
__host__ __device__ constexpr auto quad_loader(int) -> decltype(L::kQuads) { return L::kQuads; }
template <class L>
__host__ __device__ constexpr bool quad_loader(...) { return false; }

// k_chunk must be a multiple of kQuadBK.
template <class T, class ALoader, class BLoader, class Epi, class AParams, class BParams>
__global__ __launch_bounds__(kThreads, 2) void gemm_kernel_bf16q(AParams pa, BParams pb, typename Epi::Params pe, int M,
                                                                  int N, int Kd, int k_chunk, int tiles_m, int tiles_n)
{
    typedef QuadTile<T> H;
    constexpr int KS = kQuadBK / kBK, WM = T::WM, WN = T::WN, NM = WM * WN;
    __shared__ __attribute__((aligned(16))) char lds[2][H::A_BYTES + H::B_BYTES];
    __shared__ __attribute__((aligned(16))) typename BLoader::Shared shb;

    const WorkItem wi = work_item<T>(Kd, k_chunk, tiles_m, tiles_n, 0);
    const int m0 = wi.m0, n0 = wi.n0, k_begin = wi.k_begin, k_end = wi.k_end;
    if constexpr (per_split<Epi>(0)) pe.out += (long)wi.split * pe.plane;

    ALoader la;
    BLoader lb;
    la.init(pa, m0, M);
    lb.init(pb, n0, N);
    lb.setup(shb, k_begin, k_end, la);
    __syncthreads();

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm0 = (wave % T::WAVES_M) * (WM * 32), wn0 = (wave / T::WAVES_M) * (WN * 32);
    const int l32 = lane & 31, lhi = lane >> 5;

    // two sums, of every other 16 rows: half as long a chain of roundings, which pays for the longer chunks
    f32x16 acc[WM][WN], acc2[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = acc2[i][j][v] = 0.f;

    typename ALoader::Regs ra;
    typename BLoader::Regs rb;
    la.fetch(k_begin, ra, lb);
    lb.fetch(k_begin, rb, la);
    la.template stage<H::PA>(lds[0], ra);
    lb.template stage<H::PB>(lds[0] + H::A_BYTES, rb);
    if (k_begin + kQuadBK < k_end) {
        la.fetch(k_begin + kQuadBK, ra, lb);
        lb.fetch(k_begin + kQuadBK, rb, la);
    }
    __syncthreads();

    int buf = 0;
    for (int k0 = k_begin; k0 < k_end; k0 += kQuadBK) {
        if (k0 != k_begin && ((k0 - k_begin) & (PixelQuadTable::kTabRows - 1)) == 0) {
            __syncthreads();
            lb.setup(shb, k0, k_end, la);
            __syncthreads();
        }
        const char *cur = lds[buf];
        char *nxt = lds[buf ^ 1];
        bf16x8 a[2][WM], b[2][WN];
        auto read_ops = [&](int u, int slot) __attribute__((always_inline)) {  // planes 2u (lanes 0-31) and 2u+1
#pragma unroll
            for (int i = 0; i < WM; ++i)
                a[slot][i] = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const u32x4 *>(cur + ((2 * u + lhi) * H::PA + wm0 + 32 * i + l32) * 16));
#pragma unroll
            for (int j = 0; j < WN; ++j)
                b[slot][j] = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const u32x4 *>(cur + H::A_BYTES + ((2 * u + lhi) * H::PB + wn0 + 32 * j + l32) * 16));
        };
        // behind the chunk's end nothing is loaded: a short chunk would spend a good part of its loads there (what the
        // registers hold then is staged once more and not multiplied)
        const bool more = k0 + 2 * kQuadBK < k_end;
        read_ops(0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            if (u + 1 < KS) read_ops(u + 1, (u + 1) & 1);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                f32x16 &sum = u & 1 ? acc2[m / WN][m % WN] : acc[m / WN][m % WN];
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u & 1][m / WN], b[u & 1][m % WN], sum, 0, 0, 0);
            }
            // the registers hold the next tile: to the other buffer, and loaded with the one after it
            if (u == 0) {
                la.template stage<H::PA>(nxt, ra);
                if (more) la.fetch(k0 + 2 * kQuadBK, ra, lb);
            }
            if (u == 1) {
                lb.template stage<H::PB>(nxt + H::A_BYTES, rb);
                if (more) lb.fetch(k0 + 2 * kQuadBK, rb, la);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        buf ^= 1;
    }
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) acc[i][j] += acc2[i][j];
    write_tile<T, Epi, false>(pe, acc, M, N, m0, n0, wm0, wn0, l32, lhi, false);
}

}  // namespace ucd
