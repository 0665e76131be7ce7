// fp32 tile GEMM on the bf16 matrix pipe (gfx950).
//
// The fp32 matrix instructions run at the rate of the vector unit and stall it; the bf16 ones run 16 times
// as fast and beside it.  An fp32 value is the sum of three bf16 values (8 + 8 + 8 significant bits, each
// part rounded to nearest), x = h + m + l, and
//     x*y = hh' + (hm' + mh') + (mm' + hl' + lh') + (terms below 2^-24 of x*y, left out):
// six v_mfma_f32_32x32x16_bf16 cover 16 reduction rows in 192 cycles where the fp32 pipe takes 512.  Every
// product is exact in fp32 and accumulation is fp32.
//
// Error.  hh' has an accumulator of its own; the five small products share a second one that is added at the
// end.  The large accumulator is then rounded once per 16 reduction rows instead of once per two, which more
// than pays for the terms left out (relative L2 error against fp64, 256 x 256 x 1152, ReLU activations times
// normal weights: 1.5e-7; one accumulator for all six 4.9e-7; fp32 instructions 4.2e-7.  16384 rows: 7.2e-7 /
// 1.9e-6 / 1.6e-6).  Splitting by truncation instead of rounding is biased (1.8e-5 on positive operands).
//
// Range.  With all three parts rounded to nearest, x = h + m + l exactly (the last remainder has at most 7 bits)
// unless x lies so low (below 2^-102) that the remainder ends under bf16's smallest step, 2^-133, and that can be seen
// in it: its low 16 bits are no longer zero.  Those bits are collected while the operands are split (one v_or3 per two
// values).  An infinity, or a value that rounds to one in bf16, splits into inf - inf and leaves sums that are not
// finite; and sums below 2^-104 may have lost products below fp32's range.  A workgroup that finds any of the three
// after its last step computes its tile again with the fp32 instructions (fp32_tile), so that infinities, NaN and
// tiny operands give what they always gave, whatever they are multiplied with (such a tile costs both: 384 channels
// 3x3 13x13 b = 256, 560 us, all of it recomputed 1450).
#pragma once
#include "gemm_core.hpp"

namespace ucd {

// Two values -> their parts as bf16 pairs (first value in the low half).
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    // as an instruction of its own: the compiler turns the widening of one half into a second conversion
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// `rest` collects the bits of the last remainders: its low half is zero as long as every split is exact (see Range)
__device__ __forceinline__ void split_pair(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l, uint32_t &rest)
{
    h = pack_bf16(a, b);
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xFFFF0000u);
    m = pack_bf16(a, b);
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xFFFF0000u);
    // an instruction in its place: the compiler would keep the remainders in registers and combine them later
    asm("v_or3_b32 %0, %0, %1, %2" : "+v"(rest) : "v"(a), "v"(b));
    l = pack_bf16(a, b);
}

// LDS: three planes (h, m, l) per operand, each [2 halves of 8 rows][tile + pad] cells of 16 bytes: one cell is
// one lane's operand (lanes 0-31 rows 0-7 of the step, lanes 32-63 rows 8-15).
template <class T>
struct SplitTile {
    static constexpr int kCellPad = 8;  // shifts the second half's cells by 32 of the 64 banks
    static constexpr int PA = T::BM + kCellPad, PB = T::BN + kCellPad;
    static constexpr int A_BYTES = 3 * 2 * PA * 16, B_BYTES = 3 * 2 * PB * 16;
    static constexpr int BYTES = A_BYTES + B_BYTES;
    static constexpr int FP32_BYTES = T::LDS_FLOATS * 4;  // the same LDS serves fp32_tile
    static constexpr int BUF = BYTES;
};

// Loaders are templates of the tile extent; those of the eight-wave workgroups get the extent plus kWide.
constexpr int kWide = 4096;
constexpr int tile_extent(int td) { return td % kWide; }
constexpr int tile_threads(int td) { return td >= kWide ? 512 : 256; }
template <class T> constexpr int loader_tag_m() { return T::BM + (T::THREADS == 512 ? kWide : 0); }
template <class T> constexpr int loader_tag_n() { return T::BN + (T::THREADS == 512 ? kWide : 0); }

// ---- loaders: a thread holds NE consecutive reduction rows of one tile position -------------------------
// (kRows of them per position if it serves several): a run of an LDS cell, written in one piece.  erow0() is the
// first row, ecol(j) the position of run j, has_run(j) false where the tile has no such position; kLoad elements
// are loaded at a time; value(i) is element i as the product wants it.  `Fallback` is the loader that reads the same
// operand in fp32_tile.

// Dense matrix contiguous along the reduction index (KLane0's operand, row_stride 1): 16-byte loads, 8 rows per
// thread where that keeps at least three quarters of the threads busy, 4 otherwise.
// Rows past k_end read whatever lies there (the other operand's are zero; a product that is not finite for
// that reason goes the fp32 way like any other), dwords past the matrix read as zero.
template <int TDX>
struct CellK32T : NoSetup {
    static constexpr bool kBf16 = false, kSplit = true, kWideTiles = true;
    static constexpr int TD = tile_extent(TDX), NTHR = tile_threads(TDX);
    typedef KLane0T<TD, float, NTHR> Fallback;
    static std::string name() { return "CellK32"; }
    static constexpr int NE = TD * 2 * 4 >= NTHR * 3 ? 8 : 4;
    static constexpr int TPP = kBK / NE;  // threads per position
    struct Regs { float r[NE]; };
    const KLaneParams *p;
    __amdgpu_buffer_rsrc_t rsrc;
    int pos, row0;
    bool has;
    uint32_t voff;
    int k0_;

    __device__ __forceinline__ void init(const KLaneParams &prm, int origin, int)
    {
        p = &prm;
        rsrc = make_rsrc_bytes(prm.t, 0, prm.bytes);
        pos = threadIdx.x / TPP;
        row0 = NE * (threadIdx.x % TPP);
        has = TD * TPP >= NTHR || (int)threadIdx.x < TD * TPP;
        voff = has ? 4u * (uint32_t)(row0 + (origin + pos) * prm.col_stride) : kOob;
    }
    template <class Peer>
    __device__ __forceinline__ void prep(int k0, int, const Peer &) { k0_ = k0; }
    static constexpr int kLoad = 4;  // elements that one load fetches
    __device__ __forceinline__ void load(int i, Regs &g) const
    {
        const f32x4 v = buf_load4(rsrc, voff + 4u * (uint32_t)i, 4u * (uint32_t)k0_);
#pragma unroll
        for (int e = 0; e < 4; ++e) g.r[i + e] = v[e];
    }
    __device__ __forceinline__ float value(int i, const Regs &g) const { return g.r[i]; }
    static constexpr int kRows = NE;
    __device__ __forceinline__ int erow0() const { return row0; }
    __device__ __forceinline__ int ecol(int) const { return pos; }
    __device__ __forceinline__ bool has_run(int) const { return has; }
};

// The activation gather of GatherNLaneT with its row decode on the vector lanes: lane i decodes row i of a
// 64-row window every fourth step and the loads pick their row up with a read-lane (a 16-row step of this
// kernel is 768 matrix cycles per wave; the scalar decode of GatherNLaneT, on a unit that all waves of a CU share,
// takes longer).
template <int TDX, bool SMALL, bool NOMASK = false>
struct GatherCellT : GatherNLaneT<tile_extent(TDX), SMALL, float, NOMASK, tile_threads(TDX)> {
    typedef GatherNLaneT<tile_extent(TDX), SMALL, float, NOMASK, tile_threads(TDX)> Base;
    typedef Base Fallback;
    static std::string name() { return NOMASK ? "GatherCell<no padding>" : SMALL ? "GatherCell<taps<=31>" : "GatherCell<taps>31>"; }
    static constexpr bool kSplit = true;
    static constexpr bool kWideTiles = true;
    static constexpr int NE = Base::NE, kRows = NE, kLoad = 1;
    typedef typename Base::Regs Regs;
    int win_;  // first row of this thread's block, within the decoded window

    __device__ __forceinline__ void decode(int k0, int k_end)
    {
        const int kk = (k0 & ~63) + (int)(threadIdx.x & 63);
        uint32_t c, tap, tr, ts;
        this->p->taps.divmod((uint32_t)kk, c, tap);
        this->p->taps_w.divmod(tap, tr, ts);
        const bool dead = kk >= k_end;
        this->so_v = dead ? (NOMASK ? kOob : 0u)
                          : 4u * (uint32_t)(((int)c * this->p->Ht + this->p->dir * (int)tr) * this->p->Wt +
                                            this->p->dir * (int)ts + this->p->shift_row);
        this->bit_v = dead ? 31u : (SMALL ? tap : tr);
        this->ts_v = ts;
    }
    template <class Peer>
    __device__ __forceinline__ void setup(NoShared &, int k_begin, int k_end, const Peer &)
    {
        decode(k_begin, k_end);
        win_ = 0;
    }
    template <class Peer>
    __device__ __forceinline__ void prep(int k0, int k_end, const Peer &)
    {
        if ((k0 & 63) == 0) decode(k0, k_end);
        win_ = (k0 & 63) + NE * this->row0;
    }
    __device__ __forceinline__ void load(int i, Regs &g) const
    {
        const uint32_t so = (uint32_t)__builtin_amdgcn_readlane((int)this->so_v, win_ + i);
        uint32_t vo;
        if (NOMASK) {
            vo = this->voff;
        } else {
            const uint32_t bit = (uint32_t)__builtin_amdgcn_readlane((int)this->bit_v, win_ + i);
            if (SMALL) {
                vo = ((this->nmask >> bit) << 31) | this->voff;
            } else {
                const uint32_t ts = (uint32_t)__builtin_amdgcn_readlane((int)this->ts_v, win_ + i);
                vo = (((this->nmask >> bit) | (this->nmask_w >> ts)) << 31) | this->voff;
            }
        }
        g.r[i] = Elem<float>::load(this->rsrc, vo, so);
    }
    __device__ __forceinline__ float value(int i, const Regs &g) const { return g.r[i]; }
    __device__ __forceinline__ bool has_run(int) const { return true; }
    __device__ __forceinline__ int erow0() const { return NE * this->row0; }
};
template <int TD> using GatherCell = GatherCellT<TD, true>;
template <int TD> using GatherCellBig = GatherCellT<TD, false>;
template <int TD> using GatherCellFree = GatherCellT<TD, false, true>;

// BackwardFilter's operands: the reduction runs over output pixels, along which dy is contiguous in memory and x of a
// stride-1 layer is too (within an output row; where the output is as wide as the input also across rows).  A
// thread holds four consecutive rows (pixels) of TD*4/threads tile positions; four threads together read 64
// contiguous bytes.  Where a wave's four pixels are not adjacent in memory or its window touches the tensor's
// ends, it loads element by element.  What depends on the pixel alone is in an LDS table (QuadTable), refilled
// every kTabRows rows.
struct QuadTable {
    static constexpr int kCap = 128 + 3 * kBK;  // the pipeline looks three steps ahead
    uint32_t dy_off[kCap];  // byte offset of (n, a, b) in dy, kOob past the end
    uint32_t x_off[kCap];   // byte offset (signed) of the window origin in x
    uint32_t ok_a[kCap];    // MODE 1: bit r*S+s set = tap inside the image; MODE 2: bit r, of the window's rows
    uint32_t ok_b[kCap];    // MODE 2: bit s, of the window's columns
};

template <int TDX>
struct QuadBase {
    static constexpr bool kBf16 = false, kSplit = true, kWideTiles = true, kCellStore = false;
    static constexpr int TD = tile_extent(TDX), NTHR = tile_threads(TDX);
    static constexpr int CP = NTHR / 4;                    // positions per pass
    static constexpr int NQ = (TD + CP - 1) / CP, NE = 4 * NQ;
    // all of a thread's quads are loaded together, so that they can share one copy of their pixels' masks
    static constexpr int kLoad = NE, kRows = 4, kTabRows = 128;
    const KLaneParams *p;
    __amdgpu_buffer_rsrc_t rsrc;
    int q0, c0;  // first row of the thread's quad, first position

    __device__ __forceinline__ void init_quad(const KLaneParams &prm)
    {
        p = &prm;
        rsrc = make_rsrc_bytes(prm.t, 0, prm.bytes);
        q0 = 4 * (threadIdx.x & 3);
        c0 = threadIdx.x >> 2;
    }
    __device__ __forceinline__ bool has_run(int j) const { return TD % CP == 0 || c0 + CP * j < TD; }
    __device__ __forceinline__ int erow0() const { return q0; }
    __device__ __forceinline__ int ecol(int j) const { return c0 + CP * j; }
    // the four rows lie `bytes` apart
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
};

// MODE: 0 no padding, 1 at most 31 taps, 2 more.  STEP 1 or 2: the column stride that one or two 16-byte loads
// serve (others load element by element).
template <int TDX, int MODE, int STEP = 1>
struct QuadXT : QuadBase<TDX> {
    typedef QuadBase<TDX> Base;
    typedef QuadTable Shared;
    static constexpr bool kHasShared = true;
    static constexpr int NE = Base::NE, NQ = Base::NQ;
    static std::string name() { return std::string("PixelTab<x,quads") + (MODE == 0 ? ",no padding" : MODE == 2 ? ",taps>31" : "") + (STEP == 2 ? ",stride 2>" : ">"); }
    typedef typename std::conditional<MODE == 1, PixelTabX<Base::TD, float, Base::NTHR>,
                                      PixelKLane<Base::TD, true, float, MODE == 0, Base::NTHR>>::type Fallback;
    struct Regs { float r[NE]; uint32_t oka[MODE ? 4 : 1], okb[MODE == 2 ? 4 : 1]; };
    const QuadTable *tab;
    int k_begin_;
    uint32_t coff[NQ], tap[NQ];  // tap: MODE 1 bit r*S+s, MODE 2 r | s << 8
    uint32_t xo[4];
    int tab_row;
    bool adj;

    __device__ __forceinline__ void init(const KLaneParams &prm, int origin, int extent)
    {
        this->init_quad(prm);
        tab = nullptr;
        k_begin_ = 0;
        adj = false;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int j = origin + this->ecol(i);
            uint32_t c = 0, t = 0, r = 0, s = 0;
            if (j < extent) {
                prm.col_taps.divmod((uint32_t)j, c, t);
                prm.col_taps_w.divmod(t, r, s);
            }
            coff[i] = 4u * (uint32_t)(((int)c * prm.Ht + (int)r) * prm.Wt + (int)s);
            tap[i] = MODE == 1 ? t : r | (s << 8);
        }
    }
    template <class Peer>
    __device__ __forceinline__ void setup(QuadTable &sh, int k_begin, int k_end, const Peer &peer)
    {
        tab = &sh;
        k_begin_ = k_begin;
        const KLaneParams &q = *this->p;
#pragma unroll 1
        for (int e = threadIdx.x; e < QuadTable::kCap; e += Base::NTHR) {
            const int kk = k_begin + e;
            uint32_t n, rest, a, b;
            q.grid_hw.divmod((uint32_t)kk, n, rest);
            q.grid_w.divmod(rest, a, b);
            const int hb = (int)a * q.mul_h + q.add_h, wb = (int)b * q.mul_w + q.add_w;
            const bool live = kk < k_end;
            sh.dy_off[e] = live ? 4u * (uint32_t)((int)n * peer.p->n_stride + (int)rest) : kOob;
            sh.x_off[e] = MODE != 0 || live ? 4u * (uint32_t)((int)n * q.n_stride + hb * q.Wt + wb) : kOob;
            if constexpr (MODE != 0) {
                uint32_t okh = 0, okw = 0;
#pragma unroll 1
                for (int s = 0; s < q.n_tap_w; ++s)
                    if ((unsigned)(wb + s) < (unsigned)q.Wt) okw |= 1u << s;
                if constexpr (MODE == 1) {
#pragma unroll 1
                    for (int r = 0; r < q.n_tap_h; ++r)
                        if ((unsigned)(hb + r) < (unsigned)q.Ht) okh |= okw << (r * q.n_tap_w);
                } else {
#pragma unroll 1
                    for (int r = 0; r < q.n_tap_h; ++r)
                        if ((unsigned)(hb + r) < (unsigned)q.Ht) okh |= 1u << r;
                }
                sh.ok_a[e] = live ? okh : 0u;
                if constexpr (MODE == 2) sh.ok_b[e] = okw;
            }
        }
    }
    template <class Peer>
    __device__ __forceinline__ void prep(int k0, int, const Peer &)
    {
        tab_row = k0 - k_begin_ + this->q0;
        Base::read4(xo, tab->x_off + tab_row);
        adj = Base::apart(xo, 4u * (uint32_t)STEP);
    }
    // all ones where element e of quad i lies inside the image
    __device__ __forceinline__ int inside(int e, int i, const Regs &g) const
    {
        if constexpr (MODE == 1) return __builtin_amdgcn_sbfe((int)g.oka[e], tap[i], 1);
        if constexpr (MODE == 2)
            return __builtin_amdgcn_sbfe((int)g.oka[e], tap[i] & 0xffu, 1) & __builtin_amdgcn_sbfe((int)g.okb[e], tap[i] >> 8, 1);
        return -1;
    }
    __device__ __forceinline__ void load(int, Regs &g) const
    {
        if constexpr (MODE != 0) Base::read4(g.oka, tab->ok_a + tab_row);
        if constexpr (MODE == 2) Base::read4(g.okb, tab->ok_b + tab_row);
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const uint32_t start = xo[0] + coff[i];
            const bool whole = adj && start < 0x7FFFFF00u && start + 16u * STEP <= this->p->bytes;
            if (__builtin_amdgcn_ballot_w64(!whole) == 0) {
                const f32x4 v = buf_load4(this->rsrc, start);
                if constexpr (STEP == 1) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) g.r[4 * i + e] = v[e];
                } else {
                    const f32x4 u = buf_load4(this->rsrc, start + 16u);
                    g.r[4 * i] = v[0];
                    g.r[4 * i + 1] = v[2];
                    g.r[4 * i + 2] = u[0];
                    g.r[4 * i + 3] = u[2];
                }
            } else {  // only elements inside the image are dereferenced
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    g.r[4 * i + e] = Elem<float>::load(this->rsrc, inside(e, i, g) ? xo[e] + coff[i] : kOob, 0);
            }
        }
    }
    __device__ __forceinline__ float value(int k, const Regs &g) const
    {
        if constexpr (MODE == 0) return g.r[k];
        return __uint_as_float(__float_as_uint(g.r[k]) & (uint32_t)inside(k & 3, k >> 2, g));
    }
};
template <int TDX> using QuadX = QuadXT<TDX, 1>;
template <int TDX> using QuadXFree = QuadXT<TDX, 0>;
template <int TDX> using QuadXBig = QuadXT<TDX, 2>;
template <int TDX> using QuadX2 = QuadXT<TDX, 1, 2>;
template <int TDX> using QuadXFree2 = QuadXT<TDX, 0, 2>;
template <int TDX> using QuadXBig2 = QuadXT<TDX, 2, 2>;

// dy beside QuadXT<., MODE>, whose table it uses
template <int TDX, int MODE>
struct QuadDyT : QuadBase<TDX> {
    typedef QuadBase<TDX> Base;
    typedef NoShared Shared;
    static constexpr bool kHasShared = false;
    static constexpr int NE = Base::NE;
    struct Regs { float r[NE]; };
    static std::string name() { return "PixelTab<dy,quads>"; }
    typedef typename std::conditional<MODE == 1, PixelTabDy<Base::TD, float, Base::NTHR>,
                                      PixelKLane<Base::TD, false, float, false, Base::NTHR>>::type Fallback;
    uint32_t coff0, o[4];
    bool adj;

    __device__ __forceinline__ void init(const KLaneParams &prm, int origin, int)
    {
        this->init_quad(prm);
        coff0 = 4u * (uint32_t)((origin + this->c0) * prm.Ht * prm.Wt);
        adj = false;
    }
    template <class Peer>
    __device__ __forceinline__ void setup(NoShared &, int, int, const Peer &) {}
    template <class Peer>
    __device__ __forceinline__ void prep(int k0, int, const Peer &peer)
    {
        Base::read4(o, peer.tab->dy_off + (k0 - peer.k_begin_ + this->q0));
        adj = Base::apart(o, 4u);
    }
    __device__ __forceinline__ void load(int, Regs &g) const
    {
        const bool whole = __builtin_amdgcn_ballot_w64(!adj) == 0;
#pragma unroll
        for (int i = 0; i < Base::NQ; ++i) {
            const uint32_t so = 4u * (uint32_t)(Base::CP * i * this->p->Ht * this->p->Wt);
            if (whole) {
                const f32x4 v = buf_load4(this->rsrc, o[0] + coff0, so);
#pragma unroll
                for (int e = 0; e < 4; ++e) g.r[4 * i + e] = v[e];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) g.r[4 * i + e] = Elem<float>::load(this->rsrc, o[e] + coff0, so);
            }
        }
    }
    __device__ __forceinline__ float value(int k, const Regs &g) const { return g.r[k]; }
};
template <int TDX> using QuadDy = QuadDyT<TDX, 1>;
template <int TDX> using QuadDyFree = QuadDyT<TDX, 0>;

template <class L>
__host__ __device__ constexpr auto split_loader(int) -> decltype(L::kSplit) { return L::kSplit; }
template <class L>
__host__ __device__ constexpr bool split_loader(...) { return false; }
// One operand's way into LDS: its registers are split pair by pair (stage_pair); a run of kRows rows of one
// position that is complete is written to the step's planes, and registers that have been used are loaded again.
template <class L, int P, int BASE>
struct SplitStage {
    static constexpr int NE = L::NE, NP = NE / 2, RR = L::kRows;
    static_assert(RR == 8 || RR == 4, "runs of 4 or 8 rows");
    uint32_t part[3][RR / 2];
    uint32_t rest = 0;

    __device__ __forceinline__ void stage_pair(char *buf, int q, const L &ld, const typename L::Regs &g)
    {
        const int k = q % (RR / 2);
        split_pair(ld.value(2 * q, g), ld.value(2 * q + 1, g), part[0][k], part[1][k], part[2][k], rest);
        if (k + 1 < RR / 2) return;
        const int j = q / (RR / 2), row = ld.erow0();
        if (!ld.has_run(j)) return;
        char *dst = buf + BASE + (((row >> 3) * P + ld.ecol(j)) * 16 + (row & 7) * 2);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
            if constexpr (RR == 8) {
                const u32x4 v = {part[pl][0], part[pl][1], part[pl][2], part[pl][3]};
                *reinterpret_cast<u32x4 *>(dst + pl * 2 * P * 16) = v;
            } else {
                const u32x2 v = {part[pl][0], part[pl][1]};
                *reinterpret_cast<u32x2 *>(dst + pl * 2 * P * 16) = v;
            }
        }
    }
    // the loads whose registers pair q was the last to use
    __device__ __forceinline__ void reload_pair(int q, const L &ld, typename L::Regs &g)
    {
        if (L::kLoad == 1) {
            ld.load(2 * q, g);
            ld.load(2 * q + 1, g);
        } else if ((2 * q + 2) % L::kLoad == 0) {
            ld.load(2 * q + 2 - L::kLoad, g);
        }
    }
};

template <class T, class ALoader, class BLoader, class Epi, class AParams, class BParams>
__global__ __launch_bounds__(T::THREADS, 2) void gemm_kernel_split(AParams pa, BParams pb, typename Epi::Params pe,
                                                                  int M, int N, int Kd, int k_chunk, int tiles_m,
                                                                  int tiles_n, TailSplit tail)
{
    typedef SplitTile<T> H;
    typedef typename ALoader::Fallback FA;
    typedef typename BLoader::Fallback FB;
    __shared__ __attribute__((aligned(16))) char lds[3][H::BUF];
    static_assert(2 * H::FP32_BYTES + sizeof(typename FA::Shared) + sizeof(typename FB::Shared) <= 3 * H::BUF, "fp32_tile's LDS");
    __shared__ __attribute__((aligned(16))) typename ALoader::Shared sha;
    __shared__ __attribute__((aligned(16))) typename BLoader::Shared shb;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm0 = (wave % T::WAVES_M) * (T::WM * 32);
    const int wn0 = (wave / T::WAVES_M) * (T::WN * 32);
    const int l32 = lane & 31, lhi = lane >> 5;

    WorkItem wi;
    int tail_it = 0, tail_end = 0;
    const int whole_tiles = (Epi::kCanAdd && tail.tiles > 0) ? tiles_m * tiles_n - tail.tiles : 0;
    const bool tail_wg = Epi::kCanAdd && tail.tiles > 0 && (int)blockIdx.x >= whole_tiles;
    if (tail_wg) {
        const int r = (int)blockIdx.x - whole_tiles, steps = tail.tiles * tail.ksteps;
        tail_it = (int)((long)r * steps / tail.wgs);
        tail_end = (int)((long)(r + 1) * steps / tail.wgs);
        if (!next_tail_item<T>(wi, tail_it, tail_end, whole_tiles, tail.ksteps, tiles_m, Kd)) return;
    } else {
        wi = work_item<T>(Kd, k_chunk, tiles_m, tiles_n, whole_tiles);
        if constexpr (per_split<Epi>(0)) pe.out += (long)wi.split * pe.plane;
    }
    for (;;) {
        const int m0 = wi.m0, n0 = wi.n0, k_begin = wi.k_begin, k_end = wi.k_end;
        const bool accumulate = wi.accumulate;
        constexpr int WM = T::WM, WN = T::WN, NT = WM * WN;

        ALoader la;
        BLoader lb;
        la.init(pa, m0, M);
        lb.init(pb, n0, N);
        la.setup(sha, k_begin, k_end, lb);
        lb.setup(shb, k_begin, k_end, la);
        if constexpr (ALoader::kHasShared || BLoader::kHasShared) __syncthreads();

        f32x16 acc[WM][WN], low[WM][WN];
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.f;

        typedef SplitStage<ALoader, H::PA, 0> StageA;
        typedef SplitStage<BLoader, H::PB, H::A_BYTES> StageB;
        StageA sa;
        StageB sb;
        constexpr int NA = ALoader::NE, NB = BLoader::NE, NPA = StageA::NP, NPB = StageB::NP, NP = NPA + NPB;

        // Three LDS buffers: during step s the registers hold tile s+2 (loaded during step s-1), are split into
        // the buffer that tile s-1 has left and reloaded with tile s+3, while tile s+1 is complete already, so
        // that the first operands of the next step are read ahead of the barrier.
        typename ALoader::Regs ra;
        typename BLoader::Regs rb;
        {
            typename ALoader::Regs ra1;
            typename BLoader::Regs rb1;
            auto fetch = [&](int k0, typename ALoader::Regs &xa, typename BLoader::Regs &xb) __attribute__((always_inline)) {
                la.prep(k0, k_end, lb);
                lb.prep(k0, k_end, la);
#pragma unroll
                for (int i = 0; i < NA; i += ALoader::kLoad) la.load(i, xa);
#pragma unroll
                for (int i = 0; i < NB; i += BLoader::kLoad) lb.load(i, xb);
            };
            auto stage = [&](char *dst, const typename ALoader::Regs &xa, const typename BLoader::Regs &xb) __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < NPA; ++q) sa.stage_pair(dst, q, la, xa);
#pragma unroll
                for (int q = 0; q < NPB; ++q) sb.stage_pair(dst, q, lb, xb);
            };
            fetch(k_begin, ra, rb);
            fetch(k_begin + kBK, ra1, rb1);
            stage(lds[0], ra, rb);
            fetch(k_begin + 2 * kBK, ra, rb);
            stage(lds[1], ra1, rb1);
        }
        __syncthreads();

        bf16x8 a[3][WM], b[3][WN];
        auto read_plane = [&](const char *src, int pl) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < WM; ++i)
                a[pl][i] = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const u32x4 *>(src + ((pl * 2 + lhi) * H::PA + wm0 + 32 * i + l32) * 16));
#pragma unroll
            for (int j = 0; j < WN; ++j)
                b[pl][j] = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const u32x4 *>(src + H::A_BYTES +
                                                             ((pl * 2 + lhi) * H::PB + wn0 + 32 * j + l32) * 16));
        };
        read_plane(lds[0], 1);
        int o_cur = 0, o_nxt = H::BUF, o_wr = 2 * H::BUF;
        for (int k0 = k_begin; k0 < k_end; k0 += kBK) {
            if constexpr (ALoader::kHasShared || BLoader::kHasShared) {
                // the pixel table holds kTabRows rows plus the three tiles of lookahead
                if (k0 != k_begin && ((k0 - k_begin) & (BLoader::kTabRows - 1)) == 0) {
                    __syncthreads();
                    la.setup(sha, k0, k_end, lb);
                    lb.setup(shb, k0, k_end, la);
                    __syncthreads();
                }
            }
            char *base = &lds[0][0];
            read_plane(base + o_cur, 0);
            __builtin_amdgcn_sched_barrier(0);
            la.prep(k0 + 3 * kBK, k_end, lb);
            lb.prep(k0 + 3 * kBK, k_end, la);
            // six groups of one MFMA per 32x32 tile, a sixth of the staging behind each: mm' (read ahead), hm', mh',
            // hh' (its own accumulator), hl', lh'
            auto group = [&](auto gc) __attribute__((always_inline)) {
                constexpr int g = gc;
                constexpr int PL_A[6] = {1, 0, 1, 0, 0, 2}, PL_B[6] = {1, 1, 0, 0, 2, 0};
#pragma unroll
                for (int mi = 0; mi < WM; ++mi)
#pragma unroll
                    for (int mj = 0; mj < WN; ++mj) {
                        f32x16 &d = g == 3 ? acc[mi][mj] : low[mi][mj];
                        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PL_A[g]][mi], b[PL_B[g]][mj], d, 0, 0, 0);
                    }
                if (g == 1) read_plane(base + o_cur, 2);
                if (g == 3) read_plane(base + o_nxt, 1);
#pragma unroll
                for (int pr = 0; pr < NP; ++pr)
                    if (pr * 6 / NP == g) {
                        if (pr < NPA) {
                            sa.stage_pair(base + o_wr, pr, la, ra);
                            sa.reload_pair(pr, la, ra);
                        } else {
                            sb.stage_pair(base + o_wr, pr - NPA, lb, rb);
                            sb.reload_pair(pr - NPA, lb, rb);
                        }
                    }
                __builtin_amdgcn_sched_barrier(0);
            };
            static_for<6>(group);
            __syncthreads();
            const int t = o_cur;
            o_cur = o_nxt;
            o_nxt = o_wr;
            o_wr = t;
        }

        bool redo = ((sa.rest | sb.rest) & 0xFFFFu) != 0;
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    acc[i][j][v] += low[i][j][v];
                    // NaN, infinity or denormal; denormal after scaling by 2^-22
                    redo |= __builtin_amdgcn_classf(acc[i][j][v], 0x297) |
                            __builtin_amdgcn_classf(acc[i][j][v] * 0x1p-22f, 0x090);
                }
        if (__syncthreads_or(redo))
            fp32_tile<T, FA, FB, false>(pa, pb, reinterpret_cast<float(&)[2][T::LDS_FLOATS]>(lds),
                                        reinterpret_cast<typename FA::Shared &>(lds[0][2 * H::FP32_BYTES]),
                                        reinterpret_cast<typename FB::Shared &>(lds[0][2 * H::FP32_BYTES]), m0, M, n0, N,
                                        k_begin, k_end, wm0, wn0, l32, lhi, acc);
        write_tile<T, Epi, false>(pe, acc, M, N, m0, n0, wm0, wn0, l32, lhi, accumulate);
        if (!tail_wg || !next_tail_item<T>(wi, tail_it, tail_end, whole_tiles, tail.ksteps, tiles_m, Kd)) break;
    }
}

}  // namespace ucd
