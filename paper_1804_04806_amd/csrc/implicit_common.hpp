// What the three implicit-GEMM operations share: reduction split counts and the rule for vector gathers.
#pragma once
#include <cstdlib>
#include <type_traits>

#include "gemm_launch.hpp"
#include "kernels.h"

namespace ucd {

// Split counts are chosen so that the workgroup count fills its rounds of 256 x resident workgroups: workgroups of one
// launch take equally long, and a last round that is nearly empty costs as much as a full one (fp32 kernel, measured:
// the time of a Forward launch is flat from 769 to 1024 tiles).  A CU holds four workgroups of the fp32 and bf16 Forward
// / BackwardData kernels and three of the BackwardFilter ones, by registers and LDS, and needs them all to keep its
// matrix pipes busy.  The split kernel's Forward launches use the same counts although two of its workgroups fit a CU (one
// of 128 x 256 tiles): over 144 deep layers (1 to 32 images of 7x7 to 28x28) none takes longer than the fp32 kernel
// with them and the mean is 1.04 times as fast.  The BackwardFilter kernels that read runs of pixels have counts of
// their own.
inline long slots_output() { return 4l * device_cus(); }
inline long slots_filter() { return 3l * device_cus(); }

inline double round_fill(long blocks, long slots)
{
    return (double)blocks / (double)((blocks + slots - 1) / slots * slots);
}

// Among split counts in [lo, hi], the one whose workgroup count fills its rounds best (ties: the
// one nearest to `want`).
inline int best_fill(long tiles, long want, long lo, long hi, long slots)
{
    if (lo < 1) lo = 1;
    if (hi < lo) hi = lo;
    long best = want < lo ? lo : (want > hi ? hi : want);
    double best_f = round_fill(tiles * best, slots);
    for (long c = lo; c <= hi; ++c) {
        const double f = round_fill(tiles * c, slots);
        const long dc = c > want ? c - want : want - c, db = best > want ? best - want : want - best;
        if (f > best_f + 1e-9 || (f > best_f - 1e-9 && dc < db)) { best = c; best_f = f; }
    }
    return (int)best;
}

// Forward / BackwardData write each output once, so normally one workgroup owns a whole
// reduction.  When the output has too few tiles to give every CU several workgroups (deep
// layers: many channels, few pixels), the reduction is split as well and the partial results meet
// through atomics in a zero-filled output.  Chunks keep at least 512 reduction rows (measured with the fp32 kernel).
inline int output_splits(int M, int N, int Kd, bool fp32_out)
{
    if (!fp32_out) return 1;  // bf16 outputs cannot be accumulated with atomics (nor may reproducible runs)
    const long tiles = pick_tile(M, N, true, 1 << 20).blocks(M, N, 1);  // tiles at the default shape
    if (tiles >= 768) return 1;  // three workgroups per CU already
    long want = (1536 + tiles - 1) / tiles;
    const long cap = Kd / 512;
    if (want > cap) want = cap;
    if (want < 2) return 1;
    return best_fill(tiles, want, want / 2 < 2 ? 2 : want / 2, want * 2 < cap ? want * 2 : cap, slots_output());
}

// bf16 tensors, stride-1 layers whose output rows are as wide as the input rows (so that, for every
// tap, neighbouring pixels of an image are neighbours in memory), filters of at most 31 taps: the
// activation operand is fetched four pixels per load (RunNLaneT).  Tile positions run over the
// images with their pixel count rounded up to 4.
inline bool vector_gather_applies(const Dims &d, int grid_w, int tensor_w)
{
    // UCD_BF16_ELEMENTWISE=1 keeps the element-wise kernel (for comparisons)
    static const bool off = [] { const char *e = std::getenv("UCD_BF16_ELEMENTWISE"); return e && e[0] == '1'; }();
    return !off && d.dtype == 1 && d.sh == 1 && d.sw == 1 && grid_w == tensor_w && d.R * d.S <= 31;
}

}  // namespace ucd
