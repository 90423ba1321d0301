// Staging modes of the patch kernels.
#pragma once
#include "s2_internal.h"

// Staging mode, all in pieces of four columns: kWide, rows of a multiple of four columns side by side and 32-bit offsets into a slice, so
// that no piece ends with its row; kNarrow, any rows, pieces at any alignment, and element by element where a piece ends with its row
// or its columns lie apart (classes of a finer grid); kRagged, kNarrow with channel counts that are not the kernel's.
// kPairs: kWide, where the owners are the two classes of a grid of twice the longitudes, so that four columns of a
// latitude are two owners of either.
// kHalves: kNarrow, rows of an even length side by side, whose pieces astride the end of a row are two pairs of columns.
// kColumns: kNarrow, where a wavefront owns 16 rows of one column (S2ColumnRow).
enum { kWide, kNarrow, kRagged, kPairs, kColumns, kHalves };
constexpr bool is_wide(int mode) { return mode == kWide || mode == kPairs; }
inline int s2_band_mode(const S2BandSide &b, int d, int e, size_t element)
{
    if (d != e || (d != 16 && d != 32 && d != 64)) return kRagged;
    const size_t slice = size_t(d) * b.nlat_walk * b.nU * b.c_walk * element;
    if (b.c_walk != b.patches.step || b.nU * b.patches.step % 2 != 0) return kNarrow;
    if (b.nU * b.patches.step % 4 != 0 || slice >= size_t(1) << 32) return kHalves;
    return b.c_own == 2 ? kPairs : kWide;      // (the walked grid is the coarser one: step 1, nU a multiple of four)
}
// The list of workgroups for nbh slices of d and e channels: nullptr, the one where every wavefront has a patch of its own; or one of those
// for launches that their longest workgroup bounds.  By work (S2BandSide::Patches): parts of one patch up to 250, of two up to 400.
// float32, d = 32, forward / backward, us, unsplit, by halves, by quarters (work by halves, by quarters):
//   64 x 128: 1 slice (113, 152) 38 / 101, 28 / 64, 24 / 56;   2 (226, 304) 38 / 102, 28 / 69, 36 / 87;   4 (451, 609) 40 / 108, 44 / 110, 54 / 129
//   46 x 90: 2 slices (122, 163) 36 / 90, 31 / 69, 29 / 64;   8 (488, 651) 38 / 96, 42 / 95, 60 / 129
//   181 x 360: 1 slice (357, 431) 74 / 192, 61 / 147, 68 / 159;   2 (715, 862) 83 / 208, 98 / 243, 112 / 273
// 119 grids of 24 to 181 latitudes, halves against unsplit, mean, at a work of 200-250, 300-350, 350-400 and from 400 on, forward:
//   float32 d = 16 0.75 0.84 0.94 1.09   d = 32 0.74 0.80 0.88 1.00   d = 64 0.81 0.90 0.96 1.06;   bf16 d = 16 0.81 0.83 0.84 0.91   d = 32 0.77 0.83 0.89 0.93
// bf16 of more than 32 channels: a part has twice the chunks a stage and a workgroup less on a compute unit than the unsplit kernel, and
// parts read a patch's surroundings twice.  With several slices in a die's L2 quarters pay up to 200, halves up to 325 on rows of a multiple of
// four (of 45 grids forward and 29 backward none slower than unsplit; from 350 on up to 1.18), on others up to 250 (47 and 42: up to 300 a few
// by 1.09 to 1.20); one slice as above.
// Owners that are classes of a finer grid lie close together and meet few chunks, so that more of a part is start and end.  Of 100 pairs, worst
// against unsplit of the forward and of the backward: float32 halves up to 275, quarters up to 200: 1.09 and 1.05 (up to 300 1.25 on odd
// rows, up to 400 1.38 and 1.13); bf16 up to 325 and 250: 1.08 and 1.08 (400: 1.22, 1.09).  bf16 of more than 32 channels gain 0.3 % on the
// query side and lose 1 % on the key side up to 200, then 5 to 50 %: unsplit.
inline const S2BandSide::Patches::Split *s2_split_list(const S2BandSide &b, int nbh, int d, int e, size_t element)
{
    const S2BandSide::Patches &p = b.patches;
    if (s2_debug_flag(S2_DEBUG_OWN_PATCHES)) return nullptr;
    if (s2_debug_flag(S2_DEBUG_HALVES)) return size_t(nbh) * p.split[0].n < size_t(1) << 24 ? &p.split[0] : nullptr;      // (2^32 threads)
    const bool classes = b.c_own > 1, bf16 = element == 2, broad16 = bf16 && (d > 32 || e > 32);
    if (classes && broad16) return nullptr;
    double most[2] = {400.0, 250.0};
    if (classes) {
        most[0] = bf16 ? 325.0 : 275.0;
        most[1] = bf16 ? 250.0 : 200.0;
    } else if (broad16 && nbh > 1) {
        most[0] = s2_band_mode(b, d, e, element) == kWide ? 325.0 : 250.0;
        most[1] = 200.0;
    }
    for (int i = 1; i >= 0; --i)
        if (p.split[i].work > 0.0 && nbh * p.split[i].work < most[i] && size_t(nbh) * p.split[i].n < size_t(1) << 20) return &p.split[i];
    return nullptr;
}
// f(set) with the launchers of a staging mode
template <template <int> class Set, class F>
void s2_by_band_mode(int mode, F &&f)
{
    if (mode == kWide) f(Set<kWide>());
    else if (mode == kNarrow) f(Set<kNarrow>());
    else if (mode == kRagged) f(Set<kRagged>());
    else if (mode == kHalves) f(Set<kHalves>());
    else f(Set<kPairs>());
}
