// Staging modes of the patch kernels.
#pragma once
#include "s2_internal.h"

// Staging mode, all in pieces of four columns: kWide, rows of a multiple of four columns side by side and 32-bit offsets into a slice, so
// that no piece ends with its row; kNarrow, any rows, pieces at any alignment, and element by element where a piece ends with its row
// or its columns lie apart (classes of a finer grid); kRagged, kNarrow with channel counts that are not the kernel's.
// kPairs: kWide, where the owners are the two classes of a grid of twice the longitudes (an even number a class), so that four columns of a
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
    return b.c_own == 2 && b.nU % 2 == 0 ? kPairs : kWide;
}
// The list of workgroups for nbh slices: nullptr, the one where every wavefront has a patch of its own; or one of those for launches that their
// longest workgroup bounds.  By work (S2BandSide::Patches): parts of one patch up to 250, of two up to 400; a card is full at 400 to 600.
// float32, d = 32, forward / backward, us, unsplit, by halves, by quarters (work by halves, by quarters):
//   64 x 128: 1 slice (115, 155) 38 / 101, 28 / 64, 24 / 56;   2 (230, 310) 38 / 102, 28 / 69, 36 / 87;   4 (460, 620) 40 / 108, 44 / 110, 54 / 129
//   46 x 90: 2 slices 36 / 90, 31 / 69, 29 / 64;   8 38 / 96, 42 / 95, 60 / 129       181 x 360: 1 slice 74 / 192, 61 / 147, 68 / 159;   2 83 / 208, 98 / 243, 112 / 273
inline const S2BandSide::Patches::Split *s2_split_list(const S2BandSide::Patches &p, int nbh)
{
    if (s2_debug_flag(S2_DEBUG_OWN_PATCHES)) return nullptr;
    if (s2_debug_flag(S2_DEBUG_HALVES)) return &p.split[0];
    const double most[2] = {400.0, 250.0};
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
