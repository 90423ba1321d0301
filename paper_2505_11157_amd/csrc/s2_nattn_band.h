// Staging modes of the patch kernels.
#pragma once
#include "s2_internal.h"

// Staging mode, all in pieces of four columns: kWide, rows of a multiple of four columns side by side and 32-bit offsets into a slice, so
// that no piece ends with its row; kNarrow, any rows, pieces at any alignment, and element by element where a piece ends with its row
// or its columns lie apart (classes of a finer grid); kRagged, kNarrow with channel counts that are not the kernel's.
// kPairs: kWide, where the owners are the two classes of a grid of twice the longitudes (an even number a class), so that four columns of a
// latitude are two owners of either.
// kColumns: kNarrow, where a wavefront owns 16 rows of one column (S2ColumnRow).
enum { kWide, kNarrow, kRagged, kPairs, kColumns };
constexpr bool is_wide(int mode) { return mode == kWide || mode == kPairs; }
inline int s2_band_mode(const S2BandSide &b, int d, int e, size_t element)
{
    if (d != e || (d != 16 && d != 32 && d != 64)) return kRagged;
    const size_t slice = size_t(d) * b.nlat_walk * b.nU * b.c_walk * element;
    if (b.c_walk != b.patches.step || b.nU * b.patches.step % 4 != 0 || slice >= size_t(1) << 32) return kNarrow;
    return b.c_own == 2 && b.nU % 2 == 0 ? kPairs : kWide;
}
// f(set) with the launchers of a staging mode
template <template <int> class Set, class F>
void s2_by_band_mode(int mode, F &&f)
{
    if (mode == kWide) f(Set<kWide>());
    else if (mode == kNarrow) f(Set<kNarrow>());
    else if (mode == kRagged) f(Set<kRagged>());
    else f(Set<kPairs>());
}
