// Staging modes of the patch kernels.
#pragma once
#include <algorithm>

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
// The list of workgroups for nbh slices of d and e channels, forward or backward: nullptr, the one where every wavefront has a patch of its own; or one of those
// for launches that their longest workgroup bounds.  By work (S2BandSide::Patches): parts of one patch up to 250, of two up to 400
// (float32 of more than 32 channels 350, two workgroups on a compute unit: 59 x 116, theta 0.39, three slices, d = 64, work 396: 59 us, 70).
// float32, d = 32, forward / backward, us, unsplit, by halves, by quarters (work by halves, by quarters):
//   64 x 128: 1 slice (113, 152) 38 / 101, 28 / 64, 24 / 56;   2 (226, 304) 38 / 102, 28 / 69, 36 / 87;   4 (451, 609) 40 / 108, 44 / 110, 54 / 129
//   46 x 90: 2 slices (122, 163) 36 / 90, 31 / 69, 29 / 64;   8 (488, 651) 38 / 96, 42 / 95, 60 / 129
//   181 x 360: 1 slice (357, 431) 74 / 192, 61 / 147, 68 / 159;   2 (715, 862) 83 / 208, 98 / 243, 112 / 273
// 119 grids of 24 to 181 latitudes, halves against unsplit, mean, at a work of 200-250, 300-350, 350-400 and from 400 on, forward:
//   float32 d = 16 0.75 0.84 0.94 1.09   d = 32 0.74 0.80 0.88 1.00   d = 64 0.81 0.90 0.96 1.06;   bf16 d = 16 0.81 0.83 0.84 0.91   d = 32 0.77 0.83 0.89 0.93
// bf16 of more than 32 channels: a part has twice the chunks a stage and a workgroup less on a compute unit than the unsplit kernel, and
// parts read a patch's surroundings twice.  By the chunks of the heaviest workgroup, forward, 2500 launches, quarters against unsplit, mean (worst) at a work
// of 120-160, 160-200, 200-250, several slices:   rows of a multiple of four: 96-128 chunks 0.86 (0.94) 0.87 (0.87) 0.93 (0.97)
//   128-192 0.79 (0.84) 0.85 (0.95) 0.88 (1.02)   256-400 0.72 (0.77) 0.71 (0.81) 0.80 (0.96)     channels that are not the kernel's: 96-128 0.90 (0.96) 0.93 (1.05)
//   1.05 (1.30)   128-192 0.87 (1.14) 0.90 (1.20) 1.03 (1.19)   256-400 0.79 (0.94) 0.79 (1.15) 0.87 (1.16)
// halves at 200-250, 250-300, 300-350:   rows of a multiple of four 128-192 0.90 (1.07) 1.00 0.99 (1.20)   from 400 on 0.65 (0.71) 0.77 (0.86) 0.82 (1.03)
//   channels that are not the kernel's 128-192 0.94 (1.15) 0.96 (1.17) 1.09 (1.45)   from 400 on 0.69 (1.08) 0.75 (1.09) 0.89 (1.28)
// Owners that are classes of a finer grid lie close together and meet few chunks, so that more of a part is start and end.  Of 100 pairs, worst
// against unsplit of the forward and of the backward: float32 halves up to 275, quarters up to 200: 1.09 and 1.05 (up to 300 1.25 on odd
// rows, up to 400 1.38 and 1.13); bf16 up to 325 and 250: 1.08 and 1.08 (400: 1.22, 1.09).  bf16 of more than 32 channels gain 0.3 % on the
// query side and lose 1 % on the key side up to 200, then 5 to 50 %: unsplit.
// Short launches, of disks of a spacing or two: a part saves less than its start and end cost.  1800 launches of 16 to 181 latitudes, disks of 0.4 to
// 9 spacings, by the chunks of the heaviest workgroup, quarters against unsplit up to a work of 200, forward / backward, mean on equal grids:
//               16-24        24-32        32-40        40-48        48-56        56-64        64-80        80-96
//   f32 d = 16  0.99 / 1.00  0.98 / 0.99  1.00 / 0.91  1.00 / 0.91  0.99 / 0.86  0.99 / 0.82  0.99 / 0.76  0.93 / 0.79
//       d = 32  0.99 / 0.92  0.98 / 0.83  1.00 / 0.86  0.99 / 0.87  0.91 / 0.79  0.93 / 0.78  0.88 / 0.77  0.78 / 0.71
//       d = 64  0.97 / 0.86  0.91 / 0.86  0.98 / 0.88  0.93 / 0.86  0.97 / 0.91  0.92 / 0.82  0.89 / 0.81  0.90 / 0.82
//   bf16    16  1.00 / 1.01  1.00 / 0.99  0.99 / 0.99  0.97 / 0.98  1.00 / 0.92  0.99 / 0.97  0.99 / 0.92  0.98 / 0.86
//           32  1.01 / 1.03  1.01 / 1.02  1.00 / 0.95  0.99 / 0.92  1.01 / 0.96  0.99 / 0.85  0.97 / 0.84
//           64  1.14 / 1.19  1.07 / 1.16  1.05 / 1.02  1.05 / 1.03  1.00 / 0.95  1.00 / 0.95  1.00 / 0.99  0.96 / 0.95
// (single ones: 100 x 200, theta 0.016, bf16 d = 40, backward 19 us unsplit, 29 by halves).  Hence the fewest chunks below; and up to 100 chunks
// lines of 300 and 200 (58 x 117, theta 0.08, four slices, float32 d = 8, 68 chunks, work 376: forward 12 us, 15), owners of a finer grid 200 and
// 160 (113 x 226 -> 226 x 452, theta 0.018, one slice, float32 d = 16, 79 chunks, work 209: 14 us, 23).
// In all, more than 5 % above unsplit: bf16 of more than 32 channels 32 of 4400 forward and backward passes (with the first lines 661), others 15 of 2100 (51).
inline const S2BandSide::Patches::Split *s2_split_list(const S2BandSide &b, int nbh, int d, int e, size_t element, bool backward)
{
    const S2BandSide::Patches &p = b.patches;
    if (s2_debug_flag(S2_DEBUG_OWN_PATCHES)) return nullptr;
    for (int i = 0; i < 2; ++i)
        if (s2_debug_flag(i ? S2_DEBUG_QUARTERS : S2_DEBUG_HALVES)) return size_t(nbh) * p.split[i].n < size_t(1) << 24 ? &p.split[i] : nullptr;      // (2^32 threads)
    const bool classes = b.c_own > 1, bf16 = element == 2, broad16 = bf16 && (d > 32 || e > 32), wide = s2_band_mode(b, d, e, element) == kWide;
    if (classes && broad16) return nullptr;
    double most[2] = {!bf16 && (d > 32 || e > 32) ? 350.0 : 400.0, 250.0};
    if (classes) {
        most[0] = bf16 ? 325.0 : 275.0;
        most[1] = bf16 ? 250.0 : 200.0;
    } else if (broad16) {
        const bool is_long = p.heaviest >= 256;
        most[0] = wide ? is_long ? 400.0 : 300.0 : is_long ? 250.0 : 130.0;
        most[1] = wide ? is_long ? 300.0 : 200.0 : is_long ? 220.0 : 150.0;
    }
    const bool slim = d <= 16 && e <= 16;
    if (p.heaviest < (broad16 ? backward && wide ? 64 : 96 : bf16 || slim ? backward ? 32 : 64 : backward ? 20 : 48)) return nullptr;
    if (p.heaviest < 100 && !broad16) {
        most[0] = std::min(most[0], classes ? 200.0 : 300.0);
        most[1] = std::min(most[1], classes ? 160.0 : 200.0);
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
