// ppmlr_rows.hpp -- how the waves of the signal-speed kernels share the rows of
// zones along x: plain functions of sizes, the same on the host, in the kernels
// and in the CPU test of the split.
#pragma once

#if defined(__HIPCC__)
#define PPMLR_HD __host__ __device__
#else
#define PPMLR_HD
#endif

namespace ppmlr {

// The rows of a grid of nx zones along x among `waves` waves.  A wave takes a
// group of `per` rows, `lanes` lanes each, that far along x at a time (a
// column); with more waves than groups every group goes to `parts` waves,
// `width` columns each.  (A wave per group and all its columns was 60 us for
// 4000 x 1 x 1 zones, one wave over 63 columns in turn; with the columns dealt
// out 19 us.)
struct RowSplit {
    int shift, lanes, per, cols, groups, parts, width;      // lanes = 2^shift
    PPMLR_HD RowSplit(int nx, long long rows, int waves)
    {
        shift = 6;
        while (shift > 0 && (1 << (shift - 1)) >= nx) --shift;
        lanes = 1 << shift;
        per = 64 >> shift;
        cols = ((nx - 1) >> shift) + 1;
        groups = (int)((rows - 1) >> (6 - shift)) + 1;
        parts = width = 1;
        if (cols == 1) return;                               // (no divisions on the way to a short row)
        parts = waves / groups < cols ? waves / groups : cols;
        if (parts < 1) parts = 1;
        width = (cols - 1) / parts + 1;
    }
    PPMLR_HD unsigned units() const { return (unsigned)groups * (unsigned)parts; }   // at most the waves or groups
};

}  // namespace ppmlr
