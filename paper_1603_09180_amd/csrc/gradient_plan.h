// gradient_plan.h -- how many lines of an image a block of the gradient's LDS
// passes holds.  Host arithmetic, and the kernels' line length, in one place
// that needs no GPU to run.  Sides go up to 2^30, and four lines of such a side
// do not fit 32 bits: the host counts in 64.
#pragma once

#include <cstddef>
#include <cstdint>

namespace thin {

constexpr size_t kLdsBytes = 160 * 1024 - 1024;   // dynamic LDS a block may ask for

// Floats of one recursion's line in LDS: a multiple of 4, and an odd multiple,
// so that the lanes' 16-byte accesses spread over the banks.
template <typename I>
constexpr I chain_floats(I n)
{
    return 4 * (((n + 3) / 4) | 1);
}

// Floats of a column's four lines, and 4 more to spread the columns over the
// banks.
template <typename I>
constexpr I column_floats(I h)
{
    return 4 * chain_floats(h) + 4;
}

// Lines a block takes: as many blocks as compute units, or `waves` times that
// many where LDS holds no more lines (0: even that leaves lines over, and the
// passes from global memory run every line at once).
inline int lines_per_block(int64_t lines, int64_t floats, int64_t num_cus, int64_t waves)
{
    const int64_t fit = (int64_t)(kLdsBytes / sizeof(float)) / floats;
    const int64_t most = fit < 16 ? fit : 16;
    const int64_t want = (lines + num_cus - 1) / num_cus;
    if (most <= 0 || most * num_cus * waves < lines) return 0;
    return (int)(want < most ? want : most);
}

// Columns: one wave of blocks (1601x1536 in LDS 114 us a call, from global
// memory 183; a second wave gives it back, and the rows lose the sum that the
// LDS pass forms for them).
inline int columns_per_block(int64_t h, int64_t w, int64_t num_cus)
{
    return lines_per_block(w, column_floats<int64_t>(h), num_cus, 1);
}

// Rows: one wave (1792x1283 161 us, from global memory 192), and where a block
// holds four lines or fewer, so that a line's chain is longer than 2000 samples,
// two (512x5080 151 us and 259; 1024x5080 280 and 299, the third wave 414 and
// 353; shorter lines lose with the second: 1551x1600 192 and 185, 3878x640 302
// and 274).  After LDS columns (halves not set) the rows are short or few, and
// LDS is the faster up to all the waves there are (8192x150 189 us and 198).
inline int rows_per_block(int64_t h, int64_t w, int64_t num_cus, bool halves)
{
    const int64_t floats = 4 * chain_floats<int64_t>(w);
    const bool long_lines = 5 * floats * (int64_t)sizeof(float) > (int64_t)kLdsBytes;
    return lines_per_block(h, floats, num_cus, !halves ? 3 : long_lines ? 2 : 1);
}

}  // namespace thin
