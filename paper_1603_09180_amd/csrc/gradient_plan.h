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
// passes from global memory, which run every line at once, are faster: at 4000
// x 3000 six waves of column blocks and six of row blocks took 849 us, those
// 493).
inline int lines_per_block(int64_t lines, int64_t floats, int64_t num_cus, int64_t waves)
{
    const int64_t fit = (int64_t)(kLdsBytes / sizeof(float)) / floats;
    const int64_t most = fit < 16 ? fit : 16;
    const int64_t want = (lines + num_cus - 1) / num_cus;
    if (most <= 0 || most * num_cus * waves < lines) return 0;
    return (int)(want < most ? want : most);
}

// The column pass's and the row pass's lines per block.
inline int columns_per_block(int64_t h, int64_t w, int64_t num_cus)
{
    return lines_per_block(w, column_floats<int64_t>(h), num_cus, 1);
}
inline int rows_per_block(int64_t h, int64_t w, int64_t num_cus)
{
    return lines_per_block(h, 4 * chain_floats<int64_t>(w), num_cus, 3);
}

}  // namespace thin
