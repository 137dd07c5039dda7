// Which rows belong to a tensor: host and device code.
#pragma once
#include <cstdint>

namespace fairkv {

// Rows row .. row + n - 1 of n_rows; n and n_rows are not negative.  The sum of two such numbers fits 64 unsigned bits and not 63.
constexpr bool rows_within(int64_t row, int32_t n, int64_t n_rows)
{
    return row >= 0 && static_cast<uint64_t>(row) + static_cast<uint32_t>(n) <= static_cast<uint64_t>(n_rows);
}
static_assert(rows_within(0, 0, 0) && rows_within(5, 7, 12) && rows_within(INT64_MAX - 1, 1, INT64_MAX), "up to the last row");
static_assert(!rows_within(-1, 1, 9) && !rows_within(5, 8, 12) && !rows_within(INT64_MAX, 1, INT64_MAX) && !rows_within(INT64_MAX, INT32_MAX, 6000) &&
                  !rows_within(INT64_MIN, INT32_MAX, 6000),
              "no further, also where the sum is more than an int64_t holds");

}  // namespace fairkv
