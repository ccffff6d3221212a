// Average and maximum pooling with the batch dealt out evenly (pool_rows_kernel): which rows a workgroup adds up for a
// sequence.  Host and device code, so that the arithmetic can be checked without a GPU.
#pragma once
#include <cstdint>

namespace egtp {

// A token index inside the batch.  Offsets are the caller's and may hold anything; differences are only taken of what this returns.
constexpr int inside_batch(int32_t token, int64_t T)
{
    return token < 0 ? 0 : (int64_t)token > T ? (int)T : token;
}

// Rows [begin, end) that a sequence from offset `first` to offset `last` has among the rows [lo, hi) of a batch of T; none where end <= begin.
struct RowRun {
    int begin, end;
};
constexpr RowRun dealt_rows(int lo, int hi, int32_t first, int32_t last, int64_t T)
{
    const int begin = inside_batch(first, T), end = inside_batch(last, T);
    return {begin > lo ? begin : lo, end < hi ? end : hi};
}

}  // namespace egtp
