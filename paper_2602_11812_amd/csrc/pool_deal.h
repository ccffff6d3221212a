// Average and maximum pooling with the batch dealt out evenly (pool_rows_kernel): which rows a workgroup adds up for which
// sequence.  Host and device code, so that it can be checked without a GPU.
#pragma once
#include <cstdint>

namespace egtp {

// A token index inside the batch.  Offsets are the caller's and may hold anything; differences are only taken of what this returns.
constexpr int inside_batch(int32_t token, int64_t T)
{
    return token < 0 ? 0 : (int64_t)token > T ? (int)T : token;
}

// How a batch is dealt out: `deals` workgroups of `rows` rows (the last one of fewer) for each slice of `slice` 16-byte chunks.
struct Deal {
    int64_t rows, deals;
    bool even;  // false: units of the sequences' own instead
};
constexpr int POOL_DEAL_CUS = 256, POOL_DEAL_MIN = 16, POOL_DEAL_SEQUENCES = 2048, POOL_NARROW_SLICE = 128;

// Two workgroups to a compute unit, three with narrow slices; an odd number of rows (see pool_rows_kernel).
//
// From POOL_DEAL_ROWS rows on: a small batch has no workgroups to spare, and units as short as 16 tokens spread it wider.
// And for few sequences beside the rows: the lengths are known on the device alone, and a workgroup takes the sequences among its rows one after the
// other, 0.1 (wide slices, fp32) to 0.35 us (wide, bf16) each; at worst all but one are a token long and meet in one workgroup.
// Passes without the head, us, in units / dealt out, lengths of a long tail; the worst lengths:
//   d = 4096, bf16   137720 tokens, 539 rows   128 sequences 203 / 171; 227 / 216     256 -; 233 / 251     1000 -; 237 / 298
//                     70000, 275                64           98 / 90; 112 / 112       128 113 / 93; 124 / 140
//                     20000, 79                 16           33 / 30; 37 / 35          64 31 / 31; 40 / 50
//   d = 1040, bf16    70000, 137                16           35 / 28; 36 / 35          64 34 / 29; 37 / 46
//                     37008, 73                 16           22 / 19; 22 / 26          64 22 / 19; 23 / 36
//   d = 1024, fp32   137720, 269               128           98 / 87; 111 / 98        256 -; 119 / 124
//                     70000, 137                64           56 / 47; 60 / 54         128 54 / 49; 61 / 65
//                     37008, 73                 16           35 / 28; 34 / 33          64 31 / 28; 34 / 38
//   d = 344, bf16    137720, 181                45           -; 37 / 41               128 31 / 28; 36 / 52
//                     70000, 93                 16           28 / 18; 31 / 26          64 29 / 19; 31 / 34
//                     37008, 49                 16           17 / 13; 19 / 22          64 18 / 14; 19 / 27
//                      2000, 17                 16          9.7 / 10.8; 9.5 / 11.0
constexpr int POOL_DEAL_ROWS = 90, POOL_DEAL_SHARE = 4, POOL_DEAL_SHARE_WIDE_F32 = 2;  // rows for each sequence

constexpr Deal pool_deal(int64_t T, int32_t B, int slice, int64_t ysplit, bool bf16)
{
    const bool narrow = slice <= POOL_NARROW_SLICE;
    const int64_t wanted = (narrow ? 3 : 2) * POOL_DEAL_CUS / ysplit, share = narrow || bf16 ? POOL_DEAL_SHARE : POOL_DEAL_SHARE_WIDE_F32;
    int64_t rows = wanted < 1 ? T : (T + wanted - 1) / wanted;
    rows = (rows < POOL_DEAL_MIN ? POOL_DEAL_MIN : rows) | 1;
    return {rows, (T + rows - 1) / rows, rows >= POOL_DEAL_ROWS && B <= POOL_DEAL_SEQUENCES && share * B <= rows};
}

// The rows [0, n) of a workgroup, which belong to sequence b and those behind it, in order.  Rows around the end of a sequence are loaded AHEAD at a
// time, whatever sequences they are of, so that short ones cost no memory latency each.  A sequence may end below 0 and from n on.
//   whole(i)          rows i to i + AHEAD - 1, to the sequence at hand
//   load(i)           the same rows, in any way those from n on; waits for them: the stores that follow must not be waited for as well
//   begin(r), add(r)  row r of those loaded, the first or another one of the sequence at hand
//   end_of(b)         the row that sequence b ends before
//   next(b, row)      the first sequence behind b that ends behind `row`, or B
//   store(b)          sequence b is complete
// Offsets that decrease give rows to wrong sequences: no row from n on is ever added, and b only grows.
template <int AHEAD, class Whole, class Load, class Begin, class Add, class End, class Next, class Store>
__attribute__((always_inline)) constexpr void walk_rows(int n, int b, int B, Whole whole, Load load, Begin begin, Add add, End end_of, Next next, Store store)
{
    if (n <= 0 || b >= B)
        return;
    int end = end_of(b);
    for (int i = 0; i < n; i += AHEAD) {
        for (; n - i >= AHEAD && end - i >= AHEAD; i += AHEAD)
            whole(i);
        if (i >= n)
            break;
        load(i);
#pragma unroll
        for (int r = 0; r < AHEAD; ++r) {
            if (i + r >= n)
                break;
            if (i + r < end) {
                add(r);
                continue;
            }
            store(b);
            b = next(b, i + r);
            if (b >= B)  // the rows behind the last sequence
                return;
            end = end_of(b);
            begin(r);
        }
    }
    store(b);
}

}  // namespace egtp
