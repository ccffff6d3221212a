// Products of fp32 operands on the bf16 matrix cores: every value is the exact sum of three bf16 pieces, a product of two
// pieces is exact in fp32, and of the nine piece products of a pair the six largest are accumulated (the pieces are rounded to
// nearest: the other three come to 2^-24 of the product at most, fp32's own rounding, and have either sign).  Six 16x16x32
// MFMAs take the place of eight 16x16x4 ones that cost four times as many cycles.
//
// The five small products have sums of their own, so that the large sums are rounded once a step: every MFMA may cost a
// running sum an ulp.  Relative distance of the gradients of W1 and W2 (which shows layer 1) to fp64, 8 seeds, 250 samples, d = 4096,
// d_h = 500, Gaussian operands / all low mantissa bits set:
//   as it is                               2.1e-7 7.0e-8 / 2.2e-7 6.9e-8
//   one sum for all six                    3.2e-7 8.3e-8 / 2.7e-7 7.1e-8
//   ... and pieces cut off (split3_bits)   3.3e-7 1.1e-7 / 3.9e-7 3.2e-7
//   fp32 matrix instructions               3.2e-7 8.2e-8 / 3.0e-7 8.7e-8
// A step of 1024 samples, d = 4096, d_h = 1024: 128.4 us with pieces cut off and one sum, 129.1 as it is.  Device-side header.
#pragma once
#include "bf16_split.h"

namespace egtp {
namespace {

typedef __attribute__((ext_vector_type(4))) float split_f32x4;

// Workgroup tile: 4 waves one above the other, each with 16 FA rows of its own, against 16 FB columns.  A wave splits its
// rows in registers; the columns are shared through the LDS: a K step of 32 lies there as fragments (16 columns x 32 K
// elements, 1 KiB: lane l holds column l % 16, K elements 8 (l / 16) .. + 8), piece by piece.
template <int FA_, int FB_>
struct SplitTile {
    static constexpr int FA = FA_, FB = FB_, WAVES = 4, THREADS = 64 * WAVES, STEP = 32;
    static constexpr int ROWS = 16 * FA * WAVES, COLS = 16 * FB;
    static constexpr int PIECE = FB * 1024, BYTES = 3 * PIECE;
    static constexpr int LDS_BYTES = 2 * BYTES;  // a step is read while the next is staged
    static constexpr int SHARE = FB / WAVES;     // column fragments' lanes that a thread stages: 8 K elements each
};

// The order of a row of N products and of what goes beside it, where one wave has a SIMD to itself: behind each MFMA an LDS read and up to three
// vector instructions.  Left to itself the compiler puts all of them ahead of the row's MFMAs and half of the splitting behind the step:
// layer 1 of 1024 sequences, d = 4096, d_h = 1024 3100 cycles a step for 96 MFMAs of 16, now 2500; the launch 61 -> 56 us, a training step
// 117.2 -> 115.6 (the clock falls to 2.1 GHz).  Tiles of 64 columns, two waves to a SIMD and a few steps, lose by it: 12.3 -> 13.0 us for 160
// sequences, d = d_h = 1024.
template <int N>
__device__ __forceinline__ void interleave()
{
#pragma unroll
    for (int n = 0; n < N; ++n) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
        __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);  // other vector instructions
    }
}

// acc[a][b] += row fragment a . column fragment b over `steps` K steps of the tile.
//
// Everything that a step needs is under way before it: while the products of step i run, the column fragments of step i + 1
// are read from the LDS and its rows split, the columns of step i + 2 are split into the other buffer, rows of step i + 3
// and columns of step i + 4 are asked for.  There are one (tiles of 128 columns) or two waves per SIMD, so the order inside a
// step is pinned: a row of FB products at a time with its share of everything else, which hides in the cycles that an
// MFMA leaves to other instructions.  One barrier per step: behind it step i + 1 is whole and everyone has read step i.  Of a step the smallest
// products come first.
//
// Source: this thread's share of the operands; past the end of the contraction any valid place is loaded, and not used
//   load_rows(i, l, r), load_cols(i, l, r)    load number l of ROW_LOADS / COL_LOADS of step i
//   clear_rows(i, r), clear_cols(i, r)        zeros what of step i lies past the end
//   ROW_PIECES                                3, or 1 for rows that are bf16: three products instead of six
//   row_value(r, a, e), col_value(r, p, e)    K element e of row fragment a / of share p
//   row_pair(r, a, e)                         (one piece) K elements 2 e and 2 e + 1 of row fragment a
//   write_col(buf, part, n), slot()           write number n of COL_WRITES of the pieces of this thread's pairs, part[share]
//                                             [piece][pair]; the 16 bytes of a fragment that this lane reads
//   ROWS_READY                                rows lie in memory as fragments of their pieces: load_rows(i, piece, a, r) loads one, and
//                                             only the columns are split
//   ROWS_TURN                                 rows are loaded by other lanes than use them, and turned in the LDS of the wave:
//   write_row(r, l), read_row(t, l)           load number l of ROW_LOADS on its way there and back
template <class T, class Source>
__device__ __forceinline__ void split_contract(unsigned char *lds, int steps, split_f32x4 (&acc)[T::FA][T::FB],
                                               const Source &src)
{
    constexpr int FA = T::FA, FB = T::FB, SHARE = T::SHARE;
    constexpr bool TURN = Source::ROWS_TURN, READY = Source::ROWS_READY, SPREAD = READY || FB > 4;
    const int slot = src.slot();
    typename Source::Rows ra0, ra1;
    typename Source::Cols rb0, rb1;
    constexpr int PRODUCTS = Source::ROW_PIECES == 3 ? 6 : 3;
    struct RowFragments {
        split_u32x4 p[Source::ROW_PIECES][FA];
    } a0, a1;
    struct ColFragments {
        split_bf16x8 p[3][FB];
    } b0, b1;
    auto read = [&](ColFragments &f, const unsigned char *buf, int n) {
        f.p[n / FB][n % FB] = *(const split_bf16x8 *)(buf + n / FB * T::PIECE + (n % FB * 64 + slot) * 16);
    };
    auto split_rows = [&](const typename Source::Rows &r, RowFragments &f, int n) {
        const int a = n / 4, e = n % 4;
        if constexpr (Source::ROW_PIECES == 1) {
            f.p[0][a][e] = src.row_pair(r, a, e);
        } else if constexpr (!READY) {
            unsigned h, m, l;
            split3_pair_nearest(src.row_value(r, a, 2 * e), src.row_value(r, a, 2 * e + 1), h, m, l);
            if constexpr (SPREAD)
                asm volatile("" : "+v"(h), "+v"(m), "+v"(l));  // here, not where they are used (in front of the next step's products)
            f.p[0][a][e] = h, f.p[1][a][e] = m, f.p[2][a][e] = l;
        }
    };
    split_u32x4 part[SHARE][3];
    auto split_cols = [&](const typename Source::Cols &r, int n) {
        const int p = n / 4, e = n % 4;
        unsigned h, m, l;
        if constexpr (Source::ROW_PIECES == 1)  // every product is taken
            split3_pair(src.col_value(r, p, 2 * e), src.col_value(r, p, 2 * e + 1), h, m, l);
        else
            split3_pair_nearest(src.col_value(r, p, 2 * e), src.col_value(r, p, 2 * e + 1), h, m, l);
        part[p][0][e] = h, part[p][1][e] = m, part[p][2][e] = l;
    };
    auto write = [&](unsigned char *buf, int n) { src.write_col(buf, part, n); };

    constexpr int ROW_PAIRS = 4 * FA, COL_PAIRS = 4 * SHARE, WRITES = Source::COL_WRITES, READS = 3 * FB;
    constexpr int ROW_LOADS = Source::ROW_LOADS, COL_LOADS = Source::COL_LOADS;
    auto fetch_cols = [&](int i, typename Source::Cols &r) {
#pragma unroll
        for (int l = 0; l < COL_LOADS; ++l)
            src.load_cols(i, l, r);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto fetch_rows = [&](int i, typename Source::Rows &r) {
        if constexpr (!READY)
#pragma unroll
            for (int l = 0; l < ROW_LOADS; ++l)
                src.load_rows(i, l, r);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto fetch_fragments = [&](int i, RowFragments &f) {
        if constexpr (READY)
#pragma unroll
            for (int l = 0; l < 3 * FA; ++l)
                f.p[2 - l / FA][l % FA] = src.load_rows(i, 2 - l / FA, l % FA);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto stage = [&](int i, typename Source::Cols &r, unsigned char *buf) {
        src.clear_cols(i, r);
#pragma unroll
        for (int n = 0; n < COL_PAIRS; ++n)
            split_cols(r, n);
#pragma unroll
        for (int n = 0; n < WRITES; ++n)
            write(buf, n);
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch_cols(0, rb0);
    fetch_rows(0, ra0);
    fetch_fragments(0, a0);
    fetch_cols(1, rb1);
    fetch_rows(1, ra1);
    fetch_fragments(1, a1);
    stage(0, rb0, lds);
    fetch_cols(2, rb0);
    src.clear_rows(0, ra0);
    typename Source::Rows turned;
    if constexpr (TURN) {
#pragma unroll
        for (int l = 0; l < ROW_LOADS; ++l)
            src.write_row(ra0, l);
#pragma unroll
        for (int l = 0; l < ROW_LOADS; ++l)
            src.read_row(turned, l);
    }
    if constexpr (!READY)
#pragma unroll
        for (int n = 0; n < ROW_PAIRS; ++n)
            split_rows(TURN ? turned : ra0, a0, n);
    __builtin_amdgcn_sched_barrier(0);
    fetch_rows(2, ra0);
    stage(1, rb1, lds + T::BYTES);
    fetch_cols(3, rb1);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): own reads and writes of the LDS; loads stay in flight
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < READS; ++n)
        read(b0, lds, n);
    // the sums of the small products
    split_f32x4 small[FA][FB];
#pragma unroll
    for (int fa = 0; fa < FA; ++fa)
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
            small[fa][fb] = split_f32x4{0.f, 0.f, 0.f, 0.f};
    // rb: holds the columns of step i + 2; ra: the rows of step i + 1 (READY: a_next does, a is loaded again when its pieces have been used)
    auto step = [&](int i, RowFragments &a, RowFragments &a_next, const ColFragments &b, ColFragments &b_next,
                    typename Source::Rows &ra, typename Source::Cols &rb, unsigned char *mine, const unsigned char *other) {
        constexpr int PA[2][6] = {{2, 1, 0, 1, 0, 0}, {0, 0, 0}}, PB[2][6] = {{0, 1, 2, 0, 1, 0}, {2, 1, 0}};
        constexpr int WHOLE = Source::ROW_PIECES == 1 ? 1 : 0;  // rows in one piece
        // Where what goes beside the products stands, in rows of products.  Wide tiles and ready rows: spread over the step, what
        // the next step waits for early; short rows of products that split rows beside them: the splitting first.
        constexpr int ROWS = PRODUCTS * FA, SPLIT = SPREAD ? ROWS / 3 : ROWS * 2 / 3;
        constexpr int READS_TO = SPREAD ? ROWS - 2 : ROWS, ROWS_FROM = SPREAD ? SPLIT : (TURN ? 3 : 0), ROWS_TO = SPREAD ? ROWS - 1 : SPLIT;
        constexpr int WRITES_TO = SPREAD ? ROWS - 2 : ROWS, COLS_TO = SPREAD ? ROWS - 1 : ROWS, ROW_LOADS_FROM = SPREAD ? ROWS - 1 : SPLIT;
        // the part of n pieces of work, dealt to rows [from, to) of products, that is row's
        auto share = [](int row, int from, int to, int n, auto work) {
#pragma unroll
            for (int k = 0; k < n; ++k)
                if (row >= from && row < to && k >= (row - from) * n / (to - from) && k < (row - from + 1) * n / (to - from))
                    work(k);
        };
        src.clear_cols(i + 2, rb);
        src.clear_rows(i + 1, ra);
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int row = 0; row < ROWS; ++row) {
            const int t = row / FA, fa = row % FA;
#pragma unroll
            for (int fb = 0; fb < FB; ++fb)
            {
                split_f32x4 &sum = t < PRODUCTS - 1 ? small[fa][fb] : acc[fa][fb];
                sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, a.p[PA[WHOLE][t]][fa]),
                                                              b.p[PB[WHOLE][t]][fb], sum, 0, 0, 0);
            }
            share(row, 0, READS_TO, READS, [&](int n) { read(b_next, other, n); });
            if constexpr (TURN) {  // (the LDS serves a wave in order)
#pragma unroll
                for (int l = 0; l < ROW_LOADS; ++l) {
                    if (row == 0)
                        src.write_row(ra, l);
                    if (row == 1)
                        src.read_row(turned, l);
                }
            }
            share(row, 0, SPLIT, COL_PAIRS, [&](int n) { split_cols(rb, n); });
            if constexpr (!READY)
                share(row, ROWS_FROM, ROWS_TO, ROW_PAIRS, [&](int n) { split_rows(TURN ? turned : ra, a_next, n); });
            share(row, SPLIT, WRITES_TO, WRITES, [&](int n) { write(mine, n); });
            share(row, SPLIT, COLS_TO, COL_LOADS, [&](int l) { src.load_cols(i + 4, l, rb); });
            if constexpr (!READY)
                share(row, ROW_LOADS_FROM, ROWS, ROW_LOADS, [&](int l) { src.load_rows(i + 3, l, ra); });
            else if (t == 0 || t == 3 || t == 5)  // the last of this piece's products
                a.p[PA[WHOLE][t]][fa] = src.load_rows(i + 2, PA[WHOLE][t], fa);
            if constexpr (SPREAD && !READY)
                interleave<FB>();
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int i = 0;
    for (; i + 2 <= steps; i += 2) {
        step(i, a0, a1, b0, b1, ra1, rb0, lds, lds + T::BYTES);
        step(i + 1, a1, a0, b1, b0, ra0, rb1, lds + T::BYTES, lds);
    }
    if (i < steps)
        step(i, a0, a1, b0, b1, ra1, rb0, lds, lds + T::BYTES);
#pragma unroll
    for (int fa = 0; fa < FA; ++fa)
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
            acc[fa][fb] += small[fa][fb];
}

// whether every sum of the wave is finite
template <int FA, int FB>
__device__ __forceinline__ bool all_finite(const split_f32x4 (&acc)[FA][FB])
{
    float probe[4] = {0.f, 0.f, 0.f, 0.f};  // NaN as soon as one is not; four chains, not one of all elements
#pragma unroll
    for (int fa = 0; fa < FA; ++fa)
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                probe[e] = fmaf(acc[fa][fb][e], 0.f, probe[e]);
    return __builtin_amdgcn_ballot_w64((probe[0] + probe[1]) + (probe[2] + probe[3]) != 0.f) == 0;
}

// Sums that split_contract left without a finite value, again on the fp32 matrix instructions.  Pieces have no infinities: the
// lower ones of an infinite value are NaN, and infinity times a piece that is zero is NaN as well, where the product of the
// values is infinite.  (A NaN pre-activation counts as an inactive unit, and the head would give a finite number.)  Sums that
// are finite keep their bits: what lies beside an infinite operand does not depend on it.  1024 samples, d = 4096, d_h = 1024:
// a step on finite values 129 us, on NaN 290.
//   load(i, a, b)   K elements 16 i + 4 (lane / 16) + e, e = 0 .. 3, of this lane's rows and columns, zeros past the end
template <int FA, int FB, class Load>
__device__ __forceinline__ void redo_not_finite(int elements, split_f32x4 (&acc)[FA][FB], const Load &load)
{
    split_f32x4 plain[FA][FB];
#pragma unroll
    for (int fa = 0; fa < FA; ++fa)
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
            plain[fa][fb] = split_f32x4{0.f, 0.f, 0.f, 0.f};
    struct Operands {
        float a[FA][4], b[FB][4];
    } now, next;
    load(0, now.a, now.b);
#pragma unroll 1
    for (int i = 0; 16 * i < elements; ++i) {
        load(i + 1, next.a, next.b);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int fa = 0; fa < FA; ++fa)
#pragma unroll
                for (int fb = 0; fb < FB; ++fb)
                    plain[fa][fb] = __builtin_amdgcn_mfma_f32_16x16x4f32(now.a[fa][e], now.b[fb][e], plain[fa][fb], 0, 0, 0);
        now = next;
    }
#pragma unroll
    for (int fa = 0; fa < FA; ++fa)
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (!__builtin_isfinite(acc[fa][fb][e]))
                    acc[fa][fb][e] = plain[fa][fb][e];
}

}  // namespace
}  // namespace egtp
