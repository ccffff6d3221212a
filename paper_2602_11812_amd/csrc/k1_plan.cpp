// Launch geometry of the fused LM-head + entropy kernels (Eq. 2): how a batch of T tokens and a
// vocabulary of V rows is cut into (token block, vocabulary range) workgroups.  Host code only.
#include "k1_plan.h"

#include <math.h>

namespace egtp {

// ---- geometry of the fused entropy kernel ------------------------------------------------
static constexpr int TB = 256, TV = 256, TARGET_UNITS = 8192;

// compute units of the device the work is spread over (MI355X)
static constexpr int NUM_CUS = 256;
static constexpr int NSPLIT_SLACK = 8;  // how far above the minimum the number of ranges may go

// ---- the other two kernels --------------------------------------------------------------
// The three kernels are priced in ns from what one workgroup on its compute unit was measured to take, over T = 24 to
// 137720 at d = 64 to 5120 and V = 4096 to 151936: per K step, per fold of a sweep's logits, and per workgroup (filling
// the load ring, final merge and stores) -- and no plan is faster than one read of W_lm (5.7 TB/s).
//   wide     256 rows x 256 tokens        625 a step for a W_lm of 48 MB, 18.5 more per doubling up to 712 for 1.2 GB;
//            5000 a tile
//   narrow   128 rows x 64 tokens         206 a step, 624 a tile; fp32 operands, in half the steps, 300 and 1300
//   stream   512 rows x 128 tokens        642 a step (+ 400 / token blocks: fewer of them share a read of W_lm), 6200
//            a sweep; remainders of 4 and 2 fragments a wave 406 and 288, 3100 and 1550
//            256 rows x 192 tokens        700 a step, 4000 a sweep; the remainder of 128 rows 410 and 2000
// The model picks the fastest measured plan or one within 2.5 % of it.  At d = 4096, V = 151936, in us (from 193 to 256
// tokens the wide tile runs on 198 of the compute units: 288 to 297 by box for 230):
//   tokens          24   100   173   300   512   800  1217  4000  20000   45000
//   wide           286   280   280   425   475   860  1088  3525  18170   40950
//   narrow         199
//   stream, 128    198   199   289   367   495   793  1123  3320  17450   38900
//   stream, 192                236
// (d = 5120, 65088 tokens: wide 72.1 ms, stream 66.6; V = 32000, d = 2048, 10689 tokens: 986 us and 964, where WORTH_IT
// keeps the wide tile -- the 2.5 %; at d = 256 the folds decide for the wide tile, 106 against 114 us for 5000 tokens.)
static constexpr double WIDE_STEP_NS = 625.0, WIDE_STEP_NS_PER_DOUBLING = 18.5, WIDE_W_BYTES = 48e6, WIDE_FOLD_NS = 5000.0;
static constexpr double NARROW_STEP_NS = 206.0, NARROW_PIECES_STEP_NS = 300.0, NARROW_FOLD_NS = 624.0, NARROW_PIECES_FOLD_NS = 1300.0;
static constexpr double PAIR_STEP_NS = 700.0, SINGLE_STEP_NS = 410.0, PAIR_FOLD_NS = 4000.0;
static constexpr double STREAM_STEP_NS = 642.0, STREAM_ALONE_NS = 400.0, STREAM_FOLD_NS = 6200.0;
static constexpr double STREAM_STEP4_NS = 406.0, STREAM_STEP2_NS = 288.0;
static constexpr double WORKGROUP_NS = 3000.0, W_STREAM_BYTES_PER_NS = 5700.0;
static constexpr long STREAM_MIN_STEPS = 8;  // below, folds are most of the work and the wide tile folds faster
static constexpr double WORTH_IT = 0.955;  // another kernel than the wide one is worth this much of its price
// Several rounds of the stream kernel, relative to one round or to whole cohorts of 16 token blocks x 2 ranges: cohorts
// cut anywhere (65088 tokens, d = 5120, in 4 ranges 70.3 ms against 66.1; 137720, d = 4096, 122.7 against 116); whole
// ones, per doubling of the ranges (64.6, 66.1, 67.1 ms in 2, 4, 8 ranges); all in one range (131072 tokens, d = 4096:
// 119.0 ms against 109.3 in two).  The three factors rest on these eight launches of three batches, all against V = 151936.
static constexpr double CUT_COHORTS = 1.05, MORE_RANGES = 0.017, ONE_RANGE = 1.09;

// what a plan takes if a range of its takes range_ns
static double plan_ns(const K1Plan &p, long steps, double range_ns)
{
    const long units = (long)p.ntb * p.nsplit;
    const long rounds = p.whole_cohorts ? (k1_stream_cohorts(p.ntb, p.nsplit) + 7) / 8 : (units + NUM_CUS - 1) / NUM_CUS;
    double busy = (double)rounds * (range_ns + WORKGROUP_NS);
    if (p.tile_v == K1_STREAM_TILE_V) {
        if (!p.whole_cohorts)
            busy *= rounds > 1 ? CUT_COHORTS : 1.0;
        else if (p.nsplit == 1)
            busy *= ONE_RANGE;
        else
            for (int n = 4; n <= p.nsplit; n *= 2)
                busy *= 1.0 + MORE_RANGES;
    }
    const double read = (double)p.ntiles_v * p.tile_v * (double)steps * 64.0 / W_STREAM_BYTES_PER_NS;
    return (busy > read ? busy : read) + 0.1 * busy;  // of two that only wait for W_lm, the lighter one
}

static double stream_range_ns(const K1Plan &p, long steps)
{
    const int full = p.tiles_per_split / 8, rest = p.tiles_per_split % 8;
    const double step = STREAM_STEP_NS + STREAM_ALONE_NS / p.ntb;
    double ns = (double)(full + (rest > 4 ? 1 : 0)) * ((double)steps * step + STREAM_FOLD_NS);
    if (rest > 2 && rest <= 4)
        ns += (double)steps * STREAM_STEP4_NS + STREAM_FOLD_NS / 2;
    else if (rest > 0 && rest <= 2)
        ns += (double)steps * STREAM_STEP2_NS + STREAM_FOLD_NS / 4;
    return ns;
}

// the plan of another kernel where that is cheaper than the wide plan p
static K1Plan cheaper(const K1Plan &p, int dtype, int64_t T, int V, long steps)
{
    if (V <= TV || T <= 0)
        return p;  // a vocabulary inside one tile: there is nothing to divide
    K1Plan best = p;
    const double w_bytes = (double)p.ntiles_v * TV * (double)steps * 64.0;
    const double doublings = w_bytes > WIDE_W_BYTES ? log2(w_bytes / WIDE_W_BYTES) : 0.0;
    const double wide_step = WIDE_STEP_NS + WIDE_STEP_NS_PER_DOUBLING * (doublings < 5.0 ? doublings : 5.0);
    double best_ns = WORTH_IT * plan_ns(p, steps, p.tiles_per_split * ((double)steps * wide_step + WIDE_FOLD_NS));
    // Workspace is sized for what wide plans need at most: packed hidden states, partial triples, pacing counters.
    auto fits = [&](const K1Plan &q) {
        return (int64_t)q.ntb * q.tb_tokens <= (int64_t)p.ntb * TB &&
               (int64_t)q.nsplit * T <= ((int64_t)TARGET_UNITS + (1 + NSPLIT_SLACK) * (int64_t)p.ntb) * TB &&
               (int64_t)q.nsplit * q.ntb <= (int64_t)TARGET_UNITS + (1 + NSPLIT_SLACK) * (int64_t)p.ntb &&
               (!q.whole_cohorts || k1_stream_cohorts(q.ntb, q.nsplit) <= (long)k1_pace_ints_bound(T));
    };
    auto cut = [&](K1Plan &q, int tb_tokens, int tile_v, int64_t ranges) {
        q.tb_tokens = tb_tokens;
        q.tile_v = tile_v;
        q.ntb = (int)((T + tb_tokens - 1) / tb_tokens);
        q.ntiles_v = (V + tile_v - 1) / tile_v;
        q.tiles_per_split = (int)((q.ntiles_v + ranges - 1) / ranges);
        q.nsplit = (q.ntiles_v + q.tiles_per_split - 1) / q.tiles_per_split;
        // Worth it where W_lm's read is the bound: narrow plans, and one or two blocks of the stream kernel (d = 2048, V = 32000:
        // 160 tokens 196 -> 180 us, 256 240 -> 186; of more blocks, 1500 tokens, d = 1024, V = 8000 144 -> 152).
        q.pieces = dtype == DT_F32 && ((tb_tokens == K1_NARROW_TOKENS && tile_v == K1_NARROW_TILE_V) || q.ntb <= 2);
    };
    K1Plan q;
    const int64_t blocks64 = (T + 63) / 64;
    const double narrow_step = dtype == DT_F32 ? NARROW_PIECES_STEP_NS : NARROW_STEP_NS;
    const double narrow_fold = dtype == DT_F32 ? NARROW_PIECES_FOLD_NS : NARROW_FOLD_NS;
    for (int tokens = K1_NARROW_TOKENS; tokens <= K1_STREAM_WIDE_TOKENS && blocks64 <= 32;
         tokens += K1_STREAM_WIDE_TOKENS - K1_NARROW_TOKENS)
        for (int rounds = 1; rounds <= 3 && (tokens == K1_NARROW_TOKENS || steps <= K1_STREAM_MAX_STEPS); ++rounds) {
            const int64_t ranges = (int64_t)rounds * NUM_CUS * tokens / (blocks64 * 64);
            if (ranges < 1)
                continue;
            cut(q, tokens, K1_NARROW_TILE_V, ranges);
            // (of fp32 operands the narrow kernel reads every piece once, three of the six segments)
            const long read = tokens == K1_NARROW_TOKENS && dtype == DT_F32 ? steps / 2 : steps;
            const double range = tokens == K1_NARROW_TOKENS
                                     ? q.tiles_per_split * ((double)read * narrow_step + narrow_fold)
                                     : (q.tiles_per_split / 2) * ((double)steps * PAIR_STEP_NS + PAIR_FOLD_NS) +
                                           (q.tiles_per_split % 2) * ((double)steps * SINGLE_STEP_NS + PAIR_FOLD_NS / 2);
            const double ns = plan_ns(q, read, range);
            if (ns < best_ns && fits(q)) {
                best_ns = ns;
                best = q;
            }
        }
    // 1, 2, 3, ... long ranges and as many as make one to four rounds of workgroups; paced plans in whole cohorts, too
    for (int i = 1; i <= 20 && steps >= STREAM_MIN_STEPS && steps <= K1_STREAM_MAX_STEPS; ++i) {
        const int64_t ntb = (T + K1_STREAM_TOKENS - 1) / K1_STREAM_TOKENS;
        const int64_t ranges = i <= 16 ? i : (int64_t)(i - 16) * NUM_CUS / ntb;
        if (ranges < 1 || (i > 16 && ranges <= 16))
            continue;
        cut(q, K1_STREAM_TOKENS, K1_STREAM_TILE_V, ranges);
        for (int whole = 0; whole <= (k1_plan_paces(q) ? 1 : 0); ++whole) {
            q.whole_cohorts = whole != 0;
            const double ns = plan_ns(q, steps, stream_range_ns(q, steps));
            // (among plans of this kernel, fewer rounds of workgroups unless more are clearly cheaper)
            if (ns < (best.tile_v == K1_STREAM_TILE_V ? 0.99 : 1.0) * best_ns && fits(q)) {
                best_ns = ns;
                best = q;
            }
        }
        q.whole_cohorts = false;
    }
    return best;
}

// Whether a plan without the 256 x 256 tile reads bf16 hidden states where they are (the packing launch is 4 to 7 us, and packed rows past the
// batch are read like others).  Whole passes, us, packed / direct:
//   narrow   always: 24 tokens, d = 4096, V = 151936 220 / 209, 64 227 / 210, 12 tokens, d = 968, V = 20409 25.6 / 22.9, 571 tokens, d = 2528,
//            V = 6951 62.1 / 58.0
//   stream, 128 and 192 tokens, rows in whole lines of 128 bytes: 173, d = 4096, V = 151936 272 / 260, 100, d = 5120, V = 120000 223 / 212, 786,
//            d = 3520, V = 119754 571 / 555
//   rows that begin inside a line ask for two lines of each pair of steps: not for one block that streams W_lm past the Infinity Cache (173,
//            d = 3000, V = 151936 204 / 226), nor where that outgrows the packing: 376, d = 4344, V = 115887, 3 sweeps of 136 steps 361 / 378; 249,
//            d = 2136, V = 139839, 3 of 67 186 / 189, but 264, d = 1736, V = 104018, 3 of 55 153 / 138, 705, d = 1056, V = 68703, 4 of 33 124.5 /
//            118.8; sweeps of two fragments a wave, of which the hidden states are half, count for one and a half: 412, d = 4184, V = 5774, 131 steps
//            62.4 / 64.2, but 375, d = 3608, V = 9865, 113 steps 59.0 / 58.8
static constexpr double DIRECT_STEPS = 180.0;

static bool reads_directly(const K1Plan &p, int d, long steps)
{
    if (p.tile_v == K1_WIDE_TILE_V || k1_plan_paces(p))
        return false;
    if (p.tb_tokens == K1_NARROW_TOKENS || d % 64 == 0)
        return true;
    const int per_sweep = p.tile_v == K1_STREAM_TILE_V ? 8 : 2, shortest = per_sweep / 4 > 0 ? per_sweep / 4 : 1;
    const int sweeps = (p.tiles_per_split + per_sweep - 1) / per_sweep;
    return !k1_plan_streams_w(p, steps) && (double)sweeps * (double)steps * (p.tiles_per_split <= shortest ? 1.5 : 1.0) <= DIRECT_STEPS;
}

static K1Plan plan(int dtype, int64_t T, int d, int V)
{
    K1Plan p;
    p.tb_tokens = TB;
    p.tile_v = TV;
    const int target = TARGET_UNITS;
    const long dk = k1_contraction_len(dtype, d);  // what a K sweep runs over
    p.ntb = (int)((T + p.tb_tokens - 1) / p.tb_tokens);
    p.ntiles_v = (V + p.tile_v - 1) / p.tile_v;
    int ns0 = p.ntb > 0 ? (target + p.ntb - 1) / p.ntb : 1;
    if (ns0 < 1)
        ns0 = 1;
    p.nsplit = 1;
    p.tiles_per_split = p.ntiles_v;
    if (ns0 >= p.ntiles_v) {
        // A small batch: even one range per vocabulary tile gives fewer workgroups than asked for.  What
        // counts then is the number of rounds the compute units need and what every workgroup pays to
        // start and finish (filling the load ring, the final merge and stores: about START_STEPS K steps
        // of a sweep of 2 ceil(K / 64) steps per tile).  512 tokens against 594 tiles are 1188 single-tile
        // workgroups = 5 rounds of starts, or 238 workgroups of 5 tiles each = one round of the same length.
        constexpr double START_STEPS = 6.0;
        const double start_tiles = START_STEPS / (2.0 * (double)((dk + 63) / 64));
        double best_cost = 0.0;
        for (int tps = 1; tps <= p.ntiles_v && tps <= 64; ++tps) {
            const int nsplit = (p.ntiles_v + tps - 1) / tps;
            const long units = (long)p.ntb * nsplit;
            const long rounds = (units + NUM_CUS - 1) / NUM_CUS;
            const double cost = (double)rounds * ((double)tps + start_tiles);
            if (tps == 1 || cost < best_cost - 1e-9) {
                best_cost = cost;
                p.nsplit = nsplit;
                p.tiles_per_split = tps;
            }
        }
        return cheaper(p, dtype, T, V, 2 * ((dk + 63) / 64));
    }
    // One workgroup per (token block, vocabulary range), one workgroup per compute unit at a
    // time, all of about the same length: among the next few range counts take the one whose
    // last round of workgroups is fullest.
    double best = -1.0;
    for (int ns = ns0; ns <= ns0 + NSPLIT_SLACK; ++ns) {
        const int nsc = ns > p.ntiles_v ? p.ntiles_v : ns;
        const int tps = (p.ntiles_v + nsc - 1) / nsc;
        const int nsplit = (p.ntiles_v + tps - 1) / tps;
        const long units = (long)p.ntb * nsplit;
        const long rounds = (units + NUM_CUS - 1) / NUM_CUS;
        // time ~ rounds * tiles per range; work = ntb * ntiles_v tile sweeps on NUM_CUS units
        const double fill = rounds > 0 ? (double)p.ntb * p.ntiles_v / ((double)rounds * tps * NUM_CUS) : 0.0;
        if (fill > best + 1e-9) {
            best = fill;
            p.nsplit = nsplit;
            p.tiles_per_split = tps;
        }
        if (nsc == p.ntiles_v)
            break;
    }
    return cheaper(p, dtype, T, V, 2 * ((dk + 63) / 64));
}

K1Plan k1_plan(int dtype, int64_t T, int d, int V)
{
    K1Plan p = plan(dtype, T, d, V);
    p.direct = dtype == DT_BF16 && reads_directly(p, d, 2 * ((d + 63) / 64));
    return p;
}

size_t k1_partial_floats(const K1Plan &p, int64_t T) { return (size_t)3 * (size_t)p.nsplit * (size_t)T; }

size_t k1_partial_floats_bound(int64_t T)
{
    // nsplit(T') <= target / ntb(T') + 1 + NSPLIT_SLACK, so
    // nsplit(T') * T' <= (target + (1 + NSPLIT_SLACK) * ntb(T')) * tb_tokens for every T' <= T
    // (plans of the other kernels are only taken if they fit this)
    const int64_t tbk = TB;
    const int64_t target = TARGET_UNITS;
    const int64_t ntb = (T + tbk - 1) / tbk;
    return (size_t)3 * (size_t)((target + (1 + NSPLIT_SLACK) * ntb) * tbk);
}

size_t k1_pace_ints_bound(int64_t T)
{
    // units(T') = ntb(T') * nsplit(T') <= target + (1 + NSPLIT_SLACK) * ntb(T)
    const int64_t tbk = TB;
    const int64_t target = TARGET_UNITS;
    const int64_t ntb = (T + tbk - 1) / tbk;
    return (size_t)8 * (size_t)k1_pace_cohorts((long)(target + (1 + NSPLIT_SLACK) * ntb));
}

}  // namespace egtp
