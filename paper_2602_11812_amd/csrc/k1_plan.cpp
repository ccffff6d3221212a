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
// (d = 5120, 65088 tokens: wide 72.1 ms, stream 66.6; V = 32000, d = 2048, 10689 tokens: 986 us and 964, where
// WORTH_IT_OTHERS keeps the wide tile -- the 2.5 %; at d = 256 the folds decide for the wide tile, 106 against 114 us for 5000 tokens.)
static constexpr double WIDE_STEP_NS = 625.0, WIDE_STEP_NS_PER_DOUBLING = 18.5, WIDE_W_BYTES = 48e6, WIDE_FOLD_NS = 5000.0;
static constexpr double NARROW_STEP_NS = 206.0, NARROW_PIECES_STEP_NS = 300.0, NARROW_FOLD_NS = 624.0, NARROW_PIECES_FOLD_NS = 1300.0;
static constexpr double PAIR_STEP_NS = 700.0, SINGLE_STEP_NS = 410.0, PAIR_FOLD_NS = 4000.0;
static constexpr double STREAM_STEP_NS = 642.0, STREAM_ALONE_NS = 400.0, STREAM_FOLD_NS = 6200.0;
static constexpr double STREAM_STEP4_NS = 406.0, STREAM_STEP2_NS = 288.0;
static constexpr double WORKGROUP_NS = 3000.0, W_STREAM_BYTES_PER_NS = 5700.0;
static constexpr long STREAM_MIN_STEPS = 8;  // below, folds are most of the work and the wide tile folds faster
// Another kernel than the wide one is taken at this much of its price: of up to WORTH_IT_TOKENS, in whole cohorts, or else.
// Whole passes, us, wide / stream kernel:
//   few             187 tokens, d = 3152, V = 108446  216 / 178      300, d = 3400, V = 31345  123 / 108      fp32: 160, d = 3048, V = 64460  499 / 433
//   whole cohorts   46211, d = 2280, V = 123447  19354 / 18497       105153, d = 3344, V = 65385  35283 / 32145
//                   fp32: 35094, d = 600, V = 73501  13643 / 12808
//     all priced 0.98 to 1.01 of the wide tile, but:  16814, d = 1368, V = 87862  3096 / 3263      37719, d = 4896, V = 19398  5300 / 5441
//                   fp32: 19818, d = 4352, V = 15161  12672 / 13862
//   others          6338, d = 2608, V = 78554  1855 / 1896           1217, d = 4096, V = 151936  1214 / 1232
static constexpr double WORTH_IT_FEW = 1.01, WORTH_IT_FEW_PIECES = 0.985, WORTH_IT_COHORTS = 0.97, WORTH_IT_OTHERS = 0.955;  // (pieces: fp32 operands)
static constexpr int64_t WORTH_IT_TOKENS = 2 * K1_STREAM_WIDE_TOKENS;
// What the packing launch of bf16 hidden states takes at the least, which plans that read them directly leave out (direct_gain).  Whole passes, us,
// wide / stream kernel with this counted in: 595 tokens, d = 872, V = 15403 64 / 52, 1091, d = 616, V = 8145 56 / 46, 168, d = 600,
// V = 113504 76 / 66, 3189, d = 1232, V = 9789 114 / 99; in full also where unaligned rows cost more, 284, d = 4432, V = 14734 would take 89 for 82.
// Not counted up to STREAM_MIN_STEPS: 414, d = 256, V = 49778 53.5 / 54.4.
static constexpr double PACK_NS = 3500.0;
// Several rounds of the stream kernel, relative to one round or to whole cohorts of 16 token blocks x 2 ranges: cohorts
// cut anywhere (65088 tokens, d = 5120, in 4 ranges 70.3 ms against 66.1; 137720, d = 4096, 122.7 against 116); whole
// ones, per doubling of the ranges (64.6, 66.1, 67.1 ms in 2, 4, 8 ranges); all in one range (131072 tokens, d = 4096:
// 119.0 ms against 109.3 in two).  The three factors rest on these eight launches of three batches, all against V = 151936.
static constexpr double CUT_COHORTS = 1.05, MORE_RANGES = 0.017, ONE_RANGE = 1.09;

// Ranges of the wide kernel (see plan): what a workgroup pays to start and finish, in steps; of the longer ones the longest sweep and
// range, in steps, and what they have to gain
static constexpr double START_STEPS = 8.0;
static constexpr long SHORT_SWEEP = 24, RANGE_STEPS = 600;
static constexpr double WORTH_LONGER = 0.98;

static double wide_step_ns(const K1Plan &p, long steps)
{
    const double w_bytes = (double)p.ntiles_v * TV * (double)steps * 64.0;
    const double doublings = w_bytes > WIDE_W_BYTES ? log2(w_bytes / WIDE_W_BYTES) : 0.0;
    return WIDE_STEP_NS + WIDE_STEP_NS_PER_DOUBLING * (doublings < 5.0 ? doublings : 5.0);
}

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

// Plans without the 256 x 256 tile, bf16: whether hidden states are read where they are, which spares the launch that packs them (4 to 7 us) and the
// reads of rows past the batch.  Rows that begin on lines of 128 bytes: always.  Others ask for two lines of each pair of steps; where that is more than
// the packing they keep the copy.  Whole passes, us, packed / direct, d off the multiples of 64:
//   W_lm inside the Infinity Cache, or read by several blocks
//     narrow      12 tokens, d = 968, V = 20409 25.6 / 22.9; 571, 2528, 6951 62.1 / 58.0; 64, 4104, 16000 50.0 / 47.4
//     stream      264 tokens, d = 1736, V = 104018, 3 sweeps of 55 steps 153 / 138; 705, 1056, 68703, 4 of 33 124.5 / 118.8; but 249, 2136, 139839,
//                 3 of 67 186 / 189; 376, 4344, 115887, 3 of 136 361 / 378.  Sweeps of two fragments a wave, of which the hidden states are half, count
//                 for one and a half: 375, 3608, 9865, 113 steps 59.0 / 58.8; 412, 4184, 5774, 131 steps 62.4 / 64.2
//   one block that streams W_lm past it
//     stream      173 tokens, d = 3000, V = 151936 204 / 226
//     narrow      tokens                                  1            8            16           36           44           64
//                   d = 2568, V = 151936, 238 workgroups  138 / 144    140 / 143    140 / 140    141 / 139    142 / 143    141 / 154
//                   d = 4104                              209 / 214    211 / 212    211 / 209    212 / 207    213 / 210    212 / 229
//                   d = 5016                              252 / 260    253 / 259    254 / 256    255 / 249    256 / 255    254 / 277
//                   d = 2568, V = 100000, 196 workgroups  106 / 97     107 / 97     108 / 99     109 / 108    110 / 112
//                   d = 5016                              182 / 168    183 / 169    184 / 170    184 / 184    185 / 192
//                 Few rows are a few lines that all workgroups want at once, which counts where their loads fill the memory's rate.
static constexpr double DIRECT_STEPS = 180.0;
static constexpr int64_t NARROW_DIRECT_MIN = 12, NARROW_DIRECT_MAX = 36;  // tokens of a narrow plan that streams W_lm
static constexpr long FULL_CHIP = NUM_CUS - NUM_CUS / 8;                  // workgroups that do

// K steps of the sweeps of a range
static double swept_steps(const K1Plan &p, long steps)
{
    const int per_sweep = p.tile_v == K1_STREAM_TILE_V ? 8 : 2, shortest = per_sweep / 4 > 0 ? per_sweep / 4 : 1;
    const int sweeps = (p.tiles_per_split + per_sweep - 1) / per_sweep;
    return (double)sweeps * (double)steps * (p.tiles_per_split <= shortest ? 1.5 : 1.0);
}

bool k1_reads_directly(const K1Plan &p, int dtype, int64_t T, int d, bool on_lines)
{
    if (dtype != DT_BF16 || p.tile_v == K1_WIDE_TILE_V || k1_plan_paces(p))
        return false;
    if (on_lines)
        return true;
    const long steps = 2 * ((d + 63) / 64);
    if (p.tb_tokens == K1_NARROW_TOKENS)
        return !k1_plan_streams_w(p, steps) ||
               (T <= NARROW_DIRECT_MAX && (T >= NARROW_DIRECT_MIN || (long)p.ntb * p.nsplit <= FULL_CHIP));
    return !k1_plan_streams_w(p, steps) && swept_steps(p, steps) <= DIRECT_STEPS;
}

// ns that a plan saves by it: the packing launch, less what unaligned rows cost (113 steps 59.0 / 58.8 above; 316 tokens, d = 5016, V = 15128, 158 steps, in
// plans without / with 88 / 98)
static double direct_gain(const K1Plan &p, int dtype, int64_t T, int d, long steps)
{
    const bool on_lines = d % 64 == 0;
    if (!k1_reads_directly(p, dtype, T, d, on_lines))
        return 0.0;
    if (on_lines || p.tb_tokens == K1_NARROW_TOKENS)
        return PACK_NS;
    const double left = 1.0 - swept_steps(p, steps) / 113.0;
    return left > 0.0 ? PACK_NS * left : 0.0;
}

// the plan of another kernel where that is cheaper than the wide plan p
static K1Plan cheaper(const K1Plan &p, int dtype, int64_t T, int d, int V, long steps)
{
    if (V <= TV || T <= 0)
        return p;  // a vocabulary inside one tile: there is nothing to divide
    K1Plan best = p;  // of the others' plans the cheapest
    double best_ns = -1.0;
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
    // price of a plan of another kernel, `range_ns` a range
    auto price = [&](const K1Plan &q, long read, double range_ns) {
        const double worth = T <= WORTH_IT_TOKENS ? (dtype == DT_BF16 ? WORTH_IT_FEW : WORTH_IT_FEW_PIECES)
                                                  : (q.whole_cohorts ? WORTH_IT_COHORTS : WORTH_IT_OTHERS);
        return plan_ns(q, read, range_ns) / worth;
    };
    auto take = [&](const K1Plan &q, double ns, double at_least) {
        if ((best_ns < 0.0 || ns < at_least * best_ns) && fits(q)) {
            best_ns = ns;
            best = q;
        }
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
            take(q, price(q, read, range), 1.0);
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
            // (among plans of this kernel, fewer rounds of workgroups unless more are clearly cheaper)
            take(q, price(q, steps, stream_range_ns(q, steps)), best.tile_v == K1_STREAM_TILE_V ? 0.99 : 1.0);
        }
        q.whole_cohorts = false;
    }
    const double wide_ns = plan_ns(p, steps, p.tiles_per_split * ((double)steps * wide_step_ns(p, steps) + WIDE_FOLD_NS));
    const double gain_ns = steps > STREAM_MIN_STEPS ? direct_gain(best, dtype, T, d, steps) : 0.0;
    return best_ns >= 0.0 && best_ns - gain_ns < wide_ns ? best : p;
}

static K1Plan plan(int dtype, int64_t T, int d, int V)
{
    K1Plan p;
    p.tb_tokens = TB;
    p.tile_v = TV;
    const long steps = 2 * ((k1_contraction_len(dtype, d) + 63) / 64);  // of a sweep over K
    p.ntb = (int)((T + p.tb_tokens - 1) / p.tb_tokens);
    p.ntiles_v = (V + p.tile_v - 1) / p.tile_v;
    p.nsplit = 1;
    p.tiles_per_split = p.ntiles_v;
    if (p.ntb <= 0)
        return p;
    // One workgroup per (token block, vocabulary range), one workgroup per compute unit at a time, all of about the same length: the
    // number of tiles per range that is cheapest in rounds of workgroups, each of which also fills its ring and finishes.  512 tokens
    // against 594 tiles are 1188 single-tile workgroups = 5 rounds of starts, or 238 workgroups of 5 tiles each = one round of the
    // same length.
    // Batches of more than TARGET_UNITS tiles take about as many workgroups: ranges of a few tiles.  Where a sweep is no more than SHORT_SWEEP steps their starts
    // count, and longer ranges may be cheaper: kernel, us, tiles per range then / now: 7680 tokens, d = 256, V = 118784 2 657 / 14 571; 9520, d = 640,
    // V = 60646 2 720 / 12 690; whole passes 8344, d = 328, V = 118344 2 827 / 15 718, 28500, d = 432, V = 28607 2 768 / 7 697.  Not for longer sweeps, whose
    // ranges drift apart: 38353, d = 1160, V = 43820 3 3203, 6 3299; 96402, d = 4816, V = 6113 2 4601, 12 4950; nor where it is not WORTH_LONGER.
    const int64_t most = ((int64_t)TARGET_UNITS + (1 + NSPLIT_SLACK) * (int64_t)p.ntb) / p.ntb;  // ranges that the workspace has room for
    const int fewest = (int)((p.ntiles_v + most - 1) / most);
    const int64_t target = ((int64_t)TARGET_UNITS + p.ntb - 1) / p.ntb;
    const int ordinary = (int)((p.ntiles_v + target - 1) / target);  // for about TARGET_UNITS workgroups
    const bool large = target < p.ntiles_v;
    const double step_ns = wide_step_ns(p, steps), tile_ns = (double)steps * step_ns + WIDE_FOLD_NS;
    double best = 0.0;
    for (int tps = fewest; tps <= p.ntiles_v && tps < fewest + 64; ++tps) {
        const int nsplit = (p.ntiles_v + tps - 1) / tps;
        const bool longer = large && tps > ordinary;
        if (longer && (steps > SHORT_SWEEP || tps * steps > RANGE_STEPS))
            break;
        const long rounds = ((long)p.ntb * nsplit + NUM_CUS - 1) / NUM_CUS;
        const double cost = (double)rounds * ((double)tps * tile_ns + START_STEPS * step_ns);
        if (tps == fewest || cost < (longer ? WORTH_LONGER : 1.0) * best) {
            best = cost;
            p.nsplit = nsplit;
            p.tiles_per_split = tps;
        }
    }
    return cheaper(p, dtype, T, d, V, steps);
}

K1Plan k1_plan(int dtype, int64_t T, int d, int V)
{
    K1Plan p = plan(dtype, T, d, V);
    p.direct = k1_reads_directly(p, dtype, T, d, d % 64 == 0);
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
