// Launch geometry of the fused LM-head + entropy kernels (Eq. 2): how a batch of T tokens and a
// vocabulary of V rows is cut into (token block, vocabulary range) workgroups.  Host code only.
#include "k1_plan.h"

namespace egtp {

// ---- geometry of the fused entropy kernel ------------------------------------------------
static constexpr int TB = 256, TV = 256, TARGET_UNITS = 8192;

// compute units of the device the work is spread over (MI355X)
static constexpr int NUM_CUS = 256;
static constexpr int NSPLIT_SLACK = 8;  // how far above the minimum the number of ranges may go

// ---- the kernel for few tokens -----------------------------------------------------------
// Both kernels are priced in ns from what a K step of one workgroup was measured to take (d = 4096, V = 151936 and
// d = 2048, V = 32000, every block size at T = 24 ... 1000, one workgroup per compute unit): 745 for the 256 x 256
// tile, 115 + 48 NI for the 128-row tile over 32 NI tokens (its LDS fill and fragment reads, not its MFMAs), about
// 3000 for a workgroup to fill its ring and to merge and store at the end -- and no sweep is faster than one read of
// W_lm (5.7 TB/s).  The model picks the fastest measured variant at each of those sizes: T = 24, d = 4096,
// V = 151936 takes 199 us on 64-token blocks, 225 on 128, 286 on the wide tile; T = 173 262 on 192 against 279;
// T = 300 424 on the wide tile against 459 on 192; T = 309, V = 4096, d = 256 in fp32 15.4 on 64 against 37.1.
static constexpr double WIDE_STEP_NS = 745.0, NARROW_STEP_NS = 115.0, NARROW_STEP_NS_PER_NI = 48.0;
static constexpr double WORKGROUP_NS = 3000.0, W_STREAM_BYTES_PER_NS = 5700.0;

static double sweep_ns(const K1Plan &p, long steps, double step_ns)
{
    const long rounds = ((long)p.ntb * p.nsplit + NUM_CUS - 1) / NUM_CUS;
    const double busy = (double)rounds * ((double)p.tiles_per_split * (double)steps * step_ns + WORKGROUP_NS);
    const double stream = (double)p.ntiles_v * p.tile_v * (double)steps * 64.0 / W_STREAM_BYTES_PER_NS;
    return (busy > stream ? busy : stream) + 0.1 * busy;  // of two that only wait for the stream, the lighter one
}

// a narrow plan where that is cheaper than the wide plan p
static K1Plan narrower(const K1Plan &p, int64_t T, int V, long steps)
{
    if (V <= TV || T <= 0)
        return p;  // a vocabulary inside one tile: there is nothing to divide
    K1Plan best = p;
    double best_ns = 0.97 * sweep_ns(p, steps, WIDE_STEP_NS);  // (a gain within the model's error is none)
    for (int ni = 2; ni <= 8; ni += 2) {
        K1Plan q;
        q.tb_tokens = 32 * ni;
        q.tile_v = K1_NARROW_TILE_V;
        const int64_t ntb = (T + q.tb_tokens - 1) / q.tb_tokens;
        if (ntb * q.tb_tokens > (int64_t)p.ntb * TB)
            continue;  // more padding than the wide blocks (whose packed copy the workspace is sized for)
        q.ntb = (int)ntb;
        q.ntiles_v = (V + q.tile_v - 1) / q.tile_v;
        for (int rounds = 1; rounds <= 3; ++rounds) {
            const int64_t slots = (int64_t)rounds * NUM_CUS / ntb;
            if (slots < 1)
                continue;
            q.tiles_per_split = (int)((q.ntiles_v + slots - 1) / slots);
            q.nsplit = (q.ntiles_v + q.tiles_per_split - 1) / q.tiles_per_split;
            const double ns = sweep_ns(q, steps, NARROW_STEP_NS + NARROW_STEP_NS_PER_NI * ni);
            if (ns < best_ns) {
                best_ns = ns;
                best = q;
            }
        }
    }
    return best;
}

K1Plan k1_plan(int dtype, int64_t T, int d, int V)
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
        return narrower(p, T, V, 2 * ((dk + 63) / 64));
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
    return p;
}

size_t k1_partial_floats(const K1Plan &p, int64_t T) { return (size_t)3 * (size_t)p.nsplit * (size_t)T; }

size_t k1_partial_floats_bound(int64_t T)
{
    // nsplit(T') <= target / ntb(T') + 1 + NSPLIT_SLACK, so
    // nsplit(T') * T' <= (target + (1 + NSPLIT_SLACK) * ntb(T')) * tb_tokens for every T' <= T
    // (narrow plans have at most three rounds of workgroups: far less)
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
