// Launch geometry of the fused LM-head + entropy kernels (Eq. 2).  Plain host arithmetic with no
// dependency on the HIP runtime, so that it can also be compiled and checked on its own.
#pragma once
#include <stddef.h>
#include <stdint.h>

#ifdef __HIPCC__
#define EGTP_HOST_DEVICE __host__ __device__
#else
#define EGTP_HOST_DEVICE
#endif

namespace egtp {

// Storage types of hidden states / weights (values match the public enum).
enum : int { DT_F32 = 0, DT_BF16 = 1 };

// The fused kernel contracts bf16 operands on the matrix cores.  fp32 operands reach it as sums of three bf16
// pieces each (8 + 8 + 8 significant bits: exact), and the six products of pieces that matter at fp32
// precision are laid side by side along K: a contraction six times as long over segments of d rounded up to
// whole 32-element blocks.
constexpr int K1_SPLIT_TERMS = 6;
EGTP_HOST_DEVICE inline int k1_split_segment(int d) { return (d + 31) / 32 * 32; }
EGTP_HOST_DEVICE inline long k1_contraction_len(int dtype, int d)
{
    return dtype == DT_BF16 ? (long)d : (long)K1_SPLIT_TERMS * k1_split_segment(d);
}
// largest contraction length the fused kernel addresses (32-bit byte offsets inside a packed row tile)
constexpr long K1_MAX_CONTRACTION = 4194240;

// Geometry of the fused LM-head + entropy kernel: tokens are cut into blocks of `tb_tokens`,
// the vocabulary into `nsplit` ranges of `tiles_per_split` tiles of `tile_v` rows; each
// (token block, vocabulary range) pair is one workgroup and leaves one partial (m, S, U)
// triple per token.
// rows per tile of the wide kernel (256 tokens a block); tokens per block and rows per tile of the narrow kernel, for
// few tokens
constexpr int K1_WIDE_TILE_V = 256;
constexpr int K1_NARROW_TOKENS = 64, K1_NARROW_TILE_V = 128;
// ... and of the stream kernel, for the largest batches and for those between the other two: 128 tokens against tiles of
// 64 rows, or 192 against the narrow kernel's
constexpr int K1_STREAM_TOKENS = 128, K1_STREAM_TILE_V = 64;
constexpr int K1_STREAM_WIDE_TOKENS = 192;
constexpr int K1_STREAM_PACE_TILES = 16;  // its pacing points, in tiles
// A sweep of its may straddle two packed 256-row tiles of W_lm, 16 KiB per K step each, under one 32-bit byte offset:
// half of what the other kernels address.
constexpr long K1_STREAM_MAX_STEPS = 0x7fffffffL / (2 * 16384);

struct K1Plan {
    int tb_tokens;        // tokens per block
    int tile_v;           // vocabulary rows per tile
    int ntb;              // token blocks
    int ntiles_v;         // vocabulary tiles in total
    int nsplit;           // vocabulary ranges
    int tiles_per_split;  // tiles per range (last range may hold fewer)
    bool whole_cohorts = false;  // stream kernel, paced: each XCD gets whole cohorts (k1_stream_cohorts)
    // fp32 operands, narrow and stream kernel: the sweep reads the three segments that hold each piece once, and the
    // hidden states are packed into those alone
    bool pieces = false;
    // narrow and stream kernel, bf16: hidden states are read where they are instead of from a packed copy
    bool direct = false;
};

K1Plan k1_plan(int dtype, int64_t T, int d, int V);
// p.direct for T tokens whose rows begin on lines of 128 bytes, or do not
bool k1_reads_directly(const K1Plan &p, int dtype, int64_t T, int d, bool on_lines);
// floats needed for the partial triples of a plan (3 * nsplit * T)
size_t k1_partial_floats(const K1Plan &p, int64_t T);
// upper bound of k1_partial_floats over every T' <= T, whatever the shapes
size_t k1_partial_floats_bound(int64_t T);
// The kernel paces the workgroups that share an XCD with one counter per cohort of 32:
// cohorts per XCD for a grid of `units` workgroups, and ints to reserve for every T' <= T.
EGTP_HOST_DEVICE inline int k1_pace_cohorts(long units) { return (int)(((units + 7) / 8 + 31) / 32); }
size_t k1_pace_ints_bound(int64_t T);

// The stream kernel: token blocks that sweep the same ranges together, such that a cohort of 32 workgroups holds
// 32 / group ranges, and how many cohorts that makes.
inline int k1_stream_group(int nsplit) { return nsplit >= 4 ? 8 : (nsplit >= 2 ? 16 : 32); }
inline long k1_stream_cohorts(int ntb, int nsplit)
{
    const int group = k1_stream_group(nsplit), ranges = 32 / group;
    return (long)((ntb + group - 1) / group) * ((nsplit + ranges - 1) / ranges);
}

// A range has a pacing point after every K1_PACE_TILES vocabulary tiles, so only
// ranges longer than that pace at all.
constexpr int K1_PACE_TILES = 4;
// Pacing serves the token blocks that share vocabulary tiles in an XCD's L2 (groups of eight): a batch of
// fewer blocks streams W_lm once from HBM whatever the workgroups' relative progress.
inline bool k1_plan_paces(const K1Plan &p)
{
    if (p.tile_v == K1_STREAM_TILE_V)
        return p.tiles_per_split > K1_STREAM_PACE_TILES && p.ntb >= 16;
    return p.tile_v != K1_NARROW_TILE_V && p.tiles_per_split > K1_PACE_TILES && p.ntb >= 8;
}
// One token block reads W_lm once, `steps` packed blocks of every tile: whether the 256 MiB Infinity Cache cannot hold it until the next call either, so
// that its loads carry the non-temporal hint.
inline bool k1_plan_streams_w(const K1Plan &p, long steps)
{
    return p.ntb == 1 && (int64_t)p.ntiles_v * p.tile_v * steps * 64 > ((int64_t)256 << 20);
}
// counters that a plan paces with, to be zero when the fused kernel starts
inline long k1_pace_ints(const K1Plan &p)
{
    if (!k1_plan_paces(p))
        return 0;
    return p.whole_cohorts ? k1_stream_cohorts(p.ntb, p.nsplit) : 8L * k1_pace_cohorts((long)p.ntb * p.nsplit);
}

}  // namespace egtp
