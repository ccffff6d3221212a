// Fused LM-head contraction + streaming entropy (Eq. 2) for batches of few tokens: one query, a decode step with a
// few live sequences, a small model's batch.  Same formulation, packed W_lm and partial triples as the 256 x 256
// kernel; what differs is the tile and what bounds it.
//
// A few tokens make the sweep a stream over W_lm, and a 256-token tile pays for its empty columns in matrix-core
// time and in power.  Here a token block is 64 tokens, a vocabulary tile 128 rows (half a
// packed block: 8 contiguous KiB per K step), so that a step's MFMAs (8 per wave) hide under the step's share
// of the memory stream and the vocabulary divides more evenly over the compute units.  The LDS ring is as deep as
// the LDS allows: what it holds in flight per compute unit sets the rate of the stream.
//
// Workgroup = 4 waves (2 along vocabulary x 2 along tokens), wave tile 64 x 32 = 4 x 2 MFMA 16x16x32 tiles.
// One barrier per step: behind it every wave's loads of the next step have landed and every wave's fragment reads
// of the current step have returned, so its stage can be loaded again; fragments are read one step ahead of
// their MFMAs into two register sets that swap roles (the loop is unrolled by two, K is an even number of steps).
//
// fp32 operands (PIECES): W_lm and the hidden states as three bf16 pieces each, of whose nine products six matter.  The six
// segments of the packed W_lm hold pieces 2, 1, 0, 1, 0, 0; a contraction that walks them reads every piece twice on
// average.  Here a K step brings the pieces (2, 0), (1, 1), (0, 2) of (W_lm, hidden) one after the other, and the fragments
// of earlier pieces are still in registers for the other three products: half the reads and half the steps.  The leading
// product (0, 0) has accumulators of its own, one set for each half of K, so that the small ones meet only their like, as in
// the long contraction, and the large sums are half as long.  Whole decode steps: 24
// tokens against V = 151936, d = 4096 1170 to 1270 -> 670 (5.7 TB/s of pieces); 2, V = 94086, d = 1160 216 -> 125; 64, V = 32000,
// d = 2048 156 -> 87; 47, V = 6763, d = 3440 160 -> 105.
//
// bf16 hidden states are read where they are, two K steps at a time (k1_stream.h), unless the plan says otherwise (k1_plan.cpp), which spares the launch
// that packs them and the reads of rows past the batch: whole passes, d = 4096, V = 151936, 24 tokens 214 -> 207 us, 64 216 -> 208.
//
// Measured: 64 tokens against V = 151936, d = 4096: 199 us = 6.3 TB/s of W_lm (the 256 x 256 tile: 286 us on 198 of the
// 256 compute units); 309 fp32 tokens against V = 4096, d = 256: 15.4 us, 37.1 before.  Two K steps per barrier gain
// nothing.  (Blocks of 192 tokens, which ran on this kernel as well, are the stream kernel's now.)
#include <type_traits>

#include "k1_stream.h"

namespace egtp {
namespace {

constexpr int NM = K1_NARROW_TILE_V;           // vocabulary rows per tile
constexpr int W_STEP_BYTES = NM * ROW_BYTES;   // 8 KiB
constexpr int TB_GROUP = 8;                    // token blocks that sweep the same vocabulary range together
static_assert(NM == 128 && TILE_BYTES == 2 * W_STEP_BYTES, "a vocabulary tile is half a packed block");

constexpr int NI = K1_NARROW_TOKENS / 32;            // token fragments of a wave
constexpr int H_STEP_BYTES = K1_NARROW_TOKENS * ROW_BYTES;
constexpr int STAGE_BYTES = W_STEP_BYTES + H_STEP_BYTES;
constexpr int LOADS = STAGE_BYTES / 4096;           // 16-byte loads per lane and step
constexpr int STAGES = 144 * 1024 / STAGE_BYTES;    // 12
constexpr int RING_BYTES = STAGES * STAGE_BYTES;
static_assert(STAGES >= 3 && (STAGES - 1) * LOADS < 64 && STAGES % 2 == 0, "ring depth");
constexpr int H_RING = STAGES * W_STEP_BYTES;  // direct: the hidden states' stages, of two steps each, lie behind W_lm's

// DIRECT: the hidden states where they are (k1_stream.h); Hp is row-major, of rows of d
template <bool PIECES, bool STREAM_W, bool DIRECT>
__global__ __launch_bounds__(256, 1) void k1_entropy_narrow_kernel(const unsigned char *__restrict__ Wp,
                                                                   const unsigned char *__restrict__ Hp, long T, int d, int KT,
                                                                   int V, int ntb, int nsplit, int ntiles_v,
                                                                   float *__restrict__ part)
{
    static_assert(!(PIECES && DIRECT), "pieces are packed");
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1;  // vocabulary half of the tile
    const int wn = wave & 1;   // token half

    // Workgroup i runs on XCD i % 8: each XCD gets a contiguous range of logical units, token blocks varying
    // fastest, so that the blocks that read the same rows of W_lm share its L2.
    int tb, sp;
    {
        const int units = gridDim.x;
        const int q = units >> 3, r = units & 7;
        const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
        const int logical = x * q + (x < r ? x : r) + j;
        const int per_group = TB_GROUP * nsplit;
        const int g = logical / per_group;
        const int rem = logical - g * per_group;
        const int gsize = min(TB_GROUP, ntb - g * TB_GROUP);
        sp = __builtin_amdgcn_readfirstlane(rem / gsize);
        tb = __builtin_amdgcn_readfirstlane(g * TB_GROUP + (rem - sp * gsize));
    }
    // the first ntiles_v % nsplit ranges hold one tile more than the others
    const int per_range = __builtin_amdgcn_readfirstlane(ntiles_v / nsplit);
    const int longer = ntiles_v - per_range * nsplit;
    const int vt_begin = sp * per_range + min(sp, longer);
    const int vt_end = vt_begin + per_range + (sp < longer ? 1 : 0);
    const long tok0 = (long)tb * (32 * NI);
    // KT blocks of a packed row tile of W_lm, of which a sweep loads KL in turn: all, or with PIECES the first three segments,
    // segment by segment for every K step
    const int kseg = PIECES ? KT / K1_SPLIT_TERMS : KT, KL = PIECES ? 3 * kseg : KT;
    const int total = (vt_end - vt_begin) * KL;

    // ---- global -> LDS: a block is copied linearly, 1 KiB per wave-wide load
    const int lane_off = wave * 1024 + lane * 16;
    const int w_tile_bytes = KT * TILE_BYTES;  // (the launcher checks the range)
    const int h_tile_bytes = KL * H_STEP_BYTES;
    const __amdgpu_buffer_rsrc_t rH = DIRECT ? DirectRows::block(Hp, tok0, 32 * NI, T, d) : raw_buffer(Hp + (long)tb * h_tile_bytes, h_tile_bytes);
    const DirectRows rows(wave, lane, d);
    unsigned char *lds_wave = smem + wave * 1024;
    // The load stream runs ahead of the MFMAs by the ring.  Past the end it keeps re-reading the last step (into
    // stages nobody reads any more), so every step issues the same number of loads and one wait constant serves.
    const int first = DIRECT ? DirectRows::first_step(sp, KT) : 0;
    int lvt = vt_begin, lkt = first, lseg = 0, lstep = 0;  // (segment lseg: blocks lseg, lseg + kseg, ...)
    auto issue_loads = [&](int stage, bool odd) {
        lvt = __builtin_amdgcn_readfirstlane(lvt);  // a descriptor must be uniform, and known to be
        const __amdgpu_buffer_rsrc_t rW = raw_buffer(Wp + (long)(lvt >> 1) * w_tile_bytes, w_tile_bytes);
        const int woff = (lseg + lkt) * TILE_BYTES + (lvt & 1) * W_STEP_BYTES;
        const int hoff = (lseg + lkt) * H_STEP_BYTES;
        unsigned char *dst = lds_wave + stage * (DIRECT ? W_STEP_BYTES : STAGE_BYTES);
#pragma unroll
        for (int p = 0; p < W_STEP_BYTES / 4096; ++p)
            load16_to_lds<STREAM_W>(rW, lane_off, woff + p * 4096, dst + p * 4096);
        if constexpr (!DIRECT) {
#pragma unroll
            for (int p = 0; p < H_STEP_BYTES / 4096; ++p)
                load16_to_lds(rH, lane_off, hoff + p * 4096, dst + W_STEP_BYTES + p * 4096);
        } else if (odd) {  // (a pair of steps comes and goes with its second one)
#pragma unroll
            for (int q = 0; q < 2 * H_STEP_BYTES / 4096; ++q)
                load16_to_lds(rH, rows.offset(q, lkt - 1, d), (lkt - 1) * ROW_BYTES, lds_wave + H_RING + (stage >> 1) * 2 * H_STEP_BYTES + q * 4096);
        }
        const int adv = lstep + 1 < total ? 1 : 0;
        lstep += adv;
        int next = adv;  // to the next K step
        if (PIECES) {
            next = lseg + adv * kseg == 3 * kseg ? 1 : 0;
            lseg = next ? 0 : lseg + adv * kseg;
        }
        const int nk = lkt + next;
        const int wrap = nk == kseg ? 1 : 0;
        lkt = wrap ? 0 : nk;
        lvt += DIRECT ? (next && lkt == first ? 1 : 0) : wrap;
    };

    // ---- fragment reads: row r, chunk c of a block sits at r * 64 + ((c ^ swizzle_key(r)) * 16)
    const int l15 = lane & 15;
    const int kq = lane >> 4;
    const unsigned swz = (unsigned)((kq ^ swizzle_key(l15)) << 4);
    const unsigned fragA = (unsigned)(wm * 64 + l15) * ROW_BYTES + swz;
    const unsigned fragB = (unsigned)W_STEP_BYTES + (unsigned)(wn * 16 * NI + l15) * ROW_BYTES + swz;
    constexpr int FRAG_STRIDE = 16 * ROW_BYTES;
    // Loads in flight behind those that a step waits for: steps k + 2 to k + 11 of even k, half of them with a pair's loads; of odd k, k + 3 to k + 11
    constexpr int W_LOADS = W_STEP_BYTES / 4096, PAIR_LOADS = 2 * H_STEP_BYTES / 4096;
    constexpr int WAIT_EVEN = (STAGES - 2) * W_LOADS + (STAGES - 2) / 2 * PAIR_LOADS;
    constexpr int WAIT_ODD = (STAGES - 3) * W_LOADS + (STAGES - 4) / 2 * PAIR_LOADS;
    struct Frags {
        bf16x8 a[4], b[NI];
    };
    const unsigned frag_direct = (unsigned)H_RING + (unsigned)(wn * 16 * NI) * 2 * ROW_BYTES + DirectRows::fragment(lane);
    auto read_frags = [&](Frags &f, int stage, bool odd) {
        const unsigned char *s = smem + stage * (DIRECT ? W_STEP_BYTES : STAGE_BYTES);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            f.a[i] = *(const bf16x8 *)(s + fragA + i * FRAG_STRIDE);
        const unsigned char *b = DIRECT ? smem + (stage >> 1) * 2 * H_STEP_BYTES + (frag_direct ^ (odd ? DirectRows::ODD : 0u)) : s + fragB;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            f.b[i] = *(const bf16x8 *)(b + i * FRAG_STRIDE * (DIRECT ? 2 : 1));
    };

    Stats st[NI];
    f32x4 acc[4][NI], lead[4][NI], half[4][NI];  // PIECES: the small products, the leading ones of a half of K, of the first half
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        st[ni].m = NEG_BIG;
        st[ni].S = 0.f;
        st[ni].U = 0.f;
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
            acc[mi][ni] = lead[mi][ni] = half[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto multiply = [&](f32x4 (&to)[4][NI], const Frags &w, const Frags &h) {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                to[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.a[mi], h.b[ni], to[mi][ni], 0, 0, 0);
    };

#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        issue_loads(s, s & 1);
    wait_vmcnt<DIRECT ? WAIT_EVEN : (STAGES - 1) * LOADS>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    Frags f0, f1, f2;
    read_frags(f0, 0, false);
    int cstage = 0;  // stage of the step whose MFMAs are next

    // One step.  Wait for the next step's loads (the newest STAGES - 2 steps may still be
    // in flight) and for this wave's own fragment reads, meet the other waves, refill the stage just freed, read the
    // next fragments, multiply.  A bare barrier: a fence would drain the ring.
    // Direct: an even step waits for the step behind it with its pair's hidden states, an odd one for the next pair's.
    auto step = [&](auto odd_const, Frags &next, auto products) {
        constexpr bool ODD = decltype(odd_const)::value;
        wait_vmcnt<DIRECT ? (ODD ? WAIT_ODD : WAIT_EVEN) : (STAGES - 2) * LOADS>();
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), the other counters unconstrained
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const int nstage = cstage + 1 == STAGES ? 0 : cstage + 1;
        read_frags(next, nstage, !ODD);
        issue_loads(cstage, ODD);
        products();
        cstage = nstage;
        __builtin_amdgcn_sched_barrier(0);
    };

    constexpr std::false_type EVEN{};  // (of the pieces' three steps none is odd)
    for (int vt = vt_begin; vt < vt_end; ++vt) {
        if constexpr (PIECES) {
            for (int h = 0, kk = 0; h < 2; ++h) {
                for (const int end = h ? kseg : kseg / 2; kk < end; ++kk) {
                    step(EVEN, f1, [&] { multiply(acc, f0, f0); });
                    step(EVEN, f2, [&] {
                        multiply(acc, f1, f1);
                        multiply(acc, f1, f0);
                    });
                    Frags ahead;
                    step(EVEN, ahead, [&] {
                        multiply(acc, f2, f2);
                        multiply(acc, f2, f1);
                        multiply(lead, f2, f0);
                    });
                    f0 = ahead;
                }
                if (h == 0)
#pragma unroll
                    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) {
                            half[mi][ni] = lead[mi][ni];
                            lead[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
                        }
            }
        } else {
            for (int kt = 0; kt < KT; kt += 2) {
                step(EVEN, f1, [&] { multiply(acc, f0, f0); });
                step(std::true_type{}, f0, [&] { multiply(acc, f1, f1); });
            }
        }
        // a tile of logits is in registers: fold it into the statistics and forget it
        const int row_base = vt * NM + wm * 64 + 4 * kq;
        const bool masked = vt * NM + NM > V;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            float z[16];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    z[4 * q + i] = PIECES ? (half[q][ni][i] + lead[q][ni][i]) + acc[q][ni][i] : acc[q][ni][i];
                    acc[q][ni][i] = lead[q][ni][i] = 0.f;
                }
            if (masked)
                fold<true>(z, st[ni], row_base, V);
            else
                fold<false>(z, st[ni], row_base, V);
        }
    }
    wait_vmcnt<0>();
    __syncthreads();

    // ---- combine the four lanes, then the two waves, that hold the same token
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            Stats o;
            o.m = __shfl_xor(st[ni].m, off);
            o.S = __shfl_xor(st[ni].S, off);
            o.U = __shfl_xor(st[ni].U, off);
            st[ni] = merge(st[ni], o);
        }
    }
    float *red = (float *)smem;  // [wn][ni][16][3]
    if (wm == 1 && lane < 16) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            float *r = red + ((wn * NI + ni) * 16 + lane) * 3;
            r[0] = st[ni].m;
            r[1] = st[ni].S;
            r[2] = st[ni].U;
        }
    }
    __syncthreads();
    if (wm == 0 && lane < 16) {
        const long plane = (long)nsplit * T;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const float *r = red + ((wn * NI + ni) * 16 + lane) * 3;
            Stats o;
            o.m = r[0];
            o.S = r[1];
            o.U = r[2];
            const Stats f = merge(st[ni], o);
            const long tok = tok0 + (wn * NI + ni) * 16 + lane;
            if (tok < T) {
                const long idx = (long)sp * T + tok;
                part[idx] = f.m;
                part[plane + idx] = f.S;
                part[2 * plane + idx] = f.U;
            }
        }
    }
}

template <bool PIECES, bool STREAM_W, bool DIRECT>
hipError_t launch(const void *hidden, const void *w_packed, int64_t T, int d, int kt, int V, const K1Plan &p,
                  float *part, hipStream_t st)
{
    static DeviceMask lds_limit_raised{0};
    const hipError_t e = raise_dynamic_lds_limit((const void *)k1_entropy_narrow_kernel<PIECES, STREAM_W, DIRECT>, RING_BYTES,
                                                 lds_limit_raised);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((k1_entropy_narrow_kernel<PIECES, STREAM_W, DIRECT>), dim3((unsigned)(p.ntb * p.nsplit)), dim3(256), RING_BYTES,
                       st, (const unsigned char *)w_packed, (const unsigned char *)hidden, (long)T, d, kt, V, p.ntb,
                       p.nsplit, p.ntiles_v, part);
    return hipGetLastError();
}

}  // namespace

hipError_t k1_entropy_narrow(const void *hidden, const void *w_packed, int64_t T, int K, int V,
                             const K1Plan &p, float *part, hipStream_t st)
{
    const int kt = k_steps(K);
    if (p.pieces && (p.direct || kt % K1_SPLIT_TERMS != 0))
        return hipErrorInvalidValue;
    if (T <= 0 || p.tb_tokens != K1_NARROW_TOKENS || p.tile_v != NM || p.nsplit < 1 || p.nsplit > p.ntiles_v || (long)p.ntb * p.nsplit > 0x7fffffffL ||
        (int64_t)p.ntb * p.tb_tokens < T || p.ntiles_v != (V + NM - 1) / NM || (long)kt * TILE_BYTES > 0x7fffffffL)
        return hipErrorInvalidValue;
    // W_lm with the non-temporal hint where the Infinity Cache cannot hold it: 64 tokens, d = 4096, V = 151936 (1.24 GB) 225 -> 199 us = 6.3 TB/s;
    // V = 65536 and d = 2560 (336 MB) 60.5 -> 55.7; but V = 65536 and d = 2048 (268 MB) 44 -> 46 and V = 32000 (131 MB) 25 -> 26.
    const int read = p.pieces ? kt / 2 : kt;  // blocks that a sweep reads
    const bool stream = k1_plan_streams_w(p, read);
#define EGTP_NARROW(PIECES, DIRECT)                                                          \
    (stream ? launch<PIECES, true, DIRECT>(hidden, w_packed, T, K, kt, V, p, part, st)       \
            : launch<PIECES, false, DIRECT>(hidden, w_packed, T, K, kt, V, p, part, st))
    return p.pieces ? EGTP_NARROW(true, false) : (p.direct ? EGTP_NARROW(false, true) : EGTP_NARROW(false, false));
#undef EGTP_NARROW
}

}  // namespace egtp
