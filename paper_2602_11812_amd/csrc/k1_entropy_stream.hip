// Fused LM-head contraction + streaming entropy (Eq. 2), W_lm loaded straight into registers: for the largest batches
// and for those between the other two kernels.  Same formulation, packed W_lm and partial triples as theirs; what
// differs is the way of W_lm to the matrix cores.
//
// A token block is 128 or 192 tokens and a wave works alone on its rows of W_lm: a 16-row fragment of a packed block is
// one contiguous KiB in exactly the order the MFMA wants, so the wave loads it straight into registers (D K steps
// ahead) and it never passes through the LDS.  Only the hidden states do, 8 or 12 KiB per K step shared by the four
// waves -- per product less than half the LDS traffic of a tile that stages both operands.  Rows are dealt
// to waves in single fragments, so the vocabulary divides evenly over the compute units whatever its size:
//   128 tokens  a wave sweeps eight fragments at a time (8 x 8 MFMA 16x16x32 tiles, 128 rows x 128 tokens) and the
//               remainder in a shorter sweep of two, four or six;
//   192 tokens  four fragments at a time (4 x 12 tiles), the remainder in a sweep of two; two fragments to a vocabulary
//               tile.  Half as many rows in flight per step, hence four steps ahead where K is a multiple of four
//               steps (two sets of registers would hold 32 KiB of W_lm per compute unit in flight, four hold 64).
//
// Bound: bf16 MFMA at the package power limit for large batches, the read of W_lm for one token block.  Measured
// against the 256 x 256 tile, same box: 137720 tokens, d = 4096, V = 151936 118.6 -> 114.7 ms = 1.49 PFLOP/s; 65088
// tokens, d = 5120 70.5 -> 64.7 = 1.56 PFLOP/s; 4000 tokens 3.57 -> 3.37; 384 tokens 447 -> 378 us; 128 tokens 280 ->
// 199 us.  No faster: the barrier in the middle of a step (3 % slower), other spacings of the loads, four or eight ring
// stages, a pacing point every sweep or every fourth.
// 192 tokens: what limits a sweep beside the stream is the way from the L2 into the compute unit, about 42 bytes/ns
// whatever the kernel: per 256 rows and K step 28 KiB here, 40 with both operands through the LDS (the narrow kernel's
// tile, which served these batches before): 173 tokens against V = 151936 285 to 325 -> 236 to 257 us by box, V = 70812,
// d = 1800 77 -> 64.  No faster: two waves side by side on the same rows, 96 tokens each (less LDS traffic, but every
// fragment of W_lm loaded twice: 316 us), five fragments at a time (registers spill: 315).  For 256 tokens the pair of
// waves gives the 256 x 256 tile's times within 2 %, and a wave of its own on 64 rows x 256 tokens spills: not built.
//
// bf16 hidden states are read where they are, two K steps at a time (k1_stream.h), unless the plan says otherwise (k1_plan.cpp): 173 tokens, d = 4096,
// V = 151936 272 -> 260 us a pass.
//
// Pacing is that of the 256 x 256 kernel: cohorts of 32 workgroups that share blocks in an XCD's L2 count themselves in
// every second sweep and wait, bounded, for the rest; a hint that no result depends on.
#include <type_traits>

#include "k1_stream.h"

namespace egtp {
namespace {

constexpr int FRAG_BYTES = 16 * ROW_BYTES;  // 16 rows of one K step

// The two shapes: a token block is 16 NI tokens, a wave's longest sweep MAX_MI fragments of 16 rows (together they fill the
// accumulators), a tile of the plan FPW fragments for each of the four waves, and the ring holds STAGES K steps of hidden states.
template <int NI>
struct Shape {
    static constexpr int TOKENS = 16 * NI;
    static constexpr int MAX_MI = NI == 8 ? 8 : 4;
    static constexpr int FPW = NI == 8 ? 1 : 2;
    static constexpr int STAGES = NI == 8 ? 6 : 8;
    static constexpr int DIRECT_STAGES = 8;  // four pairs of steps
    static constexpr int H_STEP_BYTES = TOKENS * ROW_BYTES;
    static constexpr int H_LOADS = H_STEP_BYTES / 4096;  // 16-byte loads per lane and step
    static constexpr int LDS_BYTES = STAGES * H_STEP_BYTES, DIRECT_LDS_BYTES = DIRECT_STAGES * H_STEP_BYTES;
    static_assert((STAGES - 2) * (H_LOADS + MAX_MI) < 64 && (DIRECT_STAGES - 2) * (H_LOADS + MAX_MI) < 64, "one wait covers the ring");
};
static_assert(Shape<8>::TOKENS == K1_STREAM_TOKENS && Shape<8>::FPW * 64 == K1_STREAM_TILE_V, "plan");
static_assert(Shape<12>::TOKENS == K1_STREAM_WIDE_TOKENS && Shape<12>::FPW * 64 == K1_NARROW_TILE_V, "plan");
constexpr int PACE_SWEEPS = K1_STREAM_PACE_TILES / Shape<8>::MAX_MI;  // sweeps between two pacing points
static_assert(2L * K1_STREAM_MAX_STEPS * TILE_BYTES <= 0x7fffffffL, "two packed tiles under one offset");

// fp32 operands read by their pieces: the blocks that each K step multiplies.  Only the first three segments are read, W_lm's
// holding pieces 2, 1, 0 and the hidden states' 0, 1, 2; every K step of those is taken through the five small
// products (2,0) (1,1) (0,2) (1,0) (0,1) in turn, so that a piece is read again while it is in the L2, and the leading
// products (0,0) follow in a pass of their own: the accumulators meet the small terms first, as in the long contraction.
struct PieceWalk {
    static constexpr unsigned W_SEGMENTS = 0 | 1 << 2 | 2 << 4 | 1 << 6 | 2 << 8 | 2 << 10;  // two bits per product
    static constexpr unsigned H_SEGMENTS = 0 | 1 << 2 | 2 << 4 | 0 << 6 | 1 << 8 | 0 << 10;
    static constexpr int LEAD = K1_SPLIT_TERMS - 1;
    int kk = 0, product = 0;
    // the block of this step; moves on to the next step, from the last one to the first
    __device__ __forceinline__ int next(unsigned segments, int kseg)
    {
        const int block = (int)(segments >> (2 * product) & 3u) * kseg + kk;
        const bool lead = product == LEAD, next_k = product >= LEAD - 1;
        product = lead ? LEAD : (next_k ? 0 : product + 1);
        const int k = kk + (next_k ? 1 : 0);
        const bool end = k == kseg;
        kk = end ? 0 : k;
        product = end ? (lead ? 0 : LEAD) : product;
        return block;
    }
};

template <bool STREAM_W>
__device__ __forceinline__ bf16x8 load_fragment(__amdgpu_buffer_rsrc_t rsrc, int lane_byte_offset, int scalar_byte_offset)
{
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_byte_offset, scalar_byte_offset,
                                                                           STREAM_W ? 2 : 0));
}

template <int NI, int D, bool PIECES, bool STREAM_W, bool DIRECT>
__global__ __launch_bounds__(256, 1) void k1_entropy_stream_kernel(const unsigned char *__restrict__ Wp,
                                                                   const unsigned char *__restrict__ Hp, long T, int d, int KT,
                                                                   int V, int ntb, int nsplit, int tps, int ntiles_v, int group, bool whole_cohorts,
                                                                   float *__restrict__ part, int *__restrict__ pace)
{
    using S = Shape<NI>;
    constexpr int MAX_MI = S::MAX_MI, FPW = S::FPW, H_STAGES = DIRECT ? S::DIRECT_STAGES : S::STAGES;
    constexpr int H_STEP_BYTES = S::H_STEP_BYTES, H_LOADS = S::H_LOADS;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Which (token block, vocabulary range) this workgroup owns.  Workgroup i runs on XCD i % 8, 32 of an XCD's at a
    // time (a cohort).
    int tb, sp;
    int *pace_cnt = nullptr;  // this workgroup's cohort counter (thread 0 only)
    int pace_members = 0;
    {
        const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
        if (whole_cohorts) {
            // A cohort is `group` token blocks x 32 / group ranges, so that its blocks of both operands are shared
            // in the XCD's L2; an XCD gets whole cohorts, and a place without a unit is left empty.  (Cut
            // anywhere, cohorts of half the blocks of one group and half of the next read a third more.)
            const int ranges = COHORT / group;
            const int per_group = (nsplit + ranges - 1) / ranges;
            const int cohorts = (ntb + group - 1) / group * per_group;
            const int c = (int)((long)x * cohorts / 8) + j / COHORT;
            const int g = c / per_group, r = j % COHORT;
            tb = g * group + r % group;
            sp = (c - g * per_group) * ranges + r / group;
            if (c >= (int)((long)(x + 1) * cohorts / 8) || tb >= ntb || sp >= nsplit)
                return;
            if (pace != nullptr && tid == 0) {
                pace_cnt = pace + c;
                pace_members = min(group, ntb - g * group) * min(ranges, nsplit - (c - g * per_group) * ranges);
            }
        } else {
            // each XCD gets a contiguous range of units, token blocks varying fastest
            const int units = ntb * nsplit;
            const int q = units >> 3, r = units & 7;
            if (pace != nullptr && tid == 0) {
                const int cohort = j / COHORT;
                pace_cnt = pace + x * k1_pace_cohorts(units) + cohort;
                pace_members = min(COHORT, q + (x < r ? 1 : 0) - cohort * COHORT);
            }
            const int logical = x * q + (x < r ? x : r) + j;
            const int per_group = group * nsplit;
            const int g = logical / per_group;
            const int rem = logical - g * per_group;
            const int gsize = min(group, ntb - g * group);
            sp = rem / gsize;
            tb = g * group + (rem - sp * gsize);
        }
        sp = __builtin_amdgcn_readfirstlane(sp);
        tb = __builtin_amdgcn_readfirstlane(tb);
    }
    // this range's tiles = so many fragments for each wave
    int vt_begin, count;
    if (FPW == 2) {  // the first ntiles_v % nsplit ranges hold one tile more than the others
        const int per_range = ntiles_v / nsplit, longer = ntiles_v - per_range * nsplit;
        vt_begin = sp * per_range + min(sp, longer);
        count = per_range + (sp < longer ? 1 : 0);
    } else {
        vt_begin = sp * tps;
        count = min(tps, ntiles_v - vt_begin);
    }
    const int f_begin = FPW * (4 * vt_begin + wave * count), f_end = f_begin + FPW * count;
    const long tok0 = (long)tb * S::TOKENS;
    const int row_end = min(V, f_end * 16);

    // ---- W_lm: the fragments of a sweep, by scalar offsets from the packed block its first one lies in
    const int l15 = lane & 15;
    const int kq = lane >> 4;
    const int lane_w = l15 * ROW_BYTES + ((kq ^ swizzle_key(l15)) << 4);
    const int w_tile_bytes = KT * TILE_BYTES;  // (the launcher checks that two of them can be addressed)
    __amdgpu_buffer_rsrc_t rW;
    int frag_off[MAX_MI];
    auto set_rows = [&](int f0) {  // past the end: the last fragment, loaded and not used
        const int first = min(f0, f_end - 1);
        const int blk = __builtin_amdgcn_readfirstlane(first >> 4);
        const int blocks = __builtin_amdgcn_readfirstlane(((f_end - 1) >> 4) - blk > 0 ? 2 : 1);
        rW = raw_buffer(Wp + (long)blk * w_tile_bytes, blocks * w_tile_bytes);
#pragma unroll
        for (int m = 0; m < MAX_MI; ++m) {
            const int f = min(f0 + m, f_end - 1);
            frag_off[m] = __builtin_amdgcn_readfirstlane(((f >> 4) - blk) * w_tile_bytes + (f & 15) * FRAG_BYTES);
        }
    };
    bf16x8 wr[D][MAX_MI];
    const int kseg = KT / K1_SPLIT_TERMS;  // PIECES: K steps of a segment
    PieceWalk walk_w, walk_h;
    const int first = DIRECT ? DirectRows::first_step(sp, KT) : 0;
    auto w_offset = [&](int kt) {  // of the step whose fragments are loaded next
        if (DIRECT)
            kt = kt + first < KT ? kt + first : kt + first - KT;
        return (PIECES ? walk_w.next(PieceWalk::W_SEGMENTS, kseg) : kt) * TILE_BYTES;
    };

    // ---- hidden states: memory -> LDS ring, copied linearly, 1 KiB per wave-wide load; the same block sweep after sweep
    const int lane_h = wave * 1024 + lane * 16;
    const int h_tile_bytes = (PIECES ? 3 * kseg : KT) * H_STEP_BYTES;
    const __amdgpu_buffer_rsrc_t rH = DIRECT ? DirectRows::block(Hp, tok0, S::TOKENS, T, d) : raw_buffer(Hp + (long)tb * h_tile_bytes, h_tile_bytes);
    const DirectRows rows(wave, lane, d);
    int hkt = first;
    auto load_h = [&](int stage) {
        unsigned char *dst = smem + stage * H_STEP_BYTES + wave * 1024;
        const int off = (PIECES ? walk_h.next(PieceWalk::H_SEGMENTS, kseg) : hkt) * H_STEP_BYTES;
#pragma unroll
        for (int p = 0; p < H_LOADS; ++p)
            load16_to_lds(rH, lane_h, off + p * 4096, dst + p * 4096);
        hkt = hkt + 1 == KT ? 0 : hkt + 1;
    };
    // direct: half `part` of the loads of the pair of steps that ends with `stage`
    auto load_pair = [&](int stage, int part) {
        unsigned char *dst = smem + (stage >> 1) * 2 * H_STEP_BYTES + wave * 1024;
#pragma unroll
        for (int q = part * H_LOADS; q < (part + 1) * H_LOADS; ++q)
            load16_to_lds(rH, rows.offset(q, hkt, d), hkt * ROW_BYTES, dst + q * 4096);
        if (part == 1)
            hkt = hkt + 2 == KT ? 0 : hkt + 2;
    };
    const unsigned frag_h = DIRECT ? DirectRows::fragment(lane) : (unsigned)lane_w;
    constexpr int FRAG_STRIDE = DIRECT ? 2 * FRAG_BYTES : FRAG_BYTES;
    bf16x8 fb[2][NI];

    Stats st[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        st[ni].m = NEG_BIG;
        st[ni].S = 0.f;
        st[ni].U = 0.f;
    }

    set_rows(f_begin);
#pragma unroll
    for (int s = 0; s < H_STAGES; ++s) {
        if (!DIRECT)
            load_h(s);
        else if (s & 1)
            load_pair(s, 0), load_pair(s, 1);
    }
#pragma unroll
    for (int s = 0; s < D; ++s) {
        const int off = w_offset(s);
#pragma unroll
        for (int m = 0; m < MAX_MI; ++m)
            wr[s][m] = load_fragment<STREAM_W>(rW, lane_w, off + frag_off[m]);
    }
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
        fb[0][ni] = *(const bf16x8 *)(smem + frag_h + ni * FRAG_STRIDE);
    int cstage = 0;  // stage of the step whose MFMAs are next

    // All K steps of MI fragments from f0 on, then the fold of their logits.  Before its last D steps the loads
    // move on to the fragments of the next sweep.
    auto sweep = [&](auto mi_const, int f0, bool masked) {
        constexpr int MI = decltype(mi_const)::value;
        f32x4 acc[MI][NI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
        // One step of parity P.  The barrier: every wave's loads of the next step's hidden states have landed (the
        // newest H_STAGES - 2 steps' loads may be in flight; a step issues at least H_LOADS + MI of them) and every wave's
        // fragment reads of the current step have returned, so its stage can be loaded again.
        auto step = [&](auto p_const, int kt_load) {
            constexpr int P = decltype(p_const)::value, Q = P & 1;
            // (direct: pairs come with their odd steps, and an odd step waits for the pair behind it)
            wait_vmcnt<DIRECT && Q ? (H_STAGES - 3) * MI + (H_STAGES - 4) * H_LOADS : (H_STAGES - 2) * (H_LOADS + MI)>();
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), the other counters unconstrained
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            const int nstage = cstage + 1 == H_STAGES ? 0 : cstage + 1;
            const unsigned char *s = DIRECT ? smem + (nstage >> 1) * 2 * H_STEP_BYTES + (frag_h ^ (Q ? 0u : DirectRows::ODD))
                                            : smem + nstage * H_STEP_BYTES + frag_h;
            const int woff = w_offset(kt_load + P);
            // The order is pinned row by row: the fragment reads behind the first row's MFMAs, then in every row the
            // load of the row before it (whose registers are free by then), the hidden states' loads in rows 0 and 1.
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                if (mi == 0) {
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        fb[Q ^ 1][ni] = *(const bf16x8 *)(s + ni * FRAG_STRIDE);
                } else {
                    wr[P][mi - 1] = load_fragment<STREAM_W>(rW, lane_w, woff + frag_off[mi - 1]);
                }
                constexpr int SECOND = MI > 2 ? 2 : 1;  // (direct: the row of the second half of a pair's loads)
                int h_loads = 0;
                if (!DIRECT && mi == 1)
                    load_h(cstage), h_loads = H_LOADS;
                if (DIRECT && Q && mi == 1)
                    load_pair(cstage, 0), h_loads += H_LOADS;
                if (DIRECT && Q && mi == SECOND)
                    load_pair(cstage, 1), h_loads += H_LOADS;
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[P][mi], fb[Q][ni], acc[mi][ni], 0, 0, 0);
                if (mi == 0) {
#pragma unroll
                    for (int j = 0; j < NI; ++j) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 1 + h_loads; ++j) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x008, NI, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            wr[P][MI - 1] = load_fragment<STREAM_W>(rW, lane_w, woff + frag_off[MI - 1]);
            cstage = nstage;
            __builtin_amdgcn_sched_barrier(0);
        };
        auto steps = [&](int kt_load) {
            step(std::integral_constant<int, 0>{}, kt_load);
            step(std::integral_constant<int, 1>{}, kt_load);
            if constexpr (D == 4) {
                step(std::integral_constant<int, 2>{}, kt_load);
                step(std::integral_constant<int, 3>{}, kt_load);
            }
        };
        for (int kt = D; kt < KT; kt += D)
            steps(kt);
        set_rows(f0 + MI);
        steps(0);

        const int row0 = f0 * 16 + 4 * kq;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
            for (int h = 0; h < MI; h += 4) {
                // fragments folded at once (128 tokens: a remainder of two is folded with two that do not exist;
                // without them the compiler orders the loads of the long sweeps worse, 1 % of their time)
                constexpr int N = NI > 8 && MI < 4 ? MI : 4;
                float z[4 * N];
#pragma unroll
                for (int q = 0; q < N; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        z[4 * q + i] = h + q < MI ? acc[h + q < MI ? h + q : 0][ni][i] : NEG_BIG;
                if (masked || MI % N != 0)
                    fold<true>(z, st[ni], row0 + h * 16, h + 4 > MI ? min(row_end, (f0 + MI) * 16) : row_end);
                else
                    fold<false>(z, st[ni], row0 + h * 16, row_end);
            }
            if (NI > 8)
                __builtin_amdgcn_sched_barrier(0);  // (one token at a time, for the registers)
        }
    };
    const int max_sweeps = (tps * FPW + MAX_MI - 1) / MAX_MI;
    int sweeps = 0;
    for (int f = f_begin; f < f_end;) {
        const int rest = f_end - f;
        // pacing point: the other waves wait for this thread at the next step's barrier
        const bool pace_now = pace_cnt != nullptr && sweeps != 0 && sweeps % PACE_SWEEPS == 0;
        if (pace_now) {
            const int want = pace_members * (sweeps / PACE_SWEEPS);
            __hip_atomic_fetch_add(pace_cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bool met = false;
            for (int spin = 0; spin < PACE_SPINS && !met; ++spin) {
                met = __hip_atomic_load(pace_cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= want;
                if (!met)
                    __builtin_amdgcn_s_sleep(PACE_SLEEP);
            }
            if (!met) {
                // the cohort is not running together: count in for every later point and stop
                const int later = (max_sweeps - 1) / PACE_SWEEPS - sweeps / PACE_SWEEPS;
                if (later > 0)
                    __hip_atomic_fetch_add(pace_cnt, later, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                pace_cnt = nullptr;
            }
        }
        ++sweeps;
        if constexpr (MAX_MI == 8) {
            if (rest > 4) {
                sweep(std::integral_constant<int, 8>{}, f, rest < 8 || (f + 8) * 16 > V);
                f += 8;
                continue;
            }
        }
        if (rest > 2) {
            sweep(std::integral_constant<int, 4>{}, f, rest < 4 || (f + 4) * 16 > V);
            f += 4;
        } else {
            sweep(std::integral_constant<int, 2>{}, f, rest < 2 || (f + 2) * 16 > V);
            f += 2;
        }
    }
    if (pace_cnt != nullptr) {
        // a range with fewer sweeps than the others leaves early: count in for the points it skips
        const int skipped = (max_sweeps - 1) / PACE_SWEEPS - (sweeps - 1) / PACE_SWEEPS;
        if (skipped > 0)
            __hip_atomic_fetch_add(pace_cnt, skipped, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    wait_vmcnt<0>();
    __syncthreads();

    // ---- combine the four lanes, then the four waves, that hold the same token
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
    float *red = (float *)smem;  // [wave][token][3]
    if (lane < 16) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            float *r = red + (wave * S::TOKENS + ni * 16 + lane) * 3;
            r[0] = st[ni].m;
            r[1] = st[ni].S;
            r[2] = st[ni].U;
        }
    }
    __syncthreads();
    if (tid < S::TOKENS && tok0 + tid < T) {
        Stats a;
        a.m = red[tid * 3], a.S = red[tid * 3 + 1], a.U = red[tid * 3 + 2];
#pragma unroll
        for (int k = 1; k < 4; ++k) {
            const float *r = red + (k * S::TOKENS + tid) * 3;
            Stats o;
            o.m = r[0], o.S = r[1], o.U = r[2];
            a = merge(a, o);
        }
        const long plane = (long)nsplit * T, idx = (long)sp * T + tok0 + tid;
        part[idx] = a.m;
        part[plane + idx] = a.S;
        part[2 * plane + idx] = a.U;
    }
}

template <int NI, int D, bool PIECES, bool STREAM_W, bool DIRECT>
hipError_t launch(const void *hidden, const void *w_packed, int64_t T, int d, int kt, int V, const K1Plan &p, int group,
                  long wgs, float *part, int *pace, hipStream_t st)
{
    using S = Shape<NI>;
    constexpr int LDS_BYTES = DIRECT ? S::DIRECT_LDS_BYTES : S::LDS_BYTES;
    static_assert(4 * S::TOKENS * 3 * sizeof(float) <= LDS_BYTES, "LDS");
    static DeviceMask lds_limit_raised{0};
    const hipError_t e = raise_dynamic_lds_limit((const void *)k1_entropy_stream_kernel<NI, D, PIECES, STREAM_W, DIRECT>, LDS_BYTES,
                                                 lds_limit_raised);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((k1_entropy_stream_kernel<NI, D, PIECES, STREAM_W, DIRECT>), dim3((unsigned)wgs), dim3(256), LDS_BYTES, st,
                       (const unsigned char *)w_packed, (const unsigned char *)hidden, (long)T, d, kt, V, p.ntb,
                       p.nsplit, p.tiles_per_split, p.ntiles_v, group, p.whole_cohorts, part, pace);
    return hipGetLastError();
}

}  // namespace

hipError_t k1_entropy_stream(const void *hidden, const void *w_packed, int64_t T, int K, int V,
                             const K1Plan &p, float *part, int *pace, hipStream_t st)
{
    const int kt = k_steps(K);
    if (T <= 0 || p.nsplit < 1 || p.tiles_per_split < 1 || (long)p.nsplit * p.tiles_per_split < p.ntiles_v ||
        (long)(p.nsplit - 1) * p.tiles_per_split >= p.ntiles_v || (long)p.ntb * p.nsplit > 0x7fffffffL ||
        (int64_t)p.ntb * p.tb_tokens < T || p.ntiles_v != (V + p.tile_v - 1) / p.tile_v || kt > K1_STREAM_MAX_STEPS || (p.pieces && (kt % K1_SPLIT_TERMS != 0 || p.direct)))
        return hipErrorInvalidValue;
    const int read = p.pieces ? kt / 2 : kt;  // blocks of W_lm that a sweep needs
    const bool stream = k1_plan_streams_w(p, read);
    const int group = p.tile_v == K1_STREAM_TILE_V ? k1_stream_group(p.nsplit) : 8;
    const long units = (long)p.ntb * p.nsplit, cohorts = k1_stream_cohorts(p.ntb, p.nsplit);
    const long wgs = p.whole_cohorts ? 8 * ((cohorts + 7) / 8) * COHORT : units;
    if (wgs > 0x7fffffffL)
        return hipErrorInvalidValue;
    if (!k1_plan_paces(p))
        pace = nullptr;
#define EGTP_STREAM_OF(NI, D, PIECES, DIRECT)                                                                      \
    (stream ? launch<NI, D, PIECES, true, DIRECT>(hidden, w_packed, T, K, kt, V, p, group, wgs, part, pace, st)      \
            : launch<NI, D, PIECES, false, DIRECT>(hidden, w_packed, T, K, kt, V, p, group, wgs, part, pace, st))
#define EGTP_STREAM(NI, D) \
    (p.pieces ? EGTP_STREAM_OF(NI, D, true, false) : (p.direct ? EGTP_STREAM_OF(NI, D, false, true) : EGTP_STREAM_OF(NI, D, false, false)))
    if (p.tb_tokens == K1_STREAM_TOKENS && p.tile_v == K1_STREAM_TILE_V)
        return EGTP_STREAM(8, 2);
    if (p.tb_tokens == K1_STREAM_WIDE_TOKENS && p.tile_v == K1_NARROW_TILE_V)
        return kt % 4 == 0 ? EGTP_STREAM(12, 4) : EGTP_STREAM(12, 2);
#undef EGTP_STREAM
#undef EGTP_STREAM_OF
    return hipErrorInvalidValue;
}

}  // namespace egtp
