// Entropy-softmax weights and weighted pooling over ragged offsets (Eq. 3, Eq. 4), the
// streaming PLP fold of Eq. 8, the ablation poolers of Table 3, and the ragged plumbing.
//
// Pooling is HBM-bound: every hidden state is read once more (16 bytes per lane, a wave
// reads 1 KiB of one token row at a time).  A sequence is cut into units of at most 256 tokens
// (fewer in a small batch) so that long and short sequences load the chip evenly; each unit leaves a
// partial weighted sum relative to its own largest entropy, with that reference and the sum of its weights, and a
// finalize kernel joins a sequence's units in order.  No atomics: a call is bit-reproducible.  The unit follows the
// batch, so a sequence's sums are grouped differently beside other sequences.
//
// Units need no table: sequence b owns the unit numbers from offsets[b] / unit + b on.  Consecutive sequences
// never meet, because ceil((y - x) / unit) <= floor(y / unit) - floor(x / unit) + 1; of the
// floor(T / unit) + B numbers some stay unused.  (A scan kernel made a table, and another one the
// log-sum-exps, before: two launches more.)
//
// Averages and maxima of large batches of few sequences have the rows of the batch dealt out evenly instead, whatever sequences they
// belong to (pool_rows_kernel; the rule is in pool_deal.h); what workgroup w adds up of sequence b is unit w + b.
#include <type_traits>

#include "k1_common.h"
#include "pool_deal.h"
#include "stream_load.h"
#include "wave_reduce.h"

namespace egtp {
namespace {

constexpr float NEG_INF = -__builtin_inff();

// ---- ragged plumbing ---------------------------------------------------------------------
// offsets[0..B] = exclusive scan of lengths[b]; one workgroup walks the array in chunks
// of 256 with a running carry.
__global__ __launch_bounds__(256) void scan_kernel(const int32_t *__restrict__ in, int32_t B,
                                                   int32_t *__restrict__ out)
{
    __shared__ int sh[256];
    __shared__ int carry;
    const int tid = threadIdx.x;
    if (tid == 0) {
        carry = 0;
        out[0] = 0;
    }
    __syncthreads();
    for (int base = 0; base < B; base += 256) {
        const int b = base + tid;
        sh[tid] = b < B ? in[b] : 0;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {  // inclusive Hillis-Steele scan
            int add = tid >= o ? sh[tid - o] : 0;
            __syncthreads();
            sh[tid] += add;
            __syncthreads();
        }
        if (b < B)
            out[b + 1] = carry + sh[tid];
        __syncthreads();
        if (tid == 255)
            carry += sh[255];
        __syncthreads();
    }
}

// largest b in [0, B) with arr[b] <= t, given arr[0] <= t < arr[B], arr non-decreasing
__device__ __forceinline__ int find_segment(const int32_t *__restrict__ arr, int B, long t)
{
    int lo = 0, hi = B;  // invariant: arr[lo] <= t < arr[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (arr[mid] <= t)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(256) void seg_ids_kernel(const int32_t *__restrict__ offsets, int32_t B,
                                                      long T, int32_t *__restrict__ seg)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= T)
        return;
    seg[t] = (B > 0 && t < offsets[B]) ? find_segment(offsets, B, t) : -1;
}

// Device offsets are the caller's: whatever they hold, no token index leaves [0, T] and no unit
// index leaves the partial buffer (a malformed table gives wrong numbers, not wild accesses).
__device__ __forceinline__ long clamp_token(long t, long T) { return t < 0 ? 0 : (t > T ? T : t); }

// ---- Eq. 4: partial weighted sums per unit --------------------------------------------------
// MODE 0: weights e^{H/alpha - m} / unit (Eq. 3-4), m the unit's largest H/alpha; MODE 1: plain sums (average pooling,
// divided by the length when the units are joined); MODE 2: element-wise maxima.
// The division by the unit, a power of two, changes no bit of a result: it keeps the sum of a unit's weights at or below
// one, so that a partial is no larger than the largest hidden state and cannot overflow where the pooled vector does not.
enum : int { POOL_WEIGHTED = 0, POOL_SUM = 1, POOL_MAXIMUM = 2 };

template <bool BF16, typename Q>
__device__ __forceinline__ void widen16(const Q &q, float (&h)[BF16 ? 8 : 4])
{
    if (BF16) {
        const unsigned v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            h[2 * e] = __uint_as_float(v[e] << 16);
            h[2 * e + 1] = __uint_as_float(v[e] & 0xffff0000u);
        }
    } else {
        h[0] = __uint_as_float(q.x);
        h[1] = __uint_as_float(q.y);
        h[2] = __uint_as_float(q.z);
        h[3] = __uint_as_float(q.w);
    }
}

// first unit number of a sequence that starts at token `begin`
__device__ __forceinline__ long unit_base(int begin, int b, int unit_log2) { return (long)(max(begin, 0) >> unit_log2) + b; }

// the sequence that unit number u belongs to.  Every workgroup starts with this: up to UNIT_SCAN sequences are
// looked through by all threads at once (one memory latency), more of them by bisection.
constexpr int UNIT_SCAN = 2048;
__device__ int unit_sequence(const int32_t *__restrict__ offsets, int B, long u, int unit_log2, int *sh)
{
    if (B > UNIT_SCAN) {
        int lo = 0, hi = B;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (unit_base(offsets[mid], mid, unit_log2) <= u)
                lo = mid;
            else
                hi = mid;
        }
        return lo;
    }
    if (threadIdx.x == 0)
        *sh = 0;
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += 256)
        if (unit_base(offsets[b], b, unit_log2) <= u && u < unit_base(offsets[b + 1], b + 1, unit_log2))
            *sh = b;
    __syncthreads();
    return *sh;
}

// statistics of the whole wave in every lane, by the exchanges of wave_tree
__device__ __forceinline__ Stats wave_merge(Stats a)
{
    auto with = [](const Stats &v, auto ctrl) {
        auto move = [](float f) {
            return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(f), decltype(ctrl)::value, 0xf, 0xf, true));
        };
        return merge(v, Stats{move(v.m), move(v.S), move(v.U)});
    };
    a = with(a, std::integral_constant<int, 0xB1>{});   // lanes 1 apart
    a = with(a, std::integral_constant<int, 0x4E>{});   // 2 apart
    a = with(a, std::integral_constant<int, 0x141>{});  // quads 1 apart: mirrored within 8
    a = with(a, std::integral_constant<int, 0x140>{});  // and within 16
    auto swapped = [](const Stats &v, auto swap) {
        const auto m = swap(__float_as_uint(v.m)), S = swap(__float_as_uint(v.S)), U = swap(__float_as_uint(v.U));
        return merge(Stats{__uint_as_float(m[0]), __uint_as_float(S[0]), __uint_as_float(U[0])},
                     Stats{__uint_as_float(m[1]), __uint_as_float(S[1]), __uint_as_float(U[1])});
    };
    a = swapped(a, [](unsigned u) { return __builtin_amdgcn_permlane16_swap(u, u, false, false); });
    return swapped(a, [](unsigned u) { return __builtin_amdgcn_permlane32_swap(u, u, false, false); });
}

// Eq. 2 finished for a unit: the nsplit partial triples that the fused kernel left for each of its n tokens from t0 on are
// merged by a fixed tree -- 256 / unit threads share a token, thread g of them takes ranges g, g + 256 / unit, ... in
// order, MERGE_AHEAD fetched before any is merged, then halves join halves through LDS.  Thread t < n returns with H of
// token t0 + t.  The slices of a unit each merge for themselves; against a launch of its own in between (two slices and more
// included): four short fp32 prompts 43.2 -> 39.7 us a pass, 173 tokens, d = 4096, V = 151936 274.8 -> 268.7 (different boxes), 2500
// tokens, d = 2048, V = 32000 271 -> 262, 3600 tokens, d = 256 against 151936 rows (many ranges) 429 -> 424.
constexpr int MERGE_AHEAD = 8;
template <int AHEAD = MERGE_AHEAD>
__device__ __forceinline__ float unit_entropy(const float *__restrict__ part, int nsplit, long T, long t0, int n, int unit_log2,
                                              float (&sh)[3][256])
{
    const int tid = threadIdx.x, token = tid & ((1 << unit_log2) - 1), g = tid >> unit_log2, groups = 256 >> unit_log2;
    const long plane = (long)nsplit * T;
    const float *p = part + t0 + min(token, n - 1);
    Stats a = {NEG_BIG, 0.f, 0.f};
    for (int s0 = g; s0 < nsplit; s0 += groups * AHEAD) {
        Stats v[AHEAD];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const float *q = p + (long)min(s0 + i * groups, nsplit - 1) * T;  // past the end: a valid range, not used
            v[i].m = q[0], v[i].S = q[plane], v[i].U = q[2 * plane];
        }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
            if (s0 + i * groups < nsplit)
                a = merge(a, v[i]);
    }
    for (int o = groups >> 1; o > 0; o >>= 1) {
        if (g >= o && g < 2 * o)
            sh[0][tid] = a.m, sh[1][tid] = a.S, sh[2][tid] = a.U;
        __syncthreads();
        if (g < o) {
            const int other = tid + (o << unit_log2);
            a = merge(a, Stats{sh[0][other], sh[1][other], sh[2][other]});
        }
    }
    return logf(a.S) - a.U * 0.6931471805599453f / a.S;
}

// With part != NULL the weighted mode finishes Eq. 2 for its unit's tokens first and writes H to entropy; tokens that no
// sequence holds (a table that begins after 0 or ends before T) get theirs from two units that the grid has beyond
// those of the sequences and from the numbers that these leave unused.  (What a malformed table
// leaves out: pool_finalize_kernel.)
template <bool BF16, int MODE>
__global__ __launch_bounds__(256) void pool_partial_kernel(
    const void *__restrict__ hidden, int d, float *entropy, const float *__restrict__ part, int nsplit,
    const int32_t *__restrict__ offsets, int32_t B, long T, float inv_alpha, int unit_log2, int ysplit,
    const int32_t *__restrict__ slot, const float *state_lse, float *__restrict__ lse_old,
    float *__restrict__ partial, float2 *__restrict__ unit_stats)
{
    __shared__ float w[256];
    __shared__ float red[2][4];
    __shared__ float triples[MODE == POOL_WEIGHTED ? 3 : 1][256];
    __shared__ int seq;
    // Workgroup = (unit, feature slice), the slice varying fastest so that the slices of a unit -- pieces of
    // the same token rows -- are read at about the same time.  The grid holds pool_units_bound(T, B, unit) units:
    // u indexes inside the partial buffer.
    const int u = blockIdx.x / ysplit;
    const int yslice = blockIdx.x - u * ysplit;
    // the states' log-sum-exps, for the join (whose workgroups replace them in place): one workgroup each, there
    // are at least B
    if (MODE == POOL_WEIGHTED && state_lse != nullptr && (int64_t)blockIdx.x < B && threadIdx.x == 0)
        lse_old[blockIdx.x] = state_lse[slot ? slot[blockIdx.x] : blockIdx.x];
    const int b = unit_sequence(offsets, B, u, unit_log2, &seq);
    const int begin = offsets[b];
    const long nth = u - unit_base(begin, b, unit_log2);
    long t0 = clamp_token(begin + (nth << unit_log2), T);
    int n = (int)max(0L, min(1L << unit_log2, clamp_token(offsets[b + 1], T) - t0));
    if (n == 0 || nth < 0 || u >= (T >> unit_log2) + B) {  // an unused number, or one of the two beyond
        if constexpr (MODE == POOL_WEIGHTED)
            if (part != nullptr && yslice == 0) {
                const long first = clamp_token(offsets[0], T), last = clamp_token(offsets[B], T);
                const long behind = u - unit_base((int)last, B, unit_log2);
                long t1 = t0 = 0;
                if (u == (T >> unit_log2) + B + 1)  // before the first sequence: less than a unit ...
                    t0 = (first >> unit_log2) << unit_log2, t1 = first;
                else if (u < (first >> unit_log2))  // ... and whole ones
                    t0 = (long)u << unit_log2, t1 = t0 + (1L << unit_log2);
                else if (behind >= 0)  // behind the last sequence
                    t0 = last + (behind << unit_log2), t1 = min(t0 + (1L << unit_log2), T);
                if (t1 > t0) {
                    const float H = unit_entropy(part, nsplit, T, t0, (int)(t1 - t0), unit_log2, triples);
                    if ((int)threadIdx.x < t1 - t0)
                        entropy[t0 + threadIdx.x] = H;
                }
            }
        return;
    }
    if constexpr (MODE == POOL_WEIGHTED) {
        const int tid = threadIdx.x, wave = tid >> 6;
        static_assert(POOL_UNIT <= 256, "a token per thread");
        float H = 0.f;
        if (part != nullptr) {
            H = unit_entropy(part, nsplit, T, t0, n, unit_log2, triples);
            if (tid < n && yslice == 0)
                entropy[t0 + tid] = H;
        } else if (tid < n) {
            H = entropy[t0 + tid];
        }
        const float a = tid < n ? H * inv_alpha : NEG_INF;
        const float wm = wave_max(a);
        if ((tid & 63) == 0)
            red[0][wave] = wm;
        __syncthreads();
        const float m = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
        const float e = tid < n ? __expf(a - m) : 0.f;
        w[tid] = ldexpf(e, -unit_log2);
        const float ws = wave_sum(e);
        if ((tid & 63) == 0)
            red[1][wave] = ws;
        __syncthreads();
        if (tid == 0 && yslice == 0)
            unit_stats[u] = make_float2(m, (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]));
    }

    constexpr int VEC = BF16 ? 8 : 4;  // elements per 16-byte load
    const int nchunk = d / VEC;
    float *out = partial + (long)u * d;
    // a slice is 256 chunks of 16 bytes, one per thread (two slices at d = 4096: twice as many workgroups as
    // units, which evens out the end of the launch)
    for (int c = yslice * 256 + threadIdx.x; c < nchunk; c += 256 * ysplit) {
        float acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            acc[e] = MODE == POOL_MAXIMUM ? NEG_INF : 0.f;
        const unsigned char *p = (const unsigned char *)hidden + (t0 * d + (long)c * VEC) * (BF16 ? 2 : 4);
        const long stride = (long)d * (BF16 ? 2 : 4);
        auto fold = [&](const u32x4 &q, int i) {
            float h[VEC];
            widen16<BF16>(q, h);
            const float wi = MODE == POOL_WEIGHTED ? w[i] : 1.f;
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                acc[e] = MODE == POOL_MAXIMUM ? fmaxf(acc[e], h[e])
                         : MODE == POOL_SUM   ? acc[e] + h[e]
                                              : fmaf(wi, h[e], acc[e]);
        };
        int i = 0;
        for (; i + 8 <= n; i += 8) {  // eight rows in flight per thread
            u32x4 q[8];
#pragma unroll
            for (int r = 0; r < 8; ++r)
                q[r] = stream_load16(p + (long)(i + r) * stride);
#pragma unroll
            for (int r = 0; r < 8; ++r)
                fold(q[r], i + r);
        }
        for (; i < n; ++i)
            fold(stream_load16(p + (long)i * stride), i);
#pragma unroll
        for (int e = 0; e < VEC; e += 4)
            *(float4 *)(out + (long)c * VEC + e) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
    }
}

// ---- average and maximum of large batches: the batch dealt out evenly ------------------------
// Bound: HBM, and how many streams it is read in.  Workgroup = (rows_per_wg rows of the batch, feature slice), whatever sequences they belong to;
// two workgroups to a compute unit (three with slices of at most 128 chunks), which start together, read the same number of rows and end
// together.  Units of a sequence's own 256 tokens were five or six workgroups to a compute unit, and the launch ended with the sixth: the
// serving batch, 137720 tokens of d = 4096 in bf16, 207.6 us a pass; dealt evenly in five workgroups each 193, four 189, three 191, two 181
// = 6.6 TB/s beside the head (sixteen rows in flight instead of eight 186).  Narrow slices have fewer bytes in flight: 108703 tokens, d = 344 38.4
// us in units, in two, three, four workgroups 35.6, 33.1, 31.8; 60000, d = 512 29.6; 28.8, 25.8, 25.2; but 137720 of d = 264 in fp32 43.1; 42.2, 42.2, 45.9.
// What workgroup w adds up of sequence b is unit w + b: no two meet, since w or b grows from one to the next.  A slice is an even share of the
// 16-byte chunks of a row, at most one per thread (d = 2208 in bf16, 276 chunks, as 256 and 20: 59 us for 37008 tokens, as 138 and 138 42).  The number of
// rows is odd: rows of 8 KiB dealt in 254 or 128 took 190 to 200 us instead of 173.
// Rows are asked for ahead of the sequences' ends (pool_deal.h), which lie in the LDS; a wave holds 64 of them in its lanes and looks through
// these at once for the next sequence that is not empty.
template <bool BF16, int MODE>
__global__ __launch_bounds__(256) void pool_rows_kernel(const void *__restrict__ hidden, int d, const int32_t *__restrict__ offsets, int32_t B,
                                                        long T, int rows_per_wg, int ysplit, int slice, float *__restrict__ partial)
{
    constexpr int VEC = BF16 ? 8 : 4;  // elements per 16-byte load
    constexpr int AHEAD = 8;           // rows in flight per thread
    __shared__ int ends[POOL_DEAL_SEQUENCES];
    __shared__ int first_sh;
    const int w = blockIdx.x / ysplit, yslice = blockIdx.x - w * ysplit, lane = threadIdx.x & 63;
    const int lo = w * rows_per_wg, hi = (int)min((long)lo + rows_per_wg, T);
    // the first row that belongs to a sequence, and the sequence
    const int begin = max(lo, inside_batch(offsets[0], T)), n = hi - begin;
    if (threadIdx.x == 0)
        first_sh = B;
    __syncthreads();
    int first = B;
    for (int i = threadIdx.x; i < B; i += 256) {
        ends[i] = inside_batch(offsets[i + 1], T);
        if (ends[i] > begin)
            first = min(first, i);
    }
    if (first < B)
        atomicMin(&first_sh, first);
    __syncthreads();
    const int b = __builtin_amdgcn_readfirstlane(first_sh);
    // (lanes behind the slice read and write its last chunk as well: no lane is idle where the wave looks through its ends)
    const int first_chunk = yslice * slice, last_chunk = min(first_chunk + slice, d / VEC) - 1;
    if (b == B || n <= 0 || first_chunk + ((int)threadIdx.x & ~63) > last_chunk)
        return;
    const int c = min(first_chunk + (int)threadIdx.x, last_chunk);
    const long stride = (long)d * (BF16 ? 2 : 4);
    const unsigned char *p = (const unsigned char *)hidden + begin * stride + (long)c * 16;
    // A sum begins anew every SUM_ROWS rows, as with units: as one chain of a deal's rows it would lose with the batch (6.3 million tokens that are
    // all 1.00024, 8203 rows: 1.2e-4 off).
    constexpr int SUM_ROWS = 256;
    float acc[VEC], sums[MODE == POOL_SUM ? VEC : 1] = {};
#pragma unroll
    for (int e = 0; e < VEC; ++e)
        acc[e] = MODE == POOL_MAXIMUM ? NEG_INF : 0.f;
    auto add = [&](const u32x4 &q) {
        float h[VEC];
        widen16<BF16>(q, h);
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            acc[e] = MODE == POOL_MAXIMUM ? fmaxf(acc[e], h[e]) : acc[e] + h[e];
    };
    // where 64 sequences from `base` on end, one to a lane
    auto window_at = [&](int base) { return base + lane < B ? ends[base + lane] - begin : INT32_MIN; };
    int base = b, window = window_at(b);
    u32x4 some[AHEAD];
    walk_rows<AHEAD>(
        n, b, B,
        [&](int i) {
            const unsigned char *at = p + i * stride;
            u32x4 q[AHEAD];
#pragma unroll
            for (int r = 0; r < AHEAD; ++r)
                q[r] = stream_load16(at + r * stride);
#pragma unroll
            for (int r = 0; r < AHEAD; ++r)
                add(q[r]);
            if (MODE == POOL_SUM && i % SUM_ROWS == SUM_ROWS - AHEAD)
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    sums[e] += acc[e], acc[e] = 0.f;
        },
        [&](int i) {
#pragma unroll
            for (int r = 0; r < AHEAD; ++r)  // past the end: the last row, not used
                some[r] = stream_load16(p + min(i + r, n - 1) * stride);
#pragma unroll
            for (int r = 0; r < AHEAD; ++r)
                asm volatile("" : "+v"(some[r]));
        },
        [&](int r) {
            widen16<BF16>(some[r], acc);
            if (MODE == POOL_SUM)
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    sums[e] = 0.f;
        },
        [&](int r) { add(some[r]); },
        [&](int at) { return __builtin_amdgcn_readlane(window, at - base); },
        [&](int at, int row) {
            unsigned long long more = __ballot(window > row) & ~1ull << (at - base);
            while (more == 0) {
                base += 64;
                if (base >= B)
                    return B;
                window = window_at(base);
                more = __ballot(window > row);
            }
            return base + __builtin_ctzll(more);
        },
        [&](int at) {
            float *out = partial + (long)(w + at) * d + (long)c * VEC;
            if (MODE == POOL_SUM)
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    acc[e] += sums[e];
#pragma unroll
            for (int e = 0; e < VEC; e += 4)
                *(float4 *)(out + e) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
        });
}

// ---- joining a sequence's units ----------------------------------------------------------------
// Workgroup = JOIN_COLS features of one sequence, four consecutive ones per thread; wave q combines the units
// q, q + 4, ... of the sequence in order, JOIN_AHEAD of them fetched before any is used (one load at a time
// would make the join of a long sequence a chain of memory latencies), and the four waves' results are combined in
// order: bit-reproducible.
constexpr int JOIN_AHEAD = 8, JOIN_FACTORS = 1024, JOIN_COLS = 256;

template <int MODE>
__device__ __forceinline__ void join(float4 &r, const float4 &v, float f)
{
    if (MODE == POOL_MAXIMUM)
        r.x = fmaxf(r.x, v.x), r.y = fmaxf(r.y, v.y), r.z = fmaxf(r.z, v.z), r.w = fmaxf(r.w, v.w);
    else if (MODE == POOL_SUM)
        r.x += v.x, r.y += v.y, r.z += v.z, r.w += v.w;
    else
        r.x = fmaf(f, v.x, r.x), r.y = fmaf(f, v.y, r.y), r.z = fmaf(f, v.z, r.z), r.w = fmaf(f, v.w, r.w);
}

// r joined with this wave's share of the units [u0, u1); POOL_WEIGHTED: unit u counts scale[u - u0] times
template <int MODE>
__device__ __forceinline__ float4 join_units(const float *__restrict__ partial, long u0, long u1, int d, int k,
                                             float4 r, const float *scale)
{
    auto factor = [&](long u) { return MODE == POOL_WEIGHTED ? scale[u - u0] : 1.f; };
    long u = u0 + (threadIdx.x >> 6);
    for (; u + 4 * (JOIN_AHEAD - 1) < u1; u += 4 * JOIN_AHEAD) {
        float4 v[JOIN_AHEAD];
#pragma unroll
        for (int i = 0; i < JOIN_AHEAD; ++i)
            v[i] = *(const float4 *)(partial + (u + 4 * i) * d + k);
#pragma unroll
        for (int i = 0; i < JOIN_AHEAD; ++i)
            join<MODE>(r, v[i], factor(u + 4 * i));
    }
    for (; u < u1; u += 4)
        join<MODE>(r, *(const float4 *)(partial + u * d + k), factor(u));
    return r;
}

// the four waves' results, in wave 0
template <int MODE>
__device__ __forceinline__ float4 join_waves(float4 r, float4 (&sh)[3][64])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave > 0)
        sh[wave - 1][lane] = r;
    __syncthreads();
    if (wave == 0)
#pragma unroll
        for (int q = 0; q < 3; ++q)
            join<MODE == POOL_MAXIMUM ? POOL_MAXIMUM : POOL_SUM>(r, sh[q][lane], 1.f);
    return r;
}

// the unit numbers [u0, u1) of sequence b, inside the partial buffer whatever the offsets hold; only units that hold
// tokens, since the others' partials are not written
__device__ __forceinline__ void sequence_units(const int32_t *__restrict__ offsets, int b, long T, int unit_log2,
                                               long units_cap, long &u0, long &u1)
{
    const int begin = offsets[b];
    const long len = clamp_token(offsets[b + 1], T) - begin;
    u0 = min(unit_base(begin, b, unit_log2), units_cap);
    u1 = min(u0 + (len > 0 ? (len + (1 << unit_log2) - 1) >> unit_log2 : 0), units_cap);
}

// the same for the units of pool_rows_kernel
__device__ __forceinline__ void sequence_row_units(const int32_t *__restrict__ offsets, int b, long T, int rows_per_wg, long &u0, long &u1)
{
    const int t0 = (int)clamp_token(offsets[b], T), t1 = (int)clamp_token(offsets[b + 1], T);
    u0 = t0 / rows_per_wg + b;
    u1 = t1 > t0 ? (t1 - 1) / rows_per_wg + b + 1 : u0;
}

// Table 3 alternatives: sum / length, or maximum.  rows_per_wg > 0: the units are those of pool_rows_kernel
template <int MODE>
__global__ __launch_bounds__(256) void pool_finalize_plain_kernel(const float *__restrict__ partial,
                                                                  const int32_t *__restrict__ offsets, long T,
                                                                  int d, int unit_log2, int rows_per_wg, long units_cap,
                                                                  float *__restrict__ out_pooled)
{
    __shared__ float4 waves[3][64];
    const int b = blockIdx.x;
    const int k = blockIdx.y * JOIN_COLS + (threadIdx.x & 63) * 4;
    long u0, u1;
    if (rows_per_wg > 0)
        sequence_row_units(offsets, b, T, rows_per_wg, u0, u1);
    else
        sequence_units(offsets, b, T, unit_log2, units_cap, u0, u1);
    const int len = offsets[b + 1] - offsets[b];
    const float init = (MODE == POOL_MAXIMUM && u1 > u0) ? NEG_INF : 0.f;  // an empty sequence pools to zero
    float4 r = make_float4(init, init, init, init);
    if (k < d)
        r = join_units<MODE>(partial, u0, u1, d, k, r, nullptr);
    r = join_waves<MODE>(r, waves);
    if (threadIdx.x >= 64 || k >= d)
        return;
    if (MODE == POOL_SUM && len > 0) {
        const float inv = 1.0f / (float)len;
        r.x *= inv, r.y *= inv, r.z *= inv, r.w *= inv;
    }
    *(float4 *)(out_pooled + (long)b * d + k) = r;
}

// Eq. 3, 4 and 8: the log-sum-exp of the units and the old state, the sum of the units' partials brought to it, plus
// the rescaled old state.  Every workgroup of a sequence finds the log-sum-exp for itself.
__global__ __launch_bounds__(256) void pool_finalize_kernel(
    const float *__restrict__ partial, const float2 *__restrict__ unit_stats, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ slot, long T, int d, int unit_log2, long units_cap, const float *state_pooled,
    const float *__restrict__ lse_old, float *out_pooled, float *out_lse, float *__restrict__ entropy,
    const float *__restrict__ part, int nsplit)
{
    __shared__ union {
        float factor[JOIN_FACTORS];
        float triples[3][256];  // of a malformed table's tokens
    } lds;
    __shared__ float4 waves[3][64];
    __shared__ float red[2][4];
    float *const factor = lds.factor;
    const int b = blockIdx.x;
    const int k = blockIdx.y * JOIN_COLS + (threadIdx.x & 63) * 4;
    const int tid = threadIdx.x, wave = tid >> 6;
    const int s = slot ? slot[b] : b;
    const float L_old = lse_old ? lse_old[b] : NEG_INF;
    long u0, u1;
    sequence_units(offsets, b, T, unit_log2, units_cap, u0, u1);
    auto wrong = [&](int i) { return offsets[i + 1] < offsets[i] || offsets[i] < 0; };
    if (__builtin_expect(part != nullptr && wrong(b), 0)) {
        // Entropies belong to the tokens, whatever the table holds.  The units reach every token as long as the offsets begin
        // at 0 or later and do not decrease; the workgroups of the first sequence for which that is not so merge the
        // whole batch's triples.  (Here, two at a time: behind the join the kernel has 66 registers, a wave less per SIMD,
        // and joins 65088 tokens of 1017 sequences in 39.5 us instead of 35.5.)
        bool earlier = false;
        for (int i = threadIdx.x; i < b; i += 256)
            earlier |= wrong(i);
        if (__syncthreads_or(earlier) == 0)
            for (long t0 = (long)blockIdx.y << unit_log2; t0 < T; t0 += (long)gridDim.y << unit_log2) {
                const int n = (int)min(1L << unit_log2, T - t0);
                const float H = unit_entropy<2>(part, nsplit, T, t0, n, unit_log2, lds.triples);
                if ((int)threadIdx.x < n)
                    entropy[t0 + threadIdx.x] = H;
                __syncthreads();  // the triples have been read
            }
    }
    float mx = NEG_INF;
    for (long u = u0 + tid; u < u1; u += 256)
        mx = fmaxf(mx, unit_stats[u].x);
    mx = wave_max(mx);
    if ((tid & 63) == 0)
        red[0][wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3])), L_old);
    float sum = 0.f;
    if (mx > NEG_INF)
        for (long u = u0 + tid; u < u1; u += 256) {
            const float2 q = unit_stats[u];
            sum = fmaf(q.y, __expf(q.x - mx), sum);
        }
    sum = wave_sum(sum);
    if ((tid & 63) == 0)
        red[1][wave] = sum;
    __syncthreads();
    sum = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    // Weights are e^{m - mx} / sum: relative to the log-sum-exp, which is a number around 20, its rounding and that of
    // the difference would go into every weight (distance of a pass's outputs to fp64, 137720 tokens 9.3e-7, now 6.0e-7;
    // 65088 tokens onto states 6.7e-7, now 3.6e-7).
    float L = NEG_INF, sc = 0.f, inv = 0.f;
    if (mx > NEG_INF) {
        const float old = L_old > NEG_INF ? __expf(L_old - mx) : 0.f;
        inv = 1.0f / (sum + old);
        L = mx + __logf(sum + old);
        sc = old * inv;
    }
    if (blockIdx.y == 0 && tid == 0)
        out_lse[s] = L;

    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    for (long c0 = u0; c0 < u1; c0 += JOIN_FACTORS) {
        const long c1 = min(c0 + JOIN_FACTORS, u1);
        __syncthreads();
        for (long u = c0 + tid; u < c1; u += 256)
            factor[u - c0] = ldexpf(__expf(unit_stats[u].x - mx) * inv, unit_log2);  // (partials are divided by the unit)
        __syncthreads();
        if (k < d)
            r = join_units<POOL_WEIGHTED>(partial, c0, c1, d, k, r, factor);
    }
    r = join_waves<POOL_WEIGHTED>(r, waves);
    if (threadIdx.x < 64 && k < d) {
        if (state_pooled && sc != 0.f) {
            const float4 old = *(const float4 *)(state_pooled + (long)s * d + k);
            r.x = fmaf(old.x, sc, r.x), r.y = fmaf(old.y, sc, r.y);
            r.z = fmaf(old.z, sc, r.z), r.w = fmaf(old.w, sc, r.w);
        }
        *(float4 *)(out_pooled + (long)s * d + k) = r;
    }
}

// ---- Eq. 8 fast path: exactly one new token per sequence ------------------------------------
// With part != NULL the kernel first finishes Eq. 2 for its token -- the nsplit partial (m, S, U) triples the
// fused kernel left for it are merged by a fixed tree (thread i takes ranges i, i + 256, ... in order, then an
// xor tree inside each wave, then the four waves in order) -- and writes H to entropy[b]; otherwise entropy[b]
// is read.
// The token and its state are asked for before the triples are merged: FOLD_AHEAD chunks per thread (all of them up to d = 4096 in
// bf16), so that the kernel is two memory latencies long, not three; lanes
// exchange without the LDS.  24 sequences, d = 4096, V = 151936 6.0 -> 5.4 us (of a step of 213: no more than two runs of one differ by).
constexpr int FOLD_AHEAD = 2;

template <bool BF16>
__global__ __launch_bounds__(256) void plp_fold1_kernel(const void *__restrict__ hidden, int d, float *entropy,
                                                        const float *__restrict__ part, int nsplit, long T,
                                                        const int32_t *__restrict__ slot, float inv_alpha,
                                                        float *pooled_state, float *lse_state)
{
    __shared__ float red[4][3];
    constexpr int VEC = BF16 ? 8 : 4;
    const int b = blockIdx.x, tid = threadIdx.x;
    const int s = slot ? slot[b] : b;
    const int nchunk = d / VEC;
    const unsigned char *hp = (const unsigned char *)hidden + (long)b * d * (BF16 ? 2 : 4);
    float *pp = pooled_state + (long)s * d;
    struct Chunk {
        uint4 h;
        float4 p[VEC / 4];
    } ahead[FOLD_AHEAD];
    auto load = [&](Chunk &q, int c) {
        q.h = *(const uint4 *)(hp + (long)c * 16);
#pragma unroll
        for (int e = 0; e < VEC / 4; ++e)
            q.p[e] = *(const float4 *)(pp + (long)c * VEC + 4 * e);
    };
    const float L_old = lse_state[s];
#pragma unroll
    for (int i = 0; i < FOLD_AHEAD; ++i)  // past the end: the last chunk, not used
        load(ahead[i], min(tid + 256 * i, nchunk - 1));
    float H;
    if (part != nullptr) {
        const long plane = (long)nsplit * T;
        Stats acc = {NEG_BIG, 0.f, 0.f};
        for (int r = tid; r < nsplit; r += 256) {
            const long idx = (long)r * T + b;
            acc = merge(acc, Stats{part[idx], part[plane + idx], part[2 * plane + idx]});
        }
        acc = wave_merge(acc);
        if ((tid & 63) == 0) {
            red[tid >> 6][0] = acc.m;
            red[tid >> 6][1] = acc.S;
            red[tid >> 6][2] = acc.U;
        }
        __syncthreads();
        acc = {red[0][0], red[0][1], red[0][2]};
#pragma unroll
        for (int k = 1; k < 4; ++k)
            acc = merge(acc, Stats{red[k][0], red[k][1], red[k][2]});
        H = logf(acc.S) - acc.U * 0.6931471805599453f / acc.S;
        if (tid == 0)
            entropy[b] = H;
    } else {
        H = entropy[b];
    }
    const float a = H * inv_alpha;
    const float M = fmaxf(L_old, a);
    const float old = L_old > NEG_INF ? __expf(L_old - M) : 0.f;
    const float L = M + __logf(old + __expf(a - M));
    const float sc = L_old > NEG_INF ? __expf(L_old - L) : 0.f;
    const float wn = __expf(a - L);
    __syncthreads();  // every thread has read the old lse before it is replaced
    if (tid == 0)
        lse_state[s] = L;

    for (int c0 = 0; c0 < nchunk; c0 += 256 * FOLD_AHEAD) {
#pragma unroll
        for (int i = 0; i < FOLD_AHEAD; ++i) {
            const int c = c0 + tid + 256 * i;
            if (c >= nchunk)
                break;
            if (c0 > 0)
                load(ahead[i], c);
            float h[VEC];
            widen16<BF16>(ahead[i].h, h);
#pragma unroll
            for (int e = 0; e < VEC / 4; ++e) {
                float4 p = ahead[i].p[e];
                if (sc == 0.f)  // an empty state's vector does not count, whatever it holds
                    p = make_float4(0.f, 0.f, 0.f, 0.f);
                p.x = fmaf(p.x, sc, wn * h[4 * e]);
                p.y = fmaf(p.y, sc, wn * h[4 * e + 1]);
                p.z = fmaf(p.z, sc, wn * h[4 * e + 2]);
                p.w = fmaf(p.w, sc, wn * h[4 * e + 3]);
                *(float4 *)(pp + (long)c * VEC + 4 * e) = p;
            }
        }
    }
}

// ---- Table 3 alternative: the last token's hidden state ------------------------------------
template <bool BF16>
__global__ __launch_bounds__(256) void pool_last_kernel(const void *__restrict__ hidden, int d,
                                                        const int32_t *__restrict__ offsets, long T,
                                                        float *__restrict__ out_pooled)
{
    constexpr int VEC = BF16 ? 8 : 4;
    const int b = blockIdx.x;
    const int c = blockIdx.y * 256 + threadIdx.x;
    if (c * VEC >= d)
        return;
    const long lo = clamp_token(offsets[b], T), hi = clamp_token(offsets[b + 1], T);
    float h[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e)
        h[e] = 0.f;  // an empty sequence pools to zero
    if (hi > lo) {
        const uint4 q = *(const uint4 *)((const unsigned char *)hidden + ((hi - 1) * d + (long)c * VEC) * (BF16 ? 2 : 4));
        widen16<BF16>(q, h);
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e)
        out_pooled[(long)b * d + (long)c * VEC + e] = h[e];
}

}  // namespace

// Tokens per unit: 256, halved while a batch makes fewer than POOL_WORKGROUPS workgroups and the smaller units'
// partials fit `cap_floats`.  A workgroup walks its unit's rows eight at a time, one memory latency each: 173 tokens,
// d = 4096 in units of 128 are 6 workgroups of 16 latencies (14 us), in units of 16 25 of two (7 us).  Large units
// leave fewer partials to write and join: weighted pooling and join of 137720 tokens, d = 4096, 128 sequences take 207 us with 256, 208 with 128, 221
// with 64; average pooling of 10689 tokens, d = 2048, 30.3 us where 256 workgroups are asked for, 32.6 with 512 or 1024.
constexpr int POOL_UNIT_MIN = 16, POOL_WORKGROUPS = 256;

// workgroups a unit's features are spread over: one 16-byte chunk per thread
static unsigned pool_feature_split(int d, bool bf16)
{
    const int nchunk = d / (bf16 ? 8 : 4);
    const int n = (nchunk + 255) / 256;
    return (unsigned)(n < 1 ? 1 : (n > 64 ? 64 : n));
}

int pool_unit(int dtype, int d, int64_t T, int32_t B, size_t cap_floats)
{
    int unit = POOL_UNIT;
    const int64_t ysplit = pool_feature_split(d, dtype == DT_BF16);
    while (unit > POOL_UNIT_MIN && (T / unit) * ysplit < POOL_WORKGROUPS &&
           pool_unit_floats(d, T, B, unit / 2) <= cap_floats)
        unit /= 2;
    return unit;
}

hipError_t scan_lengths(const int32_t *lengths, int32_t B, int32_t *offsets, hipStream_t st)
{
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(256), 0, st, lengths, B, offsets);
    return hipGetLastError();
}

hipError_t segment_ids(const int32_t *offsets, int32_t B, int64_t T, int32_t *seg, hipStream_t st)
{
    if (T <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(seg_ids_kernel, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, st, offsets, B,
                       (long)T, seg);
    return hipGetLastError();
}

hipError_t pool_entropy_weighted(const PoolArgs &a, hipStream_t st)
{
    if (a.B <= 0)
        return hipSuccess;
    const bool bf16 = a.dtype == DT_BF16;
    if (a.offsets == nullptr) {  // one new token per sequence, folded in place
        if (bf16)
            hipLaunchKernelGGL(plp_fold1_kernel<true>, dim3(a.B), dim3(256), 0, st, a.hidden, a.d, a.entropy,
                               a.k1_part, a.k1_nsplit, (long)a.T, a.slot, a.inv_alpha, a.out_pooled, a.out_lse);
        else
            hipLaunchKernelGGL(plp_fold1_kernel<false>, dim3(a.B), dim3(256), 0, st, a.hidden, a.d, a.entropy,
                               a.k1_part, a.k1_nsplit, (long)a.T, a.slot, a.inv_alpha, a.out_pooled, a.out_lse);
        return hipGetLastError();
    }
    const long units = pool_units_bound(a.T, a.B, a.unit), grid = units + (a.k1_part ? 2 : 0);
    const unsigned ysplit = pool_feature_split(a.d, bf16);
    if (grid * ysplit > 0x7fffffffL)
        return hipErrorInvalidValue;
    float2 *stats = (float2 *)a.unit_stats;
    const int unit_log2 = __builtin_ctz(a.unit);
    if (bf16)
        hipLaunchKernelGGL((pool_partial_kernel<true, POOL_WEIGHTED>), dim3((unsigned)(grid * ysplit)), dim3(256), 0, st, a.hidden,
                           a.d, a.entropy, a.k1_part, a.k1_nsplit, a.offsets, a.B, (long)a.T, a.inv_alpha, unit_log2, (int)ysplit, a.slot, a.state_lse,
                           a.lse_old, a.partial, stats);
    else
        hipLaunchKernelGGL((pool_partial_kernel<false, POOL_WEIGHTED>), dim3((unsigned)(grid * ysplit)), dim3(256), 0, st, a.hidden,
                           a.d, a.entropy, a.k1_part, a.k1_nsplit, a.offsets, a.B, (long)a.T, a.inv_alpha, unit_log2, (int)ysplit, a.slot, a.state_lse,
                           a.lse_old, a.partial, stats);
    hipLaunchKernelGGL(pool_finalize_kernel, dim3(a.B, (a.d + JOIN_COLS - 1) / JOIN_COLS), dim3(256), 0, st, a.partial, stats, a.offsets,
                       a.slot, (long)a.T, a.d, unit_log2, units, a.state_pooled, a.state_lse ? a.lse_old : nullptr, a.out_pooled,
                       a.out_lse, a.entropy, a.k1_part, a.k1_nsplit);
    return hipGetLastError();
}

hipError_t pool_plain(const void *hidden, int dtype, int d, const int32_t *offsets, int32_t B, int64_t T,
                      int kind, int unit, float *partial, size_t cap_floats, float *out_pooled, hipStream_t st)
{
    if (B <= 0)
        return hipSuccess;
    const bool bf16 = dtype == DT_BF16;
    if (kind == 2) {  // last token: one row per sequence
        const int vec = bf16 ? 8 : 4;
        const dim3 grid(B, (d / vec + 255) / 256);
        if (bf16)
            hipLaunchKernelGGL(pool_last_kernel<true>, grid, dim3(256), 0, st, hidden, d, offsets, (long)T,
                               out_pooled);
        else
            hipLaunchKernelGGL(pool_last_kernel<false>, grid, dim3(256), 0, st, hidden, d, offsets, (long)T,
                               out_pooled);
        return hipGetLastError();
    }
    // average and maximum stream every token once
    const dim3 fgrid(B, (d + JOIN_COLS - 1) / JOIN_COLS);
    const unsigned ysplit = pool_feature_split(d, bf16);
    const int nchunk = d / (bf16 ? 8 : 4), slice = (nchunk + (int)ysplit - 1) / (int)ysplit;
    // The even deal (rows of at most 64 slices) where the rule is for it and its units fit ...
    const Deal deal = pool_deal(T, B, slice, ysplit, bf16);
    const bool even = deal.even && slice <= 256 && (size_t)(deal.deals + B) * (size_t)d <= cap_floats && deal.deals * ysplit <= 0x7fffffffL;
    // ... otherwise the same units as Eq. 4
    const long units = even ? (long)(deal.deals + B) : pool_units_bound(T, B, unit);
    const int unit_log2 = __builtin_ctz(unit);
    if (units * ysplit > 0x7fffffffL)
        return hipErrorInvalidValue;
#define EGTP_POOL_PLAIN(BF, MODE)                                                                          \
    do {                                                                                                   \
        if (even)                                                                                          \
            hipLaunchKernelGGL((pool_rows_kernel<BF, MODE>), dim3((unsigned)(deal.deals * ysplit)), dim3(256), 0, st, hidden, d, offsets, B, \
                               (long)T, (int)deal.rows, (int)ysplit, slice, partial);                           \
        else                                                                                               \
            hipLaunchKernelGGL((pool_partial_kernel<BF, MODE>), dim3((unsigned)(units * ysplit)), dim3(256), 0, st, hidden, \
                               d, nullptr, nullptr, 0, offsets, B, (long)T, 0.f, unit_log2, (int)ysplit, nullptr, nullptr, nullptr,    \
                               partial, nullptr);                                                          \
        hipLaunchKernelGGL(pool_finalize_plain_kernel<MODE>, fgrid, dim3(256), 0, st, partial, offsets, (long)T, d, \
                           unit_log2, even ? (int)deal.rows : 0, units, out_pooled);                            \
    } while (0)
    if (kind == 0) {
        if (bf16)
            EGTP_POOL_PLAIN(true, POOL_SUM);
        else
            EGTP_POOL_PLAIN(false, POOL_SUM);
    } else {
        if (bf16)
            EGTP_POOL_PLAIN(true, POOL_MAXIMUM);
        else
            EGTP_POOL_PLAIN(false, POOL_MAXIMUM);
    }
#undef EGTP_POOL_PLAIN
    return hipGetLastError();
}

}  // namespace egtp
