// The part of a prediction head behind layer 1, shared by scoring and training.  Device-side header.
//
// Layer 1 is split along d into slices that leave partial pre-activations in planes act_part[slice][sequence][d_h].
// What follows is a chain of memory latencies -- planes, W2, the softmax between them -- on a few hundred kilobytes, so
// it runs on workgroups of TAIL_THREADS threads that keep every load of a stage in flight at once: NS sequences each,
// four groups of 256 threads (narrow heads: sixteen of 64) that share the planes of a sequence; W2 is asked for before the planes are
// added up, and its registers serve all NS sequences.  The code is kept short and without branches around loads: a workgroup
// runs it once, so every instruction is a cold fetch (the same stages in 18 KB of code took 9.8 us where 5.5 KB take 6.0: one
// sequence, 20 bins, d_h = 1024).  Against workgroups of 256 threads with a sequence each: 9.6 -> 6.0 us there; d_h no multiple
// of four: 127 sequences, d_h = 1077, scalar 17.4 -> 6.5; 416, d_h = 1061, 33 bins 15.8 -> 10.4; training samples
// (k4_train.hip), 20 bins, d_h = 1024: 16 of them 11.5 -> 8.4, 1024 17.4 -> 13.1.
// Sums run in a fixed order: bit-reproducible.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "wave_reduce.h"

namespace egtp {
namespace {

constexpr int TAIL_THREADS = 1024, TAIL_WAVES = TAIL_THREADS / 64;
constexpr int TAIL_PLANES = 8;  // planes in flight per thread
// Columns in a pass; rows of hidden units in LDS are zero-padded to whole passes.  Heads of up to 256 units have passes of their own: in
// wide ones most of their loads were of columns that do not exist, and one group of threads took d loss / d hidden of all samples while
// the others waited.  The samples' kernel, 20 bins, with workgroups of 256 threads and a sample each / wide passes / narrow
// ones (us): 65 samples, d = 256, d_h = 64 7.3 / 9.1 / 6.6, 128, 256, 256 7.6 / 9.0 / 6.5, 300, 256, 128 7.8 / 9.5 / 7.7, 512, 256, 256 9.2 /
// 10.4 / 7.8, 700, 256, 64 7.7 / 9.2 / 8.3, and at d = 1024, d_h = 128 10.8 to 11.6 / - / 7.3 to 8.8 for 65 to 768.  Heads of fewer than four units took one
// sequence a workgroup: 3000 sequences, d_h = 2, scalar 5.8 / 34.8 / 10.2, 600 3.2 / 10.1 / 4.6.
enum TailRow { TAIL_TINY, TAIL_NARROW, TAIL_WIDE };  // fewer than four columns (no whole chunk), up to 256, more
constexpr int TAIL_NARROW_COLS = 256, TAIL_WIDE_COLS = 1024;
__host__ __device__ constexpr TailRow tail_kind(int d_h) { return d_h < 4 ? TAIL_TINY : (d_h <= TAIL_NARROW_COLS ? TAIL_NARROW : TAIL_WIDE); }
template <TailRow ROW>
struct TailPass {
    static constexpr int COLS = ROW == TAIL_WIDE ? TAIL_WIDE_COLS : TAIL_NARROW_COLS;
    static constexpr int GROUP = COLS / 4;     // threads that cover a row
    static constexpr int CHUNKS = COLS / 256;  // chunks of four columns of a W2 row that a lane holds
};
constexpr int TAIL_OUTS = 2;    // rows of W2 that a wave holds (three: 33 bins 10.4 us instead of 11.3, 20 bins 9.4 instead of 8.4)

// The four columns of chunk c of a row of n: 4 c to 4 c + 3, or, where that would run past the row, the last four; of those only
// the ones that no earlier chunk holds count (keep).  So every chunk is one vector load inside the row, and LDS rows
// of hidden units hold chunk c at 4 c with zeros in the places that do not count.  TINY: fewer than four columns.
template <bool TINY>
struct RowChunk {
    int at;
    bool keep[4];
    __device__ __forceinline__ RowChunk(int c, int n)
    {
        at = TINY ? 0 : min(4 * c, n - 4);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            keep[e] = TINY ? c == 0 && e < n : e >= 4 * c - at;
    }
};

// place of column j in an LDS row of hidden units
__device__ __forceinline__ int hidden_place(int j, int n) { return j < (n & ~3) || n < 4 ? j : j + 4 - (n & 3); }

__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(unsigned short v) { return __uint_as_float((unsigned)v << 16); }

// a chunk as it lies in memory.  Rows may begin at any element: the hardware takes vector loads there, the type tells
// the compiler.
template <typename W>
struct ChunkType {
    typedef __attribute__((ext_vector_type(4), aligned(sizeof(W)))) W type;
};
template <typename W>
using ChunkOf = typename ChunkType<W>::type;
template <bool TINY, typename W>
__device__ __forceinline__ ChunkOf<W> load_chunk(const W *__restrict__ row, const RowChunk<TINY> &c, int n)
{
    if (TINY)
        return ChunkOf<W>{row[0], row[min(1, n - 1)], row[min(2, n - 1)], row[0]};
    return *(const ChunkOf<W> *)(row + c.at);
}
// s + the chunk's weights times hidden units v
template <bool TINY, typename Q>
__device__ __forceinline__ float chunk_dot(const Q &w, const RowChunk<TINY> &c, const float4 &v, float s)
{
    s = fmaf(c.keep[0] ? widen(w[0]) : 0.f, v.x, s);
    s = fmaf(c.keep[1] ? widen(w[1]) : 0.f, v.y, s);
    s = fmaf(c.keep[2] ? widen(w[2]) : 0.f, v.z, s);
    return fmaf(c.keep[3] ? widen(w[3]) : 0.f, v.w, s);
}

// what the groups of a workgroup that share a sequence's planes pass to the first of them (four columns a thread)
template <TailRow ROW, int NS>
constexpr int tail_joins = TAIL_THREADS > NS * TailPass<ROW>::GROUP ? TAIL_THREADS - NS * TailPass<ROW>::GROUP : 1;

// hidden units of NS sequences from b0 on: ReLU(sum of the planes + bias) into a[NS][lda] (LDS) and, if `copy` is
// given, into copy[B][d_h].  `join`: tail_joins<ROW, NS> elements of LDS.  Ends with a barrier.
template <TailRow ROW, int NS>
__device__ __forceinline__ void hidden_units(const float *__restrict__ act_part, int nks, int B, int b0, int d_h,
                                             const float *__restrict__ b1, float *a, int lda, float4 *join,
                                             float *__restrict__ copy)
{
    constexpr bool TINY = ROW == TAIL_TINY;
    constexpr int GROUP = TailPass<ROW>::GROUP, GROUPS = TAIL_THREADS / GROUP / NS;  // thread groups per sequence
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / GROUP), t = threadIdx.x % GROUP;
    const int seq = group / GROUPS, part = group % GROUPS;
    const int b = min(b0 + seq, B - 1);  // past the batch: the last sequence, not kept
    const int per = (nks + GROUPS - 1) / GROUPS, s_begin = part * per, s_end = min(nks, s_begin + per);
    const long plane = (long)B * d_h;
    for (int col0 = 0; col0 < lda; col0 += TailPass<ROW>::COLS) {
        const RowChunk<TINY> c(col0 / 4 + t, d_h);
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
        ChunkOf<float> bias = {0.f, 0.f, 0.f, 0.f};
        if (b1 != nullptr)
            bias = load_chunk(b1, c, d_h);
        for (int s0 = s_begin; s0 < s_end; s0 += TAIL_PLANES) {
            ChunkOf<float> v[TAIL_PLANES];
            const float *p = act_part + s0 * plane + (long)b * d_h;
#pragma unroll
            for (int i = 0; i < TAIL_PLANES; ++i) {
                v[i] = load_chunk(p, c, d_h);
                p += s0 + i + 1 < s_end ? plane : 0;  // past the end: a valid plane, not used
            }
#pragma unroll
            for (int i = 0; i < TAIL_PLANES; ++i)
                if (s0 + i < s_end)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        sum[e] += v[i][e];
        }
        if (GROUPS > 1) {
            if (col0 > 0)
                __syncthreads();  // the joins of the previous pass have been read
            if (part > 0)
                join[(seq * (GROUPS - 1) + part - 1) * GROUP + t] = make_float4(sum[0], sum[1], sum[2], sum[3]);
            __syncthreads();
            if (part == 0)
#pragma unroll
                for (int q = 0; q < GROUPS - 1; ++q) {
                    const float4 o = join[(seq * (GROUPS - 1) + q) * GROUP + t];
                    sum[0] += o.x, sum[1] += o.y, sum[2] += o.z, sum[3] += o.w;
                }
        }
        if (part == 0) {
            const bool kept = copy != nullptr && b0 + seq < B;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float r = sum[e] + bias[e];
                sum[e] = c.keep[e] && r > 0.f ? r : 0.f;
                if (kept && c.keep[e])
                    copy[(long)b * d_h + c.at + e] = sum[e];
            }
            *(float4 *)(a + seq * lda + col0 + 4 * t) = make_float4(sum[0], sum[1], sum[2], sum[3]);
        }
    }
    __syncthreads();
}

// outputs z[NS][n_out] (LDS) = W2 a, without the bias; wave w takes rows w, w + 16, ...  `fetched`, between the first loads
// of W2 and their use, makes the hidden units.  No barrier at the end.
template <TailRow ROW, int NS, typename W, class F>
__device__ __forceinline__ void output_layer(const W *__restrict__ w2, int n_out, int d_h, const float *a, int lda, float *z,
                                             F fetched)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr bool TINY = ROW == TAIL_TINY;
    constexpr int CHUNKS = TailPass<ROW>::CHUNKS;
    ChunkOf<W> w[TAIL_OUTS][CHUNKS];
    auto load = [&](int o0, int col0) {
#pragma unroll
        for (int q = 0; q < TAIL_OUTS; ++q)
            if (o0 + q * TAIL_WAVES < n_out)
#pragma unroll
                for (int i = 0; i < CHUNKS; ++i)
                    w[q][i] = load_chunk(w2 + (long)(o0 + q * TAIL_WAVES) * d_h, RowChunk<TINY>(col0 / 4 + 64 * i + lane, d_h), d_h);
    };
    load(wave, 0);
    fetched();
    for (int o0 = wave; o0 < n_out; o0 += TAIL_OUTS * TAIL_WAVES) {
        float s[TAIL_OUTS][NS];
#pragma unroll
        for (int q = 0; q < TAIL_OUTS; ++q)
#pragma unroll
            for (int n = 0; n < NS; ++n)
                s[q][n] = 0.f;
        for (int col0 = 0; col0 < lda; col0 += TailPass<ROW>::COLS) {
            if (o0 != wave || col0 > 0)
                load(o0, col0);
#pragma unroll
            for (int i = 0; i < CHUNKS; ++i) {
                const RowChunk<TINY> c(col0 / 4 + 64 * i + lane, d_h);
#pragma unroll
                for (int n = 0; n < NS; ++n) {
                    const float4 v = *(const float4 *)(a + n * lda + col0 + 256 * i + 4 * lane);
#pragma unroll
                    for (int q = 0; q < TAIL_OUTS; ++q)  // a row past the end: computed from what is there, dropped
                        s[q][n] = chunk_dot(w[q][i], c, v, s[q][n]);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < TAIL_OUTS; ++q)
#pragma unroll
            for (int n = 0; n < NS; ++n) {
                const float t = wave_sum(s[q][n]);
                if (lane == 0 && o0 + q * TAIL_WAVES < n_out)
                    z[n * n_out + o0 + q * TAIL_WAVES] = t;
            }
    }
}

// floats of an LDS row of hidden units
__host__ __device__ __forceinline__ int tail_row(int d_h)
{
    return d_h <= TAIL_NARROW_COLS ? TAIL_NARROW_COLS : (d_h + TAIL_WIDE_COLS - 1) / TAIL_WIDE_COLS * TAIL_WIDE_COLS;
}

// Sequences per workgroup: one while every compute unit gets at most two of them, more for larger batches, which are
// bound by the reads of W2, as long as the rows fit LDS.
constexpr size_t TAIL_LDS_LIMIT = 96 * 1024;
inline int tail_sequences(int32_t B, size_t lds_per_sequence)
{
    int ns = B > 512 ? 4 : (B > 256 ? 2 : 1);
    while (ns > 1 && ns * lds_per_sequence > 64 * 1024)
        ns /= 2;
    return ns;
}

// launch(row kind, sequences per workgroup), both as constants
template <class F>
inline hipError_t tail_launch(int d_h, int ns, F launch)
{
    auto of = [&](auto row) {
        return ns == 4   ? launch(row, std::integral_constant<int, 4>{})
               : ns == 2 ? launch(row, std::integral_constant<int, 2>{})
                         : launch(row, std::integral_constant<int, 1>{});
    };
    const TailRow kind = tail_kind(d_h);
    return kind == TAIL_TINY     ? of(std::integral_constant<TailRow, TAIL_TINY>{})
           : kind == TAIL_NARROW ? of(std::integral_constant<TailRow, TAIL_NARROW>{})
                                 : of(std::integral_constant<TailRow, TAIL_WIDE>{});
}

}  // namespace
}  // namespace egtp
