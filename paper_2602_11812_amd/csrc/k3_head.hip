// Prediction head (Section 3.2): pooled vector -> perceptron d -> d_h (ReLU) -> n_out, then
// either the scalar itself (n_out == 1) or the expected value over K bins of Eq. 6.
//
// Layer 1 is a small [B x d] . [d x d_h] contraction kept entirely in fp32 (the pooled
// vector is never re-rounded), on the fp32 matrix instructions where the weights are fp32 and the batch is more
// than a handful, and as products of bf16 pieces where it is more than 64.  The contraction is split along d so that several hundred workgroups exist even for one
// small batch; the splits leave partial pre-activations that layer 2 adds in a fixed order
// (bit-reproducible) before bias and ReLU.  Layer 2 and the K-bin decode: head_tail.h.
//
// With bf16 weights and d a multiple of 8, layer 1 runs on the bf16 matrix cores without
// rounding the pooled vector: an fp32 value is the exact sum of three bf16 values (its top 8
// significant bits, the top 8 of what is left, and the rest), a bf16 x bf16 product is exact in
// fp32, so three MFMAs per weight fragment accumulate the same products an fp32 dot product
// would, in fp32.  Fragments come straight from global memory: a lane's 8 K-elements are 16
// contiguous bytes of a weight row and 32 contiguous bytes of a pooled row.
#include "head_tail.h"
#include "kernels.h"
#include "split_mfma.h"
#include "wave_reduce.h"

namespace egtp {
namespace {

typedef split_bf16x8 bf16x8;
typedef split_f32x4 f32x4;
typedef split_u32x4 u32x4;

constexpr int TM = 64;  // head rows j per tile
constexpr int TN = 64;  // sequences per tile
constexpr int TK = 16;
constexpr int PAD = 4;

// Layer 1, bf16 weights whose rows are not 16-byte aligned (d a multiple of 4 only): fp32 FMAs.
__global__ __launch_bounds__(256) void head_layer1_kernel(const float *__restrict__ x,
                                                          const int32_t *__restrict__ slot, int B, int d,
                                                          int d_h, const unsigned short *__restrict__ w1, int kchunk,
                                                          float *__restrict__ act_part)
{
    __shared__ float As[TK][TM + PAD];  // As[k][j]
    __shared__ float Bs[TK][TN + PAD];  // Bs[k][sequence]
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int j0 = blockIdx.x * TM, s0 = blockIdx.y * TN;

    const int lrow = tid >> 2;
    const int lk = (tid & 3) * 4;
    int jrow = j0 + lrow;
    jrow = jrow < d_h ? jrow : d_h - 1;  // clamped rows are computed and dropped
    int srow = s0 + lrow;
    srow = srow < B ? srow : B - 1;
    const long xrow = slot ? slot[srow] : srow;
    const float *xp = x + xrow * (long)d;

    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[i][j] = 0.f;

    const int kbeg = blockIdx.z * kchunk;
    const int kend = min(d, kbeg + kchunk);
    float *act = act_part + (long)blockIdx.z * B * d_h;
    for (int k0 = kbeg; k0 < kend; k0 += TK) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
        if (k0 + lk < kend) {
            const uint2 q = *(const uint2 *)(w1 + (long)jrow * d + k0 + lk);
            a.x = __uint_as_float(q.x << 16);
            a.y = __uint_as_float(q.x & 0xffff0000u);
            a.z = __uint_as_float(q.y << 16);
            a.w = __uint_as_float(q.y & 0xffff0000u);
            b = *(const float4 *)(xp + k0 + lk);
        }
        __syncthreads();
        As[lk + 0][lrow] = a.x;
        As[lk + 1][lrow] = a.y;
        As[lk + 2][lrow] = a.z;
        As[lk + 3][lrow] = a.w;
        Bs[lk + 0][lrow] = b.x;
        Bs[lk + 1][lrow] = b.y;
        Bs[lk + 2][lrow] = b.z;
        Bs[lk + 3][lrow] = b.w;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < TK; ++k) {
            const float4 av = *(const float4 *)&As[k][tx * 4];
            const float4 bv = *(const float4 *)&Bs[k][ty * 4];
            const float aa[4] = {av.x, av.y, av.z, av.w};
            const float bb[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = fmaf(aa[i], bb[j], acc[i][j]);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int s = s0 + ty * 4 + j;
        if (s >= B)
            continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int jj = j0 + tx * 4 + i;
            if (jj < d_h)
                act[(long)s * d_h + jj] = acc[i][j];
        }
    }
}

// Layer 1 for at most SK_SEQS sequences and fp32 weights (a training batch, a handful of requests): the work is
// one pass over W1, so the kernel is built around streaming it.  Workgroup = 16 head rows x one slice of at most
// SK_SLICE elements of d; the slice of all pooled vectors sits in LDS (zero rows for missing sequences).  A wave
// owns 4 rows; lane l takes K elements 4l .. 4l+3 of every 256: one 16-byte load per row, sixteen 16-byte LDS
// reads, 256 FMAs into 4 x 16 accumulators.  The 64 accumulators are then summed over the 64 lanes by a halving
// butterfly (a lane passes on the half it does not keep: 63 exchanges instead of 384), which leaves lane l with
// the total of (row l / 16, sequence l % 16).  Fixed order: bit-reproducible.
constexpr int SK_SEQS = 16, SK_SLICE = 512, SK_ROWS = 16;

__global__ __launch_bounds__(256) void head_layer1_skinny_kernel(const float *__restrict__ x,
                                                                 const int32_t *__restrict__ slot, int B, int d,
                                                                 int d_h, const float *__restrict__ w1, int kchunk,
                                                                 float *__restrict__ act_part)
{
    __shared__ __align__(16) float xs[SK_SEQS][SK_SLICE];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int kbeg = blockIdx.y * kchunk;
    const int klen = min(d - kbeg, kchunk);  // a multiple of 4; <= 0 past the end of d: the plane is zeros
    // lane b learns the state row of sequence b (asked for first: the counter of outstanding loads is in order)
    int my_row = lane < B ? lane : 0;
    if (slot)
        my_row = slot[my_row];
    // this lane's share of W1 next -- all of it in flight at once: a load per pass would be as many HBM
    // latencies in a row
    const int j0 = blockIdx.x * SK_ROWS + wave * 4;
    constexpr int PASSES = SK_SLICE / 256;
    float4 wv[PASSES][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int j = j0 + r < d_h ? j0 + r : d_h - 1;  // clamped rows are computed and dropped
        const float *wrow = w1 + (long)j * d + (klen > 0 ? kbeg : 0);
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            // pieces past the end of the slice: load piece 0 instead (no branch around a load, so that the
            // loads stay countable and the waits below can be exact); the staged vectors are zero there
            const int k = 4 * lane + 256 * p;
            wv[p][r] = *(const float4 *)(wrow + (k < klen ? k : 0));
        }
    }
    // meanwhile stage the slice of the pooled vectors, every thread the same 16-byte piece of several rows.  All
    // its loads are issued before the first store (addresses are clamped, not branched on: a wait per row
    // would be sixteen cache latencies in a row); rows and pieces that do not exist become zeros.
    constexpr int PIECES = SK_SLICE / 4;      // 16-byte pieces per staged row
    constexpr int ROWS_AT_ONCE = 256 / PIECES;  // rows the 256 threads cover in one go
    static_assert(256 % PIECES == 0 && PIECES % 64 == 0 && SK_SEQS % ROWS_AT_ONCE == 0, "staging layout");
    const int pc = tid % PIECES;
    const int brow = __builtin_amdgcn_readfirstlane(tid / PIECES);  // the same for a whole wave
    const bool piece_ok = 4 * pc < klen;
    const long piece = piece_ok ? (long)kbeg + 4 * pc : 0;
    float4 xv16[SK_SEQS / ROWS_AT_ONCE];
#pragma unroll
    for (int i = 0; i < SK_SEQS / ROWS_AT_ONCE; ++i) {
        // sequences past B read the row of sequence 0 (lane b of my_row holds 0 for them)
        const long xrow = __builtin_amdgcn_readlane(my_row, brow + ROWS_AT_ONCE * i);
        xv16[i] = *(const float4 *)(x + xrow * (long)d + piece);
    }
#pragma unroll
    for (int i = 0; i < SK_SEQS / ROWS_AT_ONCE; ++i) {
        const int b = brow + ROWS_AT_ONCE * i;
        const bool ok = piece_ok && b < B;
        float4 v = xv16[i];
        v.x = ok ? v.x : 0.f, v.y = ok ? v.y : 0.f, v.z = ok ? v.z : 0.f, v.w = ok ? v.w : 0.f;
        *(float4 *)&xs[b][4 * pc] = v;
    }
    __syncthreads();

    float acc[64];  // acc[16 * r + b]
#pragma unroll
    for (int i = 0; i < 64; ++i)
        acc[i] = 0.f;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int k = 4 * lane + 256 * p;  // past klen: the staged vectors are zero
#pragma unroll
        for (int b = 0; b < SK_SEQS; ++b) {
            const float4 xv = *(const float4 *)&xs[b][k];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float a = acc[16 * r + b];
                a = fmaf(wv[p][r].x, xv.x, a);
                a = fmaf(wv[p][r].y, xv.y, a);
                a = fmaf(wv[p][r].z, xv.z, a);
                a = fmaf(wv[p][r].w, xv.w, a);
                acc[16 * r + b] = a;
            }
        }
    }
    // halving butterfly over the lanes: after a step with bit o a lane holds n / 2 sums, the upper half
    // of the indices if its bit o is set
    halve_over_lanes(acc);
    const int b = lane & 15, j = j0 + (lane >> 4);
    if (b < B && j < d_h)
        act_part[((long)blockIdx.y * B + b) * d_h + j] = acc[0];
}

// Layer 1, fp32 weights, 17 to F32_MAX_SEQS sequences: fp32 matrix instructions (16x16x4, fp32 operands and accumulators: the
// precision of an FMA chain).  Bound: latency of the few chunks that a slice has.
// Workgroup = 4 waves (2 x 2), FJ = 128 head rows x 32 NS sequences; wave = 64 x 16 NS = 4 x NS tiles, weights as the
// row operand.  K is staged 16 elements at a time as 64-byte rows, 16-byte chunks XOR-ed with swizzle key (r >> 1) & 3:
// lane l reads chunk l / 16 of row l % 16, i.e. four neighbouring K elements that feed four MFMAs (an MFMA then
// contracts elements s, 4 + s, 8 + s, 12 + s of the sixteen: the order inside a sum, the same for both operands).  The
// next chunk's global loads are in flight during the current one's MFMAs; two LDS buffers.
// (On bf16 pieces, below, whose pipeline takes longer to fill: whole training steps with 32 and 64 samples 38.3 -> 41.0 us and
// 45.8 -> 47.0; 71 samples, d = 4040 52.6 -> 51.1.)
constexpr int FJ = 128, FK = 16;
constexpr int F32_WORKGROUPS = 512;  // workgroups asked for by splitting along d
constexpr int F32_MAX_SEQS = 64;

template <int NS>
__global__ __launch_bounds__(256) void head_layer1_f32_kernel(const float *__restrict__ x,
                                                              const int32_t *__restrict__ slot, int B, int d, int d_h,
                                                              const float *__restrict__ w1, int kchunk, int nks,
                                                              int jtiles, float *__restrict__ act_part)
{
    constexpr int FS = 32 * NS;
    constexpr int W_PIECES = FJ / 64, X_PIECES = (FS + 63) / 64;  // 16-byte pieces a thread stages per chunk
    __shared__ __align__(16) unsigned char lds[2][(FJ + X_PIECES * 64) * 64];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int l15 = lane & 15, kq = lane >> 4;
    // the slice index varies fastest over the grid: an XCD pulls only its own slices of both operands
    const int kslice = blockIdx.x % nks;
    const int tile = blockIdx.x / nks;
    const int j0 = (tile % jtiles) * FJ, s0 = (tile / jtiles) * FS;
    const int wj = (wave & 1) * 64, ws = (wave >> 1) * (16 * NS);

    const int prow = tid >> 2, pchunk = tid & 3;  // what this thread stages: rows prow + 64 p, this chunk
    const unsigned pdst = (unsigned)(prow * 64 + ((pchunk ^ ((prow >> 1) & 3)) << 4));
    const float *wp[W_PIECES], *xp[X_PIECES];
#pragma unroll
    for (int p = 0; p < W_PIECES; ++p) {
        const int j = min(j0 + prow + 64 * p, d_h - 1);  // clamped rows are computed and dropped
        wp[p] = w1 + (long)j * d + 4 * pchunk;
    }
#pragma unroll
    for (int p = 0; p < X_PIECES; ++p) {
        const int sq = min(s0 + prow + 64 * p, B - 1);
        xp[p] = x + (long)(slot ? slot[sq] : sq) * d + 4 * pchunk;
    }
    const int kbeg = kslice * kchunk;
    const int kend = min(d, kbeg + kchunk);
    float4 wr[W_PIECES], xr[X_PIECES];
    auto fetch = [&](int k0) {  // kend is a multiple of 4: a piece is inside the slice or outside of it
        const bool ok = k0 + 4 * pchunk < kend;
#pragma unroll
        for (int p = 0; p < W_PIECES; ++p)
            wr[p] = ok ? *(const float4 *)(wp[p] + k0) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int p = 0; p < X_PIECES; ++p)
            xr[p] = ok ? *(const float4 *)(xp[p] + k0) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    auto stage = [&](unsigned char *buf) {
#pragma unroll
        for (int p = 0; p < W_PIECES; ++p)
            *(float4 *)(buf + p * 4096 + pdst) = wr[p];
#pragma unroll
        for (int p = 0; p < X_PIECES; ++p)
            *(float4 *)(buf + FJ * 64 + p * 4096 + pdst) = xr[p];
    };

    f32x4 acc[4][NS];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < NS; ++b)
            acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const unsigned rd = (unsigned)(l15 * 64 + ((kq ^ ((l15 >> 1) & 3)) << 4));
    if (kbeg < kend) {
        fetch(kbeg);
        stage(lds[0]);
    }
    __syncthreads();
    int cur = 0;
    for (int k0 = kbeg; k0 < kend; k0 += FK) {
        const bool more = k0 + FK < kend;
        if (more)
            fetch(k0 + FK);
        const unsigned char *buf = lds[cur];
        f32x4 fa[4], fb[NS];
#pragma unroll
        for (int a = 0; a < 4; ++a)
            fa[a] = *(const f32x4 *)(buf + (wj + 16 * a) * 64 + rd);
#pragma unroll
        for (int b = 0; b < NS; ++b)
            fb[b] = *(const f32x4 *)(buf + (FJ + ws + 16 * b) * 64 + rd);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < NS; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[a][s], fb[b][s], acc[a][b], 0, 0, 0);
        if (more)
            stage(lds[cur ^ 1]);  // nobody reads that buffer now
        __syncthreads();
        cur ^= 1;
    }

    float *act = act_part + (long)kslice * B * d_h;
#pragma unroll
    for (int b = 0; b < NS; ++b) {
        const int s = s0 + ws + 16 * b + l15;
        if (s >= B)
            continue;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const int jj = j0 + wj + 16 * a + 4 * kq;
            if (jj + 3 < d_h && (d_h & 3) == 0) {
                *(f32x4 *)(act + (long)s * d_h + jj) = acc[a][b];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (jj + i < d_h)
                        act[(long)s * d_h + jj + i] = acc[a][b][i];
            }
        }
    }
}

// Layer 1, fp32 weights, more sequences: fp32 products as bf16 pieces (split_mfma.h), weights as the rows of the tile,
// sequences as its columns.  Bound: six bf16 MFMAs per 32 K elements, 34 us at the rate that the matrix cores hold for
// 1024 sequences, d = 4096, d_h = 1024, beside the splitting of both operands (208 vector instructions to 96 MFMAs).  That
// batch took 86 to 90 us on the fp32 matrix instructions (95 to 100 TFLOP/s), now 50 to 54; the error against fp64
// is 0.7 of what it was (fewer roundings: one per MFMA, of 32 products).  Tried: both operands split once per workgroup
// and read from the LDS, 8 waves 55 us and 4 waves 60 against 52 in the same run; without a pinned order of instructions 65.
// Columns of 64 instead of 128 fill the chip with two workgroups per compute unit (59 us) and hold the pipeline's start
// down: taken where a slice has fewer than SPLIT_WIDE_STEPS steps (1024 sequences, d = 1024, d_h = 300: training step
// 69.7 -> 64.1 us; 309, d = 2208, d_h = 700: 66.2 -> 62.8).
constexpr int SPLIT_WIDE_STEPS = 8;

template <class S>
struct Layer1Source {
    static constexpr int ROW_LOADS = 2 * S::FA, COL_LOADS = 2 * S::SHARE;
    static constexpr bool COLS_MAY_BE_INF = true;
    struct Rows {
        float4 v[S::FA][2];
    };
    struct Cols {
        float4 v[S::SHARE][2];
    };
    const float *w[S::FA], *x[S::SHARE];  // + 8 (lane / 16)
    int kbeg, kend, kq, wave, lane;

    // Past the end of the slice its last four elements are loaded again (no branch around a load: the loads in flight stay
    // countable) and counted as zeros; kend is a multiple of 4, so four elements are inside the slice or outside.
    __device__ __forceinline__ float4 four(const float *p, int i, int h) const
    {
        return *(const float4 *)(p + min(kbeg + i * S::STEP + 4 * h, kend - 4 - 8 * kq));
    }
    __device__ __forceinline__ void load_rows(int i, int l, Rows &r) const { r.v[l / 2][l % 2] = four(w[l / 2], i, l % 2); }
    __device__ __forceinline__ void load_cols(int i, int l, Cols &r) const { r.v[l / 2][l % 2] = four(x[l / 2], i, l % 2); }
    template <int N>
    __device__ __forceinline__ void clear(int i, float4 (&v)[N][2]) const
    {
        const int k0 = kbeg + i * S::STEP;
        if (k0 + S::STEP <= kend)
            return;
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (k0 + 8 * kq + 4 * h >= kend)
                    v[n][h] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __device__ __forceinline__ void clear_rows(int i, Rows &r) const { clear(i, r.v); }
    __device__ __forceinline__ void clear_cols(int i, Cols &r) const { clear(i, r.v); }
    __device__ __forceinline__ float row_value(const Rows &r, int a, int e) const { return (&r.v[a][e / 4].x)[e % 4]; }
    __device__ __forceinline__ float col_value(const Cols &r, int p, int e) const { return (&r.v[p][e / 4].x)[e % 4]; }
    __device__ __forceinline__ int place(int p) const { return ((wave + S::WAVES * p) * 64 + lane) * 16; }
};

template <class S>
__global__ __launch_bounds__(S::THREADS, S::FB == 4 ? 2 : 1) void head_layer1_split_kernel(
    const float *__restrict__ x, const int32_t *__restrict__ slot, int B, int d, int d_h, const float *__restrict__ w1,
    int kchunk, int nks, int jtiles, float *__restrict__ act_part)
{
    static_assert(S::ROWS == FJ, "tile");
    constexpr int FA = S::FA, FB = S::FB;
    __shared__ __align__(16) unsigned char lds[S::LDS_BYTES];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, kq = lane >> 4;
    // the slice index varies fastest over the grid: an XCD pulls only its own slices of both operands
    const int kslice = blockIdx.x % nks;
    const int tile = blockIdx.x / nks;
    const int j0 = (tile % jtiles) * S::ROWS, s0 = (tile / jtiles) * S::COLS;

    Layer1Source<S> src;
    src.kbeg = kslice * kchunk;
    src.kend = min(d, src.kbeg + kchunk);
    src.kq = kq, src.wave = wave, src.lane = lane;
#pragma unroll
    for (int a = 0; a < FA; ++a) {
        const int j = min(j0 + 16 * (wave * FA + a) + l15, d_h - 1);  // clamped rows are computed and dropped
        src.w[a] = w1 + (long)j * d + 8 * kq;
    }
#pragma unroll
    for (int p = 0; p < S::SHARE; ++p) {
        const int sq = min(s0 + 16 * (wave + S::WAVES * p) + l15, B - 1);
        src.x[p] = x + (long)(slot ? slot[sq] : sq) * d + 8 * kq;
    }
    split_f32x4 acc[FA][FB];
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int b = 0; b < FB; ++b)
            acc[a][b] = split_f32x4{0.f, 0.f, 0.f, 0.f};
    if (src.kbeg < src.kend)
        split_contract<S>(lds, (src.kend - src.kbeg + S::STEP - 1) / S::STEP, lane, acc, src);

    float *act = act_part + (long)kslice * B * d_h;
#pragma unroll
    for (int b = 0; b < FB; ++b) {
        const int s = s0 + 16 * b + l15;
        if (s >= B)
            continue;
#pragma unroll
        for (int a = 0; a < FA; ++a) {
            const int jj = j0 + 16 * (wave * FA + a) + 4 * kq;
            if (jj + 3 < d_h && (d_h & 3) == 0) {
                *(split_f32x4 *)(act + (long)s * d_h + jj) = acc[a][b];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (jj + i < d_h)
                        act[(long)s * d_h + jj + i] = acc[a][b][i];
            }
        }
    }
}

constexpr int MK = 32;  // K elements per MFMA step

// Layer 1 on the matrix cores, bf16 weights, d % 8 == 0.  Workgroup = 4 waves, MJ = 128 head rows x
// TN = 64 sequences; wave = 64 x 32 = 4 x 2 MFMA 16x16x32 tiles, weights as the row operand (lane l:
// head row l % 16, K elements 8 * (l / 16) .. + 8), pooled vectors as the column operand; in the
// accumulator a lane holds head rows 4 * (l / 16) + i of sequence l % 16.  Per K step every thread
// fetches 8 K-elements of one pooled row (32 bytes) and of two weight rows (16 bytes each), splits
// the fp32 values once, and leaves all of it in LDS in fragment order -- fragment f, lane l at
// (f * 64 + l) * 16 bytes -- so that a fragment read is one linear 16-byte read per lane.  Two
// LDS buffers; global fetches run three steps ahead in registers.
constexpr int MJ = 128;
constexpr int MFMA_W_FRAGS = MJ / 16;             // 8 weight fragments per step
constexpr int MFMA_X_FRAGS = 3 * (TN / 16);       // 3 parts x 4 sequence fragments
constexpr int MFMA_STAGE_BYTES = (MFMA_W_FRAGS + MFMA_X_FRAGS) * 1024;

__global__ __launch_bounds__(256) void head_layer1_mfma_kernel(const float *__restrict__ x,
                                                               const int32_t *__restrict__ slot, int B, int d,
                                                               int d_h, const unsigned short *__restrict__ w1,
                                                               int kchunk, int nks, int jtiles,
                                                               float *__restrict__ act_part)
{
    __shared__ __align__(16) unsigned char lds[2 * MFMA_STAGE_BYTES];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int l15 = lane & 15, kq = lane >> 4;
    // Workgroup i runs on XCD i % 8: the slice along d varies fastest, so that an XCD's L2 only
    // ever pulls its own slices of the weights and of the pooled vectors over the fabric.
    const int kslice = blockIdx.x % nks;
    const int tile = blockIdx.x / nks;
    const int j0 = (tile % jtiles) * MJ, s0 = (tile / jtiles) * TN;
    const int wj = (wave & 1) * 4;  // first of this wave's 4 weight fragments
    const int ws = (wave >> 1) * 2; // first of its 2 sequence fragments

    // what this thread stages: row 16 * wave + lane % 16 of the tile (and that row + 64 of the
    // weights), K elements 8 * (lane / 16) .. + 8 -- which is lane `lane` of fragment `wave`, so a
    // wave's 16-byte LDS writes are one linear KiB
    const int srow_l = wave * 16 + l15, kpart = kq;
    int srow = s0 + srow_l;
    srow = srow < B ? srow : B - 1;  // clamped rows are computed and dropped
    const long xrow = slot ? slot[srow] : srow;
    const float *xp = x + xrow * (long)d + 8 * kpart;
    const unsigned short *wp[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        int jrow = j0 + 64 * r + srow_l;
        jrow = jrow < d_h ? jrow : d_h - 1;
        wp[r] = w1 + (long)jrow * d + 8 * kpart;
    }
    const unsigned stage_lane = (unsigned)(lane * 16);
    const unsigned w_dst0 = (unsigned)(wave * 1024) + stage_lane;                   // rows 0..63
    const unsigned w_dst1 = (unsigned)((4 + wave) * 1024) + stage_lane;             // rows 64..127
    const unsigned x_dst = (unsigned)((MFMA_W_FRAGS + wave) * 1024) + stage_lane;   // part p: + p * 4096

    f32x4 acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
            acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int kbeg = kslice * kchunk;
    const int kend = min(d, kbeg + kchunk);
    // kend and 8 * kpart are multiples of 8: a thread's 8 elements are inside [kbeg, kend) or all outside
    struct Fetched {
        u32x4 w[2];
        float4 x[2];
    };
    auto fetch = [&](int k0, Fetched &r) {
        r.w[0] = r.w[1] = u32x4{0u, 0u, 0u, 0u};
        r.x[0] = r.x[1] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k0 + 8 * kpart < kend) {
            r.w[0] = *(const u32x4 *)(wp[0] + k0);
            r.w[1] = *(const u32x4 *)(wp[1] + k0);
            r.x[0] = *(const float4 *)(xp + k0);
            r.x[1] = *(const float4 *)(xp + k0 + 4);
        }
    };
    auto stage = [&](const Fetched &r, unsigned char *buf) {
        const float f[8] = {r.x[0].x, r.x[0].y, r.x[0].z, r.x[0].w, r.x[1].x, r.x[1].y, r.x[1].z, r.x[1].w};
        bf16x8 hi, mid, lo;
        split3(f, hi, mid, lo);
        *(u32x4 *)(buf + w_dst0) = r.w[0];
        *(u32x4 *)(buf + w_dst1) = r.w[1];
        *(bf16x8 *)(buf + x_dst) = hi;
        *(bf16x8 *)(buf + x_dst + 4096) = mid;
        *(bf16x8 *)(buf + x_dst + 8192) = lo;
    };

    // Operands are fetched three steps ahead into a ring of three register sets (the loop is
    // unrolled by three so that the ring is indexed statically) and staged one step ahead.
    Fetched ring[3];
    fetch(kbeg, ring[0]);
    fetch(kbeg + MK, ring[1]);
    fetch(kbeg + 2 * MK, ring[2]);
    stage(ring[0], lds);
    __syncthreads();
    int cur = 0;
    for (int base = kbeg; base < kend; base += 3 * MK) {
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int k0 = base + u * MK;
            if (k0 >= kend)
                break;
            fetch(k0 + 3 * MK, ring[u]);  // ring[u] held step k0, which is in LDS already
            const unsigned char *buf = lds + cur * MFMA_STAGE_BYTES;
            bf16x8 wf[4], xf[3][2];
#pragma unroll
            for (int a = 0; a < 4; ++a)
                wf[a] = *(const bf16x8 *)(buf + ((wj + a) * 64 + lane) * 16);
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    xf[p][b] = *(const bf16x8 *)(buf + ((MFMA_W_FRAGS + 4 * p + ws + b) * 64 + lane) * 16);
#pragma unroll
            for (int p = 2; p >= 0; --p)  // smallest parts first
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[a], xf[p][b], acc[a][b], 0, 0, 0);
            if (k0 + MK < kend)
                stage(ring[(u + 1) % 3], lds + (cur ^ 1) * MFMA_STAGE_BYTES);  // nobody reads that buffer now
            __syncthreads();
            cur ^= 1;
        }
    }

    float *act = act_part + (long)kslice * B * d_h;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int s = s0 + 16 * (ws + b) + l15;
        if (s >= B)
            continue;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const int jj = j0 + 16 * (wj + a) + 4 * kq;
            if (jj + 3 < d_h && (d_h & 3) == 0) {
                *(f32x4 *)(act + (long)s * d_h + jj) = acc[a][b];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (jj + i < d_h)
                        act[(long)s * d_h + jj + i] = acc[a][b][i];
            }
        }
    }
}

// Layer 2 of a scalar head: pred = b2 + w2 . act[b,:].  NS sequences per workgroup (head_tail.h); TINY: d_h < 4.
// LDS: a[NS][lda] | part[NS][TAIL_WAVES]
template <bool WBF16, bool TINY, int NS>
__global__ __launch_bounds__(TAIL_THREADS) void head_scalar_kernel(const float *__restrict__ act_part, int nks, int B,
                                                                   const float *__restrict__ b1, int d_h,
                                                                   const void *__restrict__ w2_any,
                                                                   const float *__restrict__ b2, float *__restrict__ pred)
{
    using W = std::conditional_t<WBF16, unsigned short, float>;
    const W *w2 = (const W *)w2_any;
    __shared__ float4 join[NS < 4 ? TAIL_JOIN_FLOATS / 4 : 1];
    extern __shared__ __align__(16) float a[];
    const int b0 = blockIdx.x * NS, lda = tail_row(d_h);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *part = a + NS * lda;
    // thread t takes the chunks t, t + TAIL_THREADS, ... of the dot product (fixed assignment: bit-reproducible)
    const float bias = b2 ? b2[0] : 0.f;
    ChunkOf<W> w = load_chunk(w2, RowChunk<TINY>(tid, d_h), d_h);
    hidden_units<TINY, NS>(act_part, nks, B, b0, d_h, b1, a, lda, join, nullptr);
    float s[NS] = {};
    for (int c0 = tid; 4 * c0 < lda; c0 += TAIL_THREADS) {
        const RowChunk<TINY> c(c0, d_h);
        if (c0 != tid)
            w = load_chunk(w2, c, d_h);
#pragma unroll
        for (int n = 0; n < NS; ++n)
            s[n] = chunk_dot(w, c, *(const float4 *)(a + n * lda + 4 * c0), s[n]);
    }
#pragma unroll
    for (int n = 0; n < NS; ++n) {
        const float t = wave_sum(s[n]);
        if (lane == 0)
            part[n * TAIL_WAVES + wave] = t;
    }
    __syncthreads();
    if (tid < NS && b0 + tid < B) {
        float t = part[tid * TAIL_WAVES];
#pragma unroll
        for (int q = 1; q < TAIL_WAVES; ++q)
            t += part[tid * TAIL_WAVES + q];
        pred[b0 + tid] = t + bias;
    }
}

// Layer 2 of a K-bin head: out[o] = b2[o] + w2[o,:] . act[b,:], then Eq. 6.  LDS: a[NS][lda] | z[NS][n_out]
template <bool WBF16, bool TINY, int NS>
__global__ __launch_bounds__(TAIL_THREADS) void head_bins_kernel(const float *__restrict__ act_part, int nks, int B,
                                                                 const float *__restrict__ b1, int d_h, int n_out,
                                                                 const void *__restrict__ w2,
                                                                 const float *__restrict__ b2,
                                                                 const float *__restrict__ centers,
                                                                 float *__restrict__ pred, float *__restrict__ p_hat)
{
    using W = std::conditional_t<WBF16, unsigned short, float>;
    __shared__ float4 join[NS < 4 ? TAIL_JOIN_FLOATS / 4 : 1];
    extern __shared__ __align__(16) float a[];
    const int b0 = blockIdx.x * NS, lda = tail_row(d_h);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *z = a + NS * lda;
    // bin o < 64 belongs to lane o: its bias and centre are asked for now
    const int o_near = min(lane, n_out - 1);
    const float b2_near = b2 ? b2[o_near] : 0.f, center_near = centers[o_near];
    output_layer<TINY, NS>((const W *)w2, n_out, d_h, a, lda, z,
                           [&] { hidden_units<TINY, NS>(act_part, nks, B, b0, d_h, b1, a, lda, join, nullptr); });
    __syncthreads();
    const int b = b0 + wave;
    if (wave >= NS || b >= B)
        return;
    z += wave * n_out;
    // Eq. 6: softmax over the bins (bin o by lane o % 64) and its expectation
    float m = -__builtin_inff(), den = 0.f, num = 0.f;
    for (int o = lane; o < n_out; o += 64) {
        const float v = z[o] + (o < 64 ? b2_near : (b2 ? b2[o] : 0.f));
        z[o] = v;
        m = fmaxf(m, v);
    }
    m = wave_max(m);
    for (int o = lane; o < n_out; o += 64) {
        const float e = __expf(z[o] - m);
        den += e;
        num = fmaf(e, o < 64 ? center_near : centers[o], num);
    }
    den = wave_sum(den);
    num = wave_sum(num);
    if (lane == 0)
        pred[b] = num / den;
    if (p_hat != nullptr) {  // the distribution itself, when the caller wants it
        const float inv = 1.0f / den;
        for (int o = lane; o < n_out; o += 64)
            p_hat[(long)b * n_out + o] = __expf(z[o] - m) * inv;
    }
}

}  // namespace

// slices of the skinny kernel: as few as keep a slice within its LDS buffer
static int skinny_slices(int d) { return (d + SK_SLICE - 1) / SK_SLICE; }
static bool skinny_serves(int d, int32_t B, int wdtype)
{
    return wdtype == DT_F32 && B <= SK_SEQS && d % 4 == 0 && skinny_slices(d) <= 64;
}

// Sequences per tile of the fp32 matrix kernel.  (128 x 128 tiles gain nothing for their halved operand traffic: whole
// training steps at batch 1024 199.7 us against 199.4, at d = 1024, d_h = 300, batch 256 39.1 against 34.6.)
static int f32_tile_seqs(int32_t B) { return B > 32 ? 64 : 32; }

int head_k_splits(int d, int d_h, int32_t B, int wdtype)
{
    if (skinny_serves(d, B, wdtype))
        return skinny_slices(d);
    int base = (d + 511) / 512;  // slices of at most 512 along d ...
    base = base < 1 ? 1 : (base > 8 ? 8 : base);
    const long tiles = (long)((d_h + TM - 1) / TM) * ((B + TN - 1) / TN);
    long want = tiles > 0 ? (1024 + tiles - 1) / tiles : 1;  // ... thinner when the batch has few tiles
    const int cap = (d + TK - 1) / TK < 64 ? (d + TK - 1) / TK : 64;
    long n = want > base ? want : base;
    n = n > cap ? cap : n;
    if (wdtype == DT_F32) {  // larger tiles: fewer slices
        const long ftiles = (long)((d_h + FJ - 1) / FJ) * ((B + f32_tile_seqs(B) - 1) / f32_tile_seqs(B));
        const long fwant = ftiles > 0 ? (F32_WORKGROUPS + ftiles - 1) / ftiles : 1;
        n = n > fwant ? fwant : n;
        // a slice of at least two K steps of the kernel on bf16 pieces
        if (B > F32_MAX_SEQS && n > (d + 63) / 64)
            n = (d + 63) / 64;
    }
    return n < 1 ? 1 : (int)n;
}

size_t head_act_floats_bound(int d, int d_h, int32_t B, int wdtype)
{
    // the number of planes only depends on how many 64-sequence tiles the batch has -- and, for fp32 weights,
    // on whether the batch is small enough for the skinny kernel
    size_t best = 0;
    for (int32_t st = 1; st <= (B + TN - 1) / TN; ++st) {
        const int32_t b = st * TN < B ? st * TN : B;
        const size_t f = (size_t)head_k_splits(d, d_h, b, wdtype) * (size_t)b * (size_t)d_h;
        best = f > best ? f : best;
    }
    const int32_t bs = B < SK_SEQS ? B : SK_SEQS;
    const size_t fs = (size_t)head_k_splits(d, d_h, bs, wdtype) * (size_t)bs * (size_t)d_h;
    return fs > best ? fs : best;
}

hipError_t head_layer1(const float *x, const int32_t *slot, int32_t B, int d, int d_h, const void *w1,
                       int wdtype, float *act_part, hipStream_t st)
{
    if (B <= 0)
        return hipSuccess;
    const int nks = head_k_splits(d, d_h, B, wdtype);
    if (skinny_serves(d, B, wdtype)) {
        // whole 256-element passes; nks = ceil(d / SK_SLICE) keeps a slice within the LDS buffer and leaves no
        // slice empty (a slice past the end of d would still write its plane: zeros)
        const int kchunk_s = ((d + nks - 1) / nks + 255) / 256 * 256;
        if (kchunk_s > SK_SLICE)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(head_layer1_skinny_kernel, dim3((d_h + SK_ROWS - 1) / SK_ROWS, nks), dim3(256), 0, st, x, slot,
                           B, d, d_h, (const float *)w1, kchunk_s, act_part);
        return hipGetLastError();
    }
    if (wdtype == DT_F32) {
        const bool small = B <= F32_MAX_SEQS;
        const int kstep = small ? FK : SplitTile<2, 4>::STEP;
        const int kchunk_f = ((d + nks - 1) / nks + kstep - 1) / kstep * kstep;
        const bool wide = !small && kchunk_f >= SPLIT_WIDE_STEPS * kstep;
        const int jtiles = (d_h + FJ - 1) / FJ, fs = small ? f32_tile_seqs(B) : (wide ? 128 : 64);
        const long wgs = (long)jtiles * ((B + fs - 1) / fs) * nks;
        if (d % 4 != 0 || wgs > 0x7fffffffL)
            return hipErrorInvalidValue;
#define EGTP_LAYER1_F32(KERNEL)                                                                                   \
    hipLaunchKernelGGL(KERNEL, dim3((unsigned)wgs), dim3(256), 0, st, x, slot, B, d, d_h, (const float *)w1, kchunk_f, \
                       nks, jtiles, act_part)
        if (wide)
            EGTP_LAYER1_F32((head_layer1_split_kernel<SplitTile<2, 8>>));
        else if (!small)
            EGTP_LAYER1_F32((head_layer1_split_kernel<SplitTile<2, 4>>));
        else if (fs == 64)
            EGTP_LAYER1_F32(head_layer1_f32_kernel<2>);
        else
            EGTP_LAYER1_F32(head_layer1_f32_kernel<1>);
#undef EGTP_LAYER1_F32
        return hipGetLastError();
    }
    if (wdtype == DT_BF16 && d % 8 == 0) {
        // matrix-core path: slices are multiples of the MFMA K step (late slices may be empty
        // and then write zeros)
        const int kchunk_m = ((d + nks - 1) / nks + MK - 1) / MK * MK;
        const int jtiles = (d_h + MJ - 1) / MJ;
        const long wgs = (long)jtiles * ((B + TN - 1) / TN) * nks;
        if (wgs > 0x7fffffffL)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(head_layer1_mfma_kernel, dim3((unsigned)wgs), dim3(256), 0, st, x, slot, B, d, d_h,
                           (const unsigned short *)w1, kchunk_m, nks, jtiles, act_part);
        return hipGetLastError();
    }
    const int kchunk = ((d + nks - 1) / nks + TK - 1) / TK * TK;  // multiple of the K step
    hipLaunchKernelGGL(head_layer1_kernel, dim3((d_h + TM - 1) / TM, (B + TN - 1) / TN, nks), dim3(256), 0, st, x, slot, B,
                       d, d_h, (const unsigned short *)w1, kchunk, act_part);
    return hipGetLastError();
}

template <bool WBF16, bool TINY, int NS>
static hipError_t launch_layer2(const HeadArgs &a, int nks, size_t lds, hipStream_t st)
{
    static DeviceMask raised_scalar{0}, raised_bins{0};
    const dim3 grid((a.B - 1) / NS + 1), block(TAIL_THREADS);
    hipError_t e;
    if (a.n_out == 1) {
        e = raise_dynamic_lds_limit((const void *)head_scalar_kernel<WBF16, TINY, NS>, (int)TAIL_LDS_LIMIT, raised_scalar);
        if (e == hipSuccess)
            hipLaunchKernelGGL((head_scalar_kernel<WBF16, TINY, NS>), grid, block, NS * lds, st, a.act, nks, a.B, a.b1, a.d_h,
                               a.w2, a.b2, a.pred);
    } else {
        e = raise_dynamic_lds_limit((const void *)head_bins_kernel<WBF16, TINY, NS>, (int)TAIL_LDS_LIMIT, raised_bins);
        if (e == hipSuccess)
            hipLaunchKernelGGL((head_bins_kernel<WBF16, TINY, NS>), grid, block, NS * lds, st, a.act, nks, a.B, a.b1, a.d_h,
                               a.n_out, a.w2, a.b2, a.bin_centers, a.pred, a.p_hat);
    }
    return e == hipSuccess ? hipGetLastError() : e;
}

template <bool WBF16>
static hipError_t launch_layer2(const HeadArgs &a, int nks, size_t lds, hipStream_t st)
{
    if (a.d_h < 4)
        return launch_layer2<WBF16, true, 1>(a, nks, lds, st);
    const int ns = tail_sequences(a.B, lds);
    return ns == 4 ? launch_layer2<WBF16, false, 4>(a, nks, lds, st)
           : ns == 2 ? launch_layer2<WBF16, false, 2>(a, nks, lds, st) : launch_layer2<WBF16, false, 1>(a, nks, lds, st);
}

hipError_t head_forward(const HeadArgs &a, hipStream_t st)
{
    if (a.B <= 0)
        return hipSuccess;
    const int nks = head_k_splits(a.d, a.d_h, a.B, a.wdtype);
    const size_t lds = ((size_t)tail_row(a.d_h) + (size_t)(a.n_out > TAIL_WAVES ? a.n_out : TAIL_WAVES)) * sizeof(float);
    if (lds > TAIL_LDS_LIMIT)
        return hipErrorInvalidValue;
    hipError_t e = head_layer1(a.x, a.slot, a.B, a.d, a.d_h, a.w1, a.wdtype, a.act, st);
    if (e != hipSuccess)
        return e;
    return a.wdtype == DT_BF16 ? launch_layer2<true>(a, nks, lds, st) : launch_layer2<false>(a, nks, lds, st);
}

}  // namespace egtp
