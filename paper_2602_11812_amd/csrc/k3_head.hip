// Prediction head (Section 3.2): pooled vector -> perceptron d -> d_h (ReLU) -> n_out, then
// either the scalar itself (n_out == 1) or the expected value over K bins of Eq. 6.
//
// Layer 1 is a small [B x d] . [d x d_h] contraction kept entirely in fp32 (the pooled
// vector is never re-rounded), on the fp32 matrix instructions where the weights are fp32 and the batch is more
// than a handful, and as products of bf16 pieces where it is more than 64 and the contraction not small.  It is split
// along d so that several hundred workgroups exist even for one small batch; the splits leave partial pre-activations that
// layer 2 adds in a fixed order (bit-reproducible) before bias and ReLU.  Layer 2 and the K-bin decode: head_tail.h.
//
// With bf16 weights and d a multiple of 8, layer 1 runs on the bf16 matrix cores without rounding the pooled vector: an
// fp32 value is the exact sum of three bf16 values, a bf16 x bf16 product is exact in fp32, so three MFMAs per weight fragment
// accumulate the same products an fp32 dot product would, in fp32 (split_mfma.h).
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

// Layer 1, fp32 weights, 17 to F32_MAX_SEQS sequences and small contractions of more (f32_serves): fp32 matrix instructions (16x16x4, fp32 operands and accumulators: the
// precision of an FMA chain).  Bound: latency of the few chunks that a slice has.
// Workgroup = 4 waves (2 x 2), FJ = 128 head rows x 32 NS sequences; wave = 64 x 16 NS = 4 x NS tiles, weights as the
// row operand.  K is staged 16 elements at a time as 64-byte rows, 16-byte chunks XOR-ed with swizzle key (r >> 1) & 3:
// lane l reads chunk l / 16 of row l % 16, i.e. four neighbouring K elements that feed four MFMAs (an MFMA then
// contracts elements s, 4 + s, 8 + s, 12 + s of the sixteen: the order inside a sum, the same for both operands).  The
// next chunk's global loads are in flight during the current one's MFMAs; two LDS buffers.
// (On bf16 pieces, below, whose pipeline takes longer to fill: whole training steps with 32 and 64 samples, d = 4096, d_h = 1024 38.3 ->
// 41.0 us and 45.8 -> 47.0; 71 samples, d = 4040 52.6 -> 51.1.)
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

// Layer 1, bf16 weights (d % 8 == 0) or fp32 weights and more sequences: products of bf16 pieces (split_mfma.h), weights as the rows,
// sequences as the columns of the tile.  Bound (fp32): six bf16 MFMAs per 32 K elements, 34 us at the rate that the matrix cores hold for
// 1024 sequences, d = 4096, d_h = 1024, beside the splitting of both operands (208 vector instructions to 96 MFMAs).  That
// batch took 86 to 90 us on the fp32 matrix instructions (95 to 100 TFLOP/s), now 50 to 54; the error against fp64
// is 0.7 of what it was (fewer roundings: one per MFMA, of 32 products).  Tried: both operands split once per workgroup
// and read from the LDS, 8 waves 55 us and 4 waves 60 against 52 in the same run; without a pinned order of instructions 65.
// Columns of 64 instead of 128 fill the chip with two workgroups per compute unit (59 us) and hold the pipeline's start
// down: taken where a slice has fewer than SPLIT_WIDE_STEPS steps (1024 sequences, d = 1024, d_h = 300: training step
// 69.7 -> 64.1 us; 309, d = 2208, d_h = 700: 66.2 -> 62.8).
// Loads: in fragment order the lanes of a quad ask for four different rows, four lines each time, and the address unit takes
// them one by one.  Here a quad loads one line of a row and the operands turn on their way through the LDS: the columns,
// which pass through it anyway, and in tiles of 64 columns the rows (bf16, 1017 sequences, d = 4096, d_h = 1024 44.6 ->
// 36.4 us, d = 5120, d_h = 1280 63 -> 50; fp32, 512, d = 2048 20.5 -> 18; in tiles of 128 the LDS is the tighter bound:
// 50 -> 52).  The kernel of their own that served bf16 weights before staged both operands, two waves a row of tiles: 512
// sequences, d = 4096, d_h = 1024 27.3 -> 22.9 us, 128 16.9 -> 12.4, 24 9.0 -> 7.5; tiles of 128 columns are slower there
// (12 -> 16 us for 128 sequences, 32 -> 44 for 512 at d = 5120).
constexpr int SPLIT_WIDE_STEPS = 8;
typedef SplitTile<2, 8> WideTile;
typedef SplitTile<2, 4> NarrowTile;

template <class S, typename W>
struct Layer1Source {
    static constexpr bool BF16 = sizeof(W) == 2;
    static constexpr int ROW_PIECES = BF16 ? 1 : 3, ROW_LOADS = BF16 ? S::FA : 2 * S::FA, COL_LOADS = 2 * S::SHARE,
                         COL_WRITES = 3 * S::SHARE;
    static constexpr bool ROWS_READY = false, ROWS_TURN = S::FB == 4;
    static constexpr int TURN_BYTES = 16 * S::STEP * sizeof(W);  // a fragment of rows as it lies in memory
    struct Rows {
        std::conditional_t<BF16, u32x4, float4> v[S::FA][BF16 ? 1 : 2];
    };
    struct Cols {
        float4 v[S::SHARE][2];
    };
    const W *w[S::FA];
    const float *x[S::SHARE];
    int kbeg, kend, row, chunk, wave, lane;  // this lane loads 8 elements, from 8 chunk on, of row `row` of every fragment ...
    int wchunk;                              // ... (of w: where its rows do not turn, of the row and chunk that it uses)
    unsigned char *turn;                     // FA fragments of the wave's own

    // Past the end of the slice its last elements are loaded again (no branch around a load: the loads in flight stay
    // countable) and counted as zeros; kend is a multiple of 4 (bf16: 8), so the elements of a load are inside the slice or outside.
    __device__ __forceinline__ float4 four(const float *p, int c, int i, int h) const
    {
        return *(const float4 *)(p + min(kbeg + i * S::STEP + 8 * c + 4 * h, kend - 4));
    }
    __device__ __forceinline__ void load_rows(int i, int l, Rows &r) const
    {
        if constexpr (BF16)
            r.v[l][0] = *(const u32x4 *)(w[l] + min(kbeg + i * S::STEP + 8 * wchunk, kend - 8));
        else
            r.v[l / 2][l % 2] = four(w[l / 2], wchunk, i, l % 2);
    }
    __device__ __forceinline__ void load_cols(int i, int l, Cols &r) const { r.v[l / 2][l % 2] = four(x[l / 2], chunk, i, l % 2); }
    template <class V, int N, int H>
    __device__ __forceinline__ void clear(int i, int c, V (&v)[N][H]) const
    {
        const int k0 = kbeg + i * S::STEP;
        if (k0 + S::STEP <= kend)
            return;
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int h = 0; h < H; ++h)
                if (k0 + 8 * c + 4 * h >= kend)
                    v[n][h] = V{};
    }
    __device__ __forceinline__ void clear_rows(int i, Rows &r) const { clear(i, wchunk, r.v); }
    __device__ __forceinline__ void clear_cols(int i, Cols &r) const { clear(i, chunk, r.v); }
    // Places of 16 bytes in the LDS, keyed so that the eight lanes that are served at a time meet eight different ones both
    // ways: a row of 8 (bf16: 4) of them on the way in, a column of rows on the way out.
    __device__ __forceinline__ unsigned char *turn_place(int r, int c, int l) const
    {
        return BF16 ? turn + l * TURN_BYTES + r * 64 + ((c ^ (r >> 1 & 3)) << 4)
                    : turn + l / 2 * TURN_BYTES + r * 128 + ((2 * c + l % 2) ^ (r & 7)) * 16;
    }
    __device__ __forceinline__ void write_row(const Rows &r, int l) const
    {
        *(u32x4 *)turn_place(row, chunk, l) = __builtin_bit_cast(u32x4, BF16 ? r.v[l % S::FA][0] : r.v[l / 2][BF16 ? 0 : l % 2]);
    }
    __device__ __forceinline__ void read_row(Rows &r, int l) const
    {
        auto &v = BF16 ? r.v[l % S::FA][0] : r.v[l / 2][BF16 ? 0 : l % 2];
        v = __builtin_bit_cast(std::remove_reference_t<decltype(v)>, *(const u32x4 *)turn_place(lane & 15, lane >> 4, l));
    }
    __device__ __forceinline__ float row_value(const Rows &r, int a, int e) const { return (&r.v[a][e / 4].x)[e % 4]; }
    __device__ __forceinline__ unsigned row_pair(const Rows &r, int a, int e) const { return r.v[a][0][e]; }
    __device__ __forceinline__ float col_value(const Cols &r, int p, int e) const { return (&r.v[p][e / 4].x)[e % 4]; }
    __device__ __forceinline__ static int fragment_place(int r, int c) { return c * 16 + (r ^ 2 * c); }
    __device__ __forceinline__ void write_col(unsigned char *buf, const u32x4 (&part)[S::SHARE][3], int n) const
    {
        *(u32x4 *)(buf + n % 3 * S::PIECE + ((wave + S::WAVES * (n / 3)) * 64 + fragment_place(row, chunk)) * 16) = part[n / 3][n % 3];
    }
    __device__ __forceinline__ int slot() const { return fragment_place(lane & 15, lane >> 4); }
};

template <typename T>
__device__ __forceinline__ void four_or_zeros(const T *__restrict__ p, bool in, float (&v)[4])
{
    const ChunkOf<T> q = *(const ChunkOf<T> *)p;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        v[e] = in ? widen(q[e]) : 0.f;
}

template <class S, typename W>
__global__ __launch_bounds__(S::THREADS, S::FB == 4 ? 2 : 1) void head_layer1_split_kernel(
    const float *__restrict__ x, const int32_t *__restrict__ slot, int B, int d, int d_h, const W *__restrict__ w1,
    int kchunk, int nks, int jtiles, float *__restrict__ act_part)
{
    static_assert(S::ROWS == FJ, "tile");
    constexpr int FA = S::FA, FB = S::FB;
    constexpr bool TURNS = Layer1Source<S, W>::ROWS_TURN;
    constexpr int TURN = TURNS ? FA * Layer1Source<S, W>::TURN_BYTES : 0;
    __shared__ __align__(16) unsigned char lds[S::LDS_BYTES + S::WAVES * TURN];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, kq = lane >> 4;
    // the slice index varies fastest over the grid: an XCD pulls only its own slices of both operands
    const int kslice = blockIdx.x % nks;
    const int tile = blockIdx.x / nks;
    const int j0 = (tile % jtiles) * S::ROWS, s0 = (tile / jtiles) * S::COLS;

    Layer1Source<S, W> src;
    src.kbeg = kslice * kchunk;
    src.kend = min(d, src.kbeg + kchunk);
    src.row = lane >> 2, src.chunk = lane & 3, src.wave = wave, src.lane = lane;
    src.wchunk = TURNS ? src.chunk : kq;
    src.turn = lds + S::LDS_BYTES + wave * TURN;
#pragma unroll
    for (int a = 0; a < FA; ++a) {
        const int j = min(j0 + 16 * (wave * FA + a) + (TURNS ? src.row : l15), d_h - 1);  // clamped rows are computed and dropped
        src.w[a] = w1 + (long)j * d;
    }
#pragma unroll
    for (int p = 0; p < S::SHARE; ++p) {
        const int sq = min(s0 + 16 * (wave + S::WAVES * p) + src.row, B - 1);
        src.x[p] = x + (long)(slot ? slot[sq] : sq) * d;
    }
    split_f32x4 acc[FA][FB];
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int b = 0; b < FB; ++b)
            acc[a][b] = split_f32x4{0.f, 0.f, 0.f, 0.f};
    if (src.kbeg < src.kend)
        split_contract<S>(lds, (src.kend - src.kbeg + S::STEP - 1) / S::STEP, acc, src);
    if (__builtin_expect(!all_finite(acc), 0)) {  // (behind the kernel: in between, its code is a cold fetch for all)
        const W *wp[FA];
        const float *xp[FB];
#pragma unroll
        for (int a = 0; a < FA; ++a)
            wp[a] = w1 + (long)min(j0 + 16 * (wave * FA + a) + l15, d_h - 1) * d;
#pragma unroll
        for (int b = 0; b < FB; ++b) {
            const int sq = min(s0 + 16 * b + l15, B - 1);
            xp[b] = x + (long)(slot ? slot[sq] : sq) * d;
        }
        redo_not_finite(src.kend - src.kbeg, acc, [&](int i, float (&av)[FA][4], float (&bv)[FB][4]) {
            // a slice is a multiple of 4 long: the four elements are inside or past the end
            const int k = src.kbeg + 16 * i + 4 * kq, at = min(k, src.kend - 4);
#pragma unroll
            for (int a = 0; a < FA; ++a)
                four_or_zeros(wp[a] + at, k < src.kend, av[a]);
#pragma unroll
            for (int b = 0; b < FB; ++b)
                four_or_zeros(xp[b] + at, k < src.kend, bv[b]);
        });
    }

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

// Layer 2 of a scalar head: pred = b2 + w2 . act[b,:].  NS sequences per workgroup (head_tail.h).
// LDS: a[NS][lda] | part[NS][TAIL_WAVES]
template <bool WBF16, TailRow ROW, int NS>
__global__ __launch_bounds__(TAIL_THREADS) void head_scalar_kernel(const float *__restrict__ act_part, int nks, int B,
                                                                   const float *__restrict__ b1, int d_h,
                                                                   const void *__restrict__ w2_any,
                                                                   const float *__restrict__ b2, float *__restrict__ pred)
{
    using W = std::conditional_t<WBF16, unsigned short, float>;
    constexpr bool TINY = ROW == TAIL_TINY;
    const W *w2 = (const W *)w2_any;
    __shared__ float4 join[tail_joins<ROW, NS>];
    extern __shared__ __align__(16) float a[];
    const int b0 = blockIdx.x * NS, lda = tail_row(d_h);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *part = a + NS * lda;
    // thread t takes the chunks t, t + TAIL_THREADS, ... of the dot product (fixed assignment: bit-reproducible)
    const float bias = b2 ? b2[0] : 0.f;
    ChunkOf<W> w = load_chunk(w2, RowChunk<TINY>(tid, d_h), d_h);
    hidden_units<ROW, NS>(act_part, nks, B, b0, d_h, b1, a, lda, join, nullptr);
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
template <bool WBF16, TailRow ROW, int NS>
__global__ __launch_bounds__(TAIL_THREADS) void head_bins_kernel(const float *__restrict__ act_part, int nks, int B,
                                                                 const float *__restrict__ b1, int d_h, int n_out,
                                                                 const void *__restrict__ w2,
                                                                 const float *__restrict__ b2,
                                                                 const float *__restrict__ centers,
                                                                 float *__restrict__ pred, float *__restrict__ p_hat)
{
    using W = std::conditional_t<WBF16, unsigned short, float>;
    __shared__ float4 join[tail_joins<ROW, NS>];
    extern __shared__ __align__(16) float a[];
    const int b0 = blockIdx.x * NS, lda = tail_row(d_h);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *z = a + NS * lda;
    // bin o < 64 belongs to lane o: its bias and centre are asked for now
    const int o_near = min(lane, n_out - 1);
    const float b2_near = b2 ? b2[o_near] : 0.f, center_near = centers[o_near];
    output_layer<ROW, NS>((const W *)w2, n_out, d_h, a, lda, z,
                          [&] { hidden_units<ROW, NS>(act_part, nks, B, b0, d_h, b1, a, lda, join, nullptr); });
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

// More sequences: from F32_MAX_PRODUCTS on, the pieces.  They take 5.6 us at the least where the fp32 kernel, in thinner slices, takes
// 4.5.  Both at 121 sizes, 65 to 1024 sequences, d = 256 to 2048, d_h = 64 to 1024, fp32 instructions / pieces (us):
//   2^21 to 2^23 products   4.5 to 5.2 / 5.6 to 6.3           3 2^23   5.8 to 7.3 / 6.1 to 6.9
//   2^24                    4.7 to 6.0 / 5.7 to 6.5           2^25     5.6 to 8.1 / 6.2 to 7.4
//   3 2^24                  7.2 to 10.6 / 6.6 to 7.4          2^26     6.6 to 16.7 / 6.7 to 7.9
// Counted in whole tiles of 64 x 64, of which the instructions take all, and so that the number of planes follows the number
// of tiles of sequences alone, on which its bound rests.
constexpr long F32_MAX_PRODUCTS = 1L << 24;
static bool f32_serves(int d, int d_h, int32_t B)
{
    return B <= F32_MAX_SEQS || (long)((B + TN - 1) / TN) * ((d_h + TM - 1) / TM) <= F32_MAX_PRODUCTS / (TM * TN) / d;
}

// Slices of layer 1 on bf16 pieces, fp32 weights, n of them asked for.  Tiles of 128 columns run one to a compute unit: from n down
// to half of it, the number whose rounds take the fewest steps (one more for a round's start), the smaller of two (planes).
// 512 sequences, d = 5120, d_h = 1280: 320 tiles in two rounds 71.6 us, 240 in one 43; 1017 115 -> 77; 300, d = 4096, d_h = 1024 36 -> 25.
static int split_slices(int n, int d, int d_h, int32_t B)
{
    constexpr int STEP = WideTile::STEP, UNITS = 256;
    const long tiles = (long)((d_h + FJ - 1) / FJ) * ((B + WideTile::COLS - 1) / WideTile::COLS);
    int best = n;
    long best_steps = 0;
    for (int m = n; m >= (n + 1) / 2; --m) {
        const long steps = ((d + m - 1) / m + STEP - 1) / STEP, cost = (tiles * m + UNITS - 1) / UNITS * (steps + 1);
        if (m == n && steps < SPLIT_WIDE_STEPS)
            break;  // tiles of 64 columns
        if (m == n || cost <= best_steps)
            best = m, best_steps = cost;
    }
    return best;
}

int head_k_splits(int d, int d_h, int32_t B, int wdtype)
{
    if (skinny_serves(d, B, wdtype))
        return skinny_slices(d);
    int base = (d + 511) / 512;  // slices of at most 512 along d ...
    base = base < 1 ? 1 : (base > 8 ? 8 : base);
    const long tiles = (long)((d_h + TM - 1) / TM) * ((B + TN - 1) / TN);
    // (bf16, d = 4096, d_h = 1024, both layers: twice as many slices cost 24 sequences 15.8 us for 12.0, 128 22.2 for 17.0)
    const int wanted = wdtype == DT_F32 ? 1024 : 512;
    long want = tiles > 0 ? (wanted + tiles - 1) / tiles : 1;  // ... thinner when the batch has few tiles
    const int cap = (d + TK - 1) / TK < 64 ? (d + TK - 1) / TK : 64;
    long n = want > base ? want : base;
    n = n > cap ? cap : n;
    if (wdtype == DT_F32) {  // larger tiles: fewer slices
        const long ftiles = (long)((d_h + FJ - 1) / FJ) * ((B + f32_tile_seqs(B) - 1) / f32_tile_seqs(B));
        const long fwant = ftiles > 0 ? (F32_WORKGROUPS + ftiles - 1) / ftiles : 1;
        n = n > fwant ? fwant : n;
        if (!f32_serves(d, d_h, B))
            n = split_slices((int)(n > (d + 63) / 64 ? (d + 63) / 64 : n), d, d_h, B);  // a slice of at least two K steps
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
        const bool small = f32_serves(d, d_h, B);
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
            EGTP_LAYER1_F32((head_layer1_split_kernel<WideTile, float>));
        else if (!small)
            EGTP_LAYER1_F32((head_layer1_split_kernel<NarrowTile, float>));
        else if (fs == 64)
            EGTP_LAYER1_F32(head_layer1_f32_kernel<2>);
        else
            EGTP_LAYER1_F32(head_layer1_f32_kernel<1>);
#undef EGTP_LAYER1_F32
        return hipGetLastError();
    }
    if (wdtype == DT_BF16 && d % 8 == 0) {
        constexpr int STEP = NarrowTile::STEP;
        const int kchunk_b = ((d + nks - 1) / nks + STEP - 1) / STEP * STEP;  // (late slices may be empty and then write zeros)
        const int jtiles = (d_h + FJ - 1) / FJ;
        const long wgs = (long)jtiles * ((B + NarrowTile::COLS - 1) / NarrowTile::COLS) * nks;
        if (wgs > 0x7fffffffL)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL((head_layer1_split_kernel<NarrowTile, unsigned short>), dim3((unsigned)wgs), dim3(256), 0, st, x, slot, B,
                           d, d_h, (const unsigned short *)w1, kchunk_b, nks, jtiles, act_part);
        return hipGetLastError();
    }
    const int kchunk = ((d + nks - 1) / nks + TK - 1) / TK * TK;  // multiple of the K step
    hipLaunchKernelGGL(head_layer1_kernel, dim3((d_h + TM - 1) / TM, (B + TN - 1) / TN, nks), dim3(256), 0, st, x, slot, B,
                       d, d_h, (const unsigned short *)w1, kchunk, act_part);
    return hipGetLastError();
}

template <bool WBF16, TailRow ROW, int NS>
static hipError_t launch_layer2(const HeadArgs &a, int nks, size_t lds, hipStream_t st)
{
    static DeviceMask raised_scalar{0}, raised_bins{0};
    const dim3 grid((a.B - 1) / NS + 1), block(TAIL_THREADS);
    hipError_t e;
    if (a.n_out == 1) {
        e = raise_dynamic_lds_limit((const void *)head_scalar_kernel<WBF16, ROW, NS>, (int)TAIL_LDS_LIMIT, raised_scalar);
        if (e == hipSuccess)
            hipLaunchKernelGGL((head_scalar_kernel<WBF16, ROW, NS>), grid, block, NS * lds, st, a.act, nks, a.B, a.b1, a.d_h,
                               a.w2, a.b2, a.pred);
    } else {
        e = raise_dynamic_lds_limit((const void *)head_bins_kernel<WBF16, ROW, NS>, (int)TAIL_LDS_LIMIT, raised_bins);
        if (e == hipSuccess)
            hipLaunchKernelGGL((head_bins_kernel<WBF16, ROW, NS>), grid, block, NS * lds, st, a.act, nks, a.B, a.b1, a.d_h,
                               a.n_out, a.w2, a.b2, a.bin_centers, a.pred, a.p_hat);
    }
    return e == hipSuccess ? hipGetLastError() : e;
}

template <bool WBF16>
static hipError_t launch_layer2(const HeadArgs &a, int nks, size_t lds, hipStream_t st)
{
    return tail_launch(a.d_h, tail_sequences(a.B, lds), [&](auto row, auto ns) {
        return launch_layer2<WBF16, decltype(row)::value, decltype(ns)::value>(a, nks, lds, st);
    });
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
