// One optimisation step of a K-bin prediction head on frozen features (Section 3.2, 3.3):
// soft labels of Eq. 5, the joint loss of Eq. 7, the per-sequence step average of Eq. 9
// (as a per-sample weight), the backward pass through the head only, and AdamW.
//
// Master weights, moments, activations and sums are fp32.  For large batches (layer 1 from 65 samples and 2^24 products on, W1's
// gradient from 192 samples on) fp32 products are formed from bf16 pieces, six of the nine of a pair; what is left out is 2^-24 of a product at most
// (split_mfma.h).  Three launches:
//   1. layer 1 forward     partial pre-activations, split along d   (shared with scoring)
//   2. per-sample kernel   ReLU, logits, softmax, expected value, soft label, the two loss
//                          terms, d loss / d logits and d loss / d pre-activation
//   3. the updates, one grid of three kinds of workgroups that only need what 2. left behind:
//      W1                  gradient tile [64 x 64] of  dact^T . x  accumulated over the batch in
//                          registers and consumed by AdamW on the spot (128 x 64 for large
//                          batches) -- the d_h x d gradient is never written unless the
//                          caller asks for a copy.  With the
//                          paper's batch of 16 this part is a pure stream over W1 and its two
//                          moments (read and written once each).
//      small parameters    gradient of W2, b2 and b1, 64 columns a workgroup, reduced over the batch in a fixed
//                          order and consumed by AdamW on the spot
//      loss                fixed-order sum of the per-sample terms (the last workgroup)
// No floating-point atomics anywhere: results are bit-reproducible.
#include "head_tail.h"
#include "kernels.h"
#include "split_mfma.h"
#include "wave_reduce.h"

namespace egtp {
namespace {

struct Adam {
    float lr, beta1, beta2, omb1, omb2, eps, wd, corr1, corr2;
    float step, inv_corr2, decay;  // lr / corr1, 1 / corr2, lr wd
    bool quick;                    // eps is at least QUICK_EPS
};

// Decoupled weight decay: w <- w - lr wd w - lr mhat / (sqrt(vhat) + eps).
// With the divisions and the square root rounded correctly this is 59 vector instructions, 13 as it is: the quotients by the
// corrections are products, root and reciprocal the hardware's (within one unit in the last place each, of an update that is
// lr of the weight).  The root flushes denormals, 1e-19 beside an eps of at least QUICK_EPS.  64 samples, d = 4096, d_h = 1024 42.9 -> 38.8 us a
// step, 256 60.3 -> 56.9, 1024 127.5 -> 123.8; 16, the stream of W1 and its moments, 31.4 -> 31.0.
constexpr float QUICK_EPS = 1e-12f;
__device__ __forceinline__ void adamw(const Adam &h, float g, float &w, float &m, float &v)
{
    m = h.beta1 * m + h.omb1 * g;
    v = h.beta2 * v + h.omb2 * g * g;
    if (__builtin_expect(h.quick, 1)) {
        const float r = __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(v * h.inv_corr2) + h.eps);
        w = fmaf(-h.decay, w, w);
        w = fmaf(-(h.step * m), r, w);
    } else {
        const float mhat = m / h.corr1;
        const float vhat = v / h.corr2;
        w = w - h.lr * h.wd * w - h.lr * mhat / (sqrtf(vhat) + h.eps);
    }
}

// ---- 2. the samples, NS per workgroup (head_tail.h) ---------------------------------------
// LDS: a[NS][lda] | z[NS][K] | dz[NS][K]
constexpr int DACT_ROWS = 20;  // rows of W2 in flight per thread

template <TailRow ROW, int NS>
__global__ __launch_bounds__(TAIL_THREADS) void train_sample_kernel(
    const float *__restrict__ act_part, int nks, int B, int d_h, int K, const float *__restrict__ b1,
    const float *__restrict__ w2, const float *__restrict__ b2, const float *__restrict__ centers,
    const int32_t *__restrict__ bin, const float *__restrict__ y, const int32_t *__restrict__ steps, int n_seqs,
    float lambda, float *__restrict__ act, float *__restrict__ dact, float *__restrict__ dz_out,
    float *__restrict__ loss_part)
{
    __shared__ float4 join[tail_joins<ROW, NS>];
    extern __shared__ __align__(16) float a[];
    const int b0 = blockIdx.x * NS, lda = tail_row(d_h);
    float *z = a + NS * lda;
    float *dz = z + NS * K;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // what the softmax of wave w's sample needs is asked for now; bin o < 64 belongs to lane o
    const int b = min(b0 + min(wave, NS - 1), B - 1);
    const int o_near = min(lane, K - 1), bin_b = bin[b], steps_b = steps ? steps[b] : 0;
    const float y_b = y[b], b2_near = b2[o_near], center_near = centers[o_near];
    output_layer<ROW, NS>(w2, K, d_h, a, lda, z,
                          [&] { hidden_units<ROW, NS>(act_part, nks, B, b0, d_h, b1, a, lda, join, act); });
    // ... and before the softmax the first rows of this thread's column of W2
    float w[DACT_ROWS];
    auto load_rows = [&](int o0, int j) {
        const float *p = w2 + (long)o0 * d_h;
#pragma unroll
        for (int o = 0; o < DACT_ROWS; ++o) {
            w[o] = p[j];
            p += o0 + o + 1 < K ? d_h : 0;  // past the end: a valid row, not used
        }
    };
    // (wide: a thread's columns tid, tid + 1024, ... of all samples; narrow: a group of 256 threads for each sample)
    constexpr bool NARROW = ROW != TAIL_WIDE;
    const int j0 = NARROW ? tid % TAIL_NARROW_COLS : tid, n0 = NARROW ? tid / TAIL_NARROW_COLS : 0;
    const bool busy = !NARROW || n0 < NS;  // the same for a wave
    if (busy)
        load_rows(0, min(j0, d_h - 1));
    __syncthreads();
    if (wave < NS) {
        const bool kept = b0 + wave < B;
        float *zs = z + wave * K, *ds = dz + wave * K;
        const int i = bin_b < 0 ? 0 : (bin_b >= K ? K - 1 : bin_b);
        float m = -__builtin_inff();
#pragma unroll 1
        for (int o = lane; o < K; o += 64) {
            const float v = zs[o] + (o < 64 ? b2_near : b2[o]);
            zs[o] = v;
            m = fmaxf(m, v);
        }
        m = wave_max(m);
        float S = 0.f, Zl = 0.f;  // normalisers of the prediction and of the soft label (Eq. 5)
#pragma unroll 1
        for (int o = lane; o < K; o += 64) {
            const float e = expf(zs[o] - m);
            ds[o] = e;
            S += e;
            Zl += expf(-fabsf((float)(o - i)));
        }
        S = wave_sum(S);
        Zl = wave_sum(Zl);
        const float lnS = logf(S);
        float yhat = 0.f, ce = 0.f;
#pragma unroll 1
        for (int o = lane; o < K; o += 64) {
            const float ph = ds[o] / S;
            const float p = expf(-fabsf((float)(o - i))) / Zl;
            yhat = fmaf(ph, o < 64 ? center_near : centers[o], yhat);  // Eq. 6
            ce -= p * ((zs[o] - m) - lnS);
        }
        yhat = wave_sum(yhat);
        ce = wave_sum(ce);
        const float err = yhat - y_b;
        // Eq. 9: a sequence's steps share its 1/N; without step counts every sample weighs 1/B
        const float wb = steps ? 1.0f / ((float)n_seqs * (float)steps_b) : 1.0f / (float)B;
#pragma unroll 1
        for (int o = lane; o < K; o += 64) {
            const float ph = ds[o] / S;
            const float p = expf(-fabsf((float)(o - i))) / Zl;
            const float center = o < 64 ? center_near : centers[o];
            const float g = wb * (lambda * (ph - p) + (1.0f - lambda) * 2.0f * err * ph * (center - yhat));
            ds[o] = g;
            if (kept)
                dz_out[(long)b * K + o] = g;
        }
        if (lane == 0 && kept) {
            loss_part[2 * b] = wb * ce;
            loss_part[2 * b + 1] = wb * err * err;
        }
    }
    __syncthreads();
    // d loss / d pre-activation = (W2^T dz) where the unit is active
    if (!busy)
        return;
    constexpr int PER = NARROW ? 1 : NS;  // samples of a thread
#pragma unroll 1
    for (int j = j0; j < d_h; j += TAIL_THREADS) {
        float s[PER] = {};
#pragma unroll 1
        for (int o0 = 0; o0 < K; o0 += DACT_ROWS) {
            if (j != j0 || o0 > 0)
                load_rows(o0, j);
#pragma unroll
            for (int o = 0; o < DACT_ROWS; ++o)
                if (o0 + o < K)
#pragma unroll
                    for (int n = 0; n < PER; ++n)
                        s[n] = fmaf(dz[(n0 + n) * K + o0 + o], w[o], s[n]);
        }
#pragma unroll
        for (int n = 0; n < PER; ++n)
            if (b0 + n0 + n < B)
                dact[(long)(b0 + n0 + n) * d_h + j] = a[(n0 + n) * lda + hidden_place(j, d_h)] > 0.f ? s[n] : 0.f;
    }
}

// ---- 5. loss = {lambda CE + (1 - lambda) MSE, CE, MSE}, fixed summation order -----------------
// (one workgroup of 256 threads; runs as the last workgroup of the update launch)
__device__ void sum_loss(const float *__restrict__ loss_part, int B, float lambda, float *__restrict__ loss)
{
    __shared__ float red[2][256];
    const int tid = threadIdx.x;
    float ce = 0.f, mse = 0.f;
    for (int b = tid; b < B; b += 256) {
        ce += loss_part[2 * b];
        mse += loss_part[2 * b + 1];
    }
    red[0][tid] = ce;
    red[1][tid] = mse;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) {
            red[0][tid] += red[0][tid + s];
            red[1][tid] += red[1][tid + s];
        }
        __syncthreads();
    }
    if (tid == 0) {
        loss[0] = lambda * red[0][0] + (1.0f - lambda) * red[1][0];
        loss[1] = red[0][0];
        loss[2] = red[1][0];
    }
}

// ---- 3. W2, b2, b1: sums over the batch of columns of act, dz and dact ----------------------
// Workgroup = 64 columns; wave q adds the samples b = q, q + 4, ... (each a coalesced load of 64 columns, SAMPLES_AHEAD in
// flight: one sample after the other is a chain of cache latencies), then the four partial sums are joined in order.
// These workgroups start when the first W1 tiles end and are the end of a large batch's launch: with eight samples in
// flight and dz loaded beside each the whole step took 205.5 us at batch 1024, now 202.2; at batch 309, d = 2208, 55.8, 54.6.
// NO > 0: the column is weighted with dz[b][o0 .. o0 + NO - 1] (rows of W2's gradient; a load of act serves all of
// them); NO = 0: a plain column sum (the biases).  Parameter (o, column) sits at base + o * ld + column.
constexpr int W2_ROWS = 4;  // rows of W2 per workgroup
constexpr int SAMPLES_AHEAD = 32;

struct Params {
    float *w, *m, *v, *g;
};

template <int NO>
__device__ __forceinline__ void column_update(const float *__restrict__ mat, long ld, int n, int col0,
                                              const float *__restrict__ dz, int K, int o0, int B, const Adam &h,
                                              const Params &p, float *__restrict__ red)
{
    constexpr int NR = NO > 0 ? NO : 1;
    static_assert(NR <= 4 && SAMPLES_AHEAD == 32, "two factors per lane");
    const int lane = threadIdx.x & 63, q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = min(col0 + lane, n - 1);  // clamped columns are computed and dropped
    float s[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r)
        s[r] = 0.f;
    // The factors of a chunk of samples are spread over the lanes, two each, and read from there: loaded by every lane
    // they would be four loads for each of act.
    for (int b0 = q; b0 < B; b0 += 4 * SAMPLES_AHEAD) {
        const int n = (B - b0 + 3) / 4;  // samples of this wave from b0 on
        float v[SAMPLES_AHEAD], f[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < SAMPLES_AHEAD; ++i)  // past the end: the last sample, not used
            v[i] = mat[min(b0 + 4 * i, B - 1) * ld + col];
        if (NO > 0) {
            const int b = min(b0 + 4 * (lane & (SAMPLES_AHEAD - 1)), B - 1), o = o0 + lane / SAMPLES_AHEAD;
            f[0] = dz[(long)b * K + min(o, K - 1)];
            f[1] = dz[(long)b * K + min(o + 2, K - 1)];
        }
#pragma unroll
        for (int i = 0; i < SAMPLES_AHEAD; ++i)
            if (i < n)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    s[r] = NO > 0 ? fmaf(__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f[r >> 1]),
                                                                                  i + SAMPLES_AHEAD * (r & 1))),
                                         v[i], s[r])
                                  : s[r] + v[i];
    }
#pragma unroll
    for (int r = 0; r < NR; ++r)
        red[(q * NR + r) * 64 + lane] = s[r];
    __syncthreads();
    // wave q finishes the rows q, q + 4, ...
    for (int r = q; r < NR; r += 4) {
        if (col0 + lane >= n || (NO > 0 && o0 + r >= K))
            continue;
        float g = red[r * 64 + lane];
#pragma unroll
        for (int k = 1; k < 4; ++k)
            g += red[(k * NR + r) * 64 + lane];
        const long e = NO > 0 ? (o0 + r) * ld + col : col;
        float wv = p.w[e], mv = p.m[e], vv = p.v[e];
        adamw(h, g, wv, mv, vv);
        p.w[e] = wv;
        p.m[e] = mv;
        p.v[e] = vv;
        if (p.g)
            p.g[e] = g;
    }
}

// ---- 4. W1: gradient tile in registers, AdamW in the epilogue -------------------------------
// gradient[j][k] = sum over samples of dact[b][j] x[b][k], on the fp32 matrix cores (16x16x4: fp32 operands, products
// and sums).  Two bounds: the stream over W1 and its two moments (24 bytes per parameter, whatever the batch) and, from
// a few hundred samples on, the fp32 matrix rate.  Workgroup = 4 waves; a wave's tile is 16 rows j x 64 columns k.
// Both operands lie with the sample as the slow index, so a K step of four samples is staged and read as rows: lane l
// reads row j = l % 16 and four neighbouring k of sample 4 s + l / 16, which makes column tile n of a wave the
// columns 4 (column) + n; a lane then ends up with four neighbouring columns of a row, one 16-byte access each to W1
// and the moments.  Batch 1024, the launch with its small parameters: 390 us with 64 x 64 tiles of fp32 FMAs, now 117 to 120.
// 64 x 64 per workgroup, 32 samples per LDS stage.  128 x 128 tiles halve the operand traffic and gain nothing for it
// (whole step at batch 1024, d = 4096, d_h = 1024: 198 us against 199) while few of them leave the chip idle (batch
// 1024, d = 1024, d_h = 300: 131 us against 65).
constexpr int GM = 64, GN = 64, GB = 32;
constexpr int GRAD_STAGE_FLOATS = GB * (GM + GN);  // As[GB][GM] | Bs[GB][GN]

__device__ __forceinline__ void w1_update(int tile_k, int tile_j, const float *__restrict__ x,
                                          const float *__restrict__ dact, int B, int d, int d_h, const Adam &h,
                                          float *__restrict__ w1, float *__restrict__ m_w1, float *__restrict__ v_w1,
                                          float *__restrict__ g_w1, float *__restrict__ lds)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    constexpr int A_PIECES = GB * GM / 1024, B_PIECES = GB * GN / 1024;  // 16-byte pieces per thread
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l15 = lane & 15, kq = lane >> 4;
    const int k0 = tile_k * GN, j0 = tile_j * GM;
    const int wj = wave * 16;

    float4 ar[A_PIECES], br[B_PIECES];
    const bool whole = (d_h & 3) == 0;  // rows of dact are 16-byte aligned
    auto fetch = [&](int b0) {
#pragma unroll
        for (int p = 0; p < A_PIECES; ++p) {
            const int e = (tid + 256 * p) * 4, b = b0 + e / GM, j = j0 + e % GM;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (b < B) {
                const float *dp = dact + (long)b * d_h + j;
                if (whole && j < d_h) {
                    v = *(const float4 *)dp;
                } else {
                    v.x = j + 0 < d_h ? dp[0] : 0.f;
                    v.y = j + 1 < d_h ? dp[1] : 0.f;
                    v.z = j + 2 < d_h ? dp[2] : 0.f;
                    v.w = j + 3 < d_h ? dp[3] : 0.f;
                }
            }
            ar[p] = v;
        }
#pragma unroll
        for (int p = 0; p < B_PIECES; ++p) {
            const int e = (tid + 256 * p) * 4, b = b0 + e / GN, k = k0 + e % GN;
            br[p] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (b < B && k < d)  // d is a multiple of 4: the whole piece is inside the row
                br[p] = *(const float4 *)(x + (long)b * d + k);
        }
    };
    auto stage = [&](float *buf) {
#pragma unroll
        for (int p = 0; p < A_PIECES; ++p)
            *(float4 *)(buf + (tid + 256 * p) * 4) = ar[p];
#pragma unroll
        for (int p = 0; p < B_PIECES; ++p)
            *(float4 *)(buf + GB * GM + (tid + 256 * p) * 4) = br[p];
    };

    f32x4 acc[4];
#pragma unroll
    for (int n = 0; n < 4; ++n)
        acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    fetch(0);
    // the tile's parameters and moments are asked for now, so that the stream runs beside the contraction
    const int k = k0 + 4 * l15;
    float4 w[4], m[4], v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // rows and columns that do not exist: a valid place, not used
        const long at = (long)min(j0 + wj + 4 * kq + i, d_h - 1) * d + min(k, d - 4);
        w[i] = *(const float4 *)(w1 + at);
        m[i] = *(const float4 *)(m_w1 + at);
        v[i] = *(const float4 *)(v_w1 + at);
    }
    stage(lds);
    __syncthreads();
    int cur = 0;
    for (int b0 = 0; b0 < B; b0 += GB) {
        const bool more = b0 + GB < B;
        if (more)
            fetch(b0 + GB);
        const float *buf = lds + cur * GRAD_STAGE_FLOATS;
#pragma unroll
        for (int s = 0; s < GB / 4; ++s) {
            const float av = buf[(4 * s + kq) * GM + wj + l15];
            const f32x4 bv = *(const f32x4 *)(buf + GB * GM + (4 * s + kq) * GN + 4 * l15);
#pragma unroll
            for (int n = 0; n < 4; ++n)
                acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[n], acc[n], 0, 0, 0);
        }
        if (more)
            stage(lds + (cur ^ 1) * GRAD_STAGE_FLOATS);  // nobody reads that buffer now
        __syncthreads();
        cur ^= 1;
    }
    if (k >= d)
        return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = j0 + wj + 4 * kq + i;
        if (j >= d_h)
            continue;
        const long at = (long)j * d + k;
        adamw(h, acc[0][i], w[i].x, m[i].x, v[i].x);
        adamw(h, acc[1][i], w[i].y, m[i].y, v[i].y);
        adamw(h, acc[2][i], w[i].z, m[i].z, v[i].z);
        adamw(h, acc[3][i], w[i].w, m[i].w, v[i].w);
        *(float4 *)(w1 + at) = w[i];
        *(float4 *)(m_w1 + at) = m[i];
        *(float4 *)(v_w1 + at) = v[i];
        if (g_w1)
            *(float4 *)(g_w1 + at) = make_float4(acc[0][i], acc[1][i], acc[2][i], acc[3][i]);
    }
}

// The same for more samples: fp32 products as bf16 pieces (split_mfma.h).  Workgroup = 128 rows j x 64 columns k, a wave 32
// rows of its own.  The contraction runs over the samples, the slow index of both operands, of which a fragment wants eight
// in a lane: a lane loads two neighbouring j of eight samples and deals them to two fragments, so that row c of a wave's
// fragment a is j = 2 c + a; of the columns it loads four neighbouring k of two samples, a pair of K elements for each of four
// fragments, so that column c of fragment b is k = 4 c + b.  A lane ends up with four neighbouring k of a row j, one 16-byte
// access each to W1 and the moments.
// Two workgroups per compute unit; the workgroups of the small parameters, chains of cache latencies, start before the
// tiles, which puts some tiles' parameter streams beside others' products (512 samples 92.7 -> 89.1 us a step).
// Bound: the splitting beside the MFMAs, 49 us per 1024 samples at d = 4096, d_h = 1024, and about 30 us for the parameters.
// 1024 samples: the launch 117 to 120 us on the fp32 matrix instructions, then 75 to 82; the way of loaded data back into
// the compute unit was the busiest part of it (69 %), a quarter of what a load of one k per lane fetched was used.  With
// four k per lane, a quarter of these loads: whole steps of 1024 samples 135.2 -> 127.4 us, 256 62.3 -> 58.4, 1024 at d = 5120,
// d_h = 1280 213 -> 195.5; the launch alone, clocks warm, 65 (75 to 85 in a short run).  128 x 128 tiles: 85.  Rows by
// 16-byte loads as well, turned in the LDS: no faster.
typedef SplitTile<2, 4> GradTile;
// From this many samples and tiles on.  Whole steps, us, fp32 instructions / pieces:
//   512 tiles (d = 4096, d_h = 1024)   128 samples 55.2 / 56.4   160 66.8 / 64.0   192 70.5 / 67.1   256 72.9 / 67.4
//   144 tiles (d = 1024, d_h = 1100)   192 samples 39.6 / 38.0   512 63.3 / 54.9   768 83.0 / 68.7
//   128 tiles (d = 1024, d_h = 1024)   192 samples 32.0 / 34.2   384 44.5 / 44.8   512 46.7 / 45.9   768 64.4 / 61.7
//    48 tiles (d = 1024, d_h = 384)    192 samples 25.0 / 27.5   512 38.6 / 39.0   1024 62.0 / 58.9
// At up to 128 tiles, where half the compute units stay without one, the two meet at 400 to 500 samples, elsewhere
// at about 150: the line is up to 7 % off on its corner, 128 tiles and fewer than 384 samples.
constexpr int SPLIT_SAMPLES = 192, SPLIT_TILES = 128;

struct GradSource {
    static constexpr int ROW_PIECES = 3, ROW_LOADS = 8, COL_LOADS = 2, COL_WRITES = 12;
    static constexpr bool ROWS_TURN = false;
    struct Rows {
        float2 v[8];
    };
    struct Cols {
        float4 v[2];
    };
    const float *dact, *x;
    unsigned row_at, col_at;  // this lane's columns of the two operands and its first sample of a step, in bytes
    long d_h, d;
    int B, kq, wave, l15;

    // The last step (and those that are only asked for) takes the last 32 samples, of which the ones that an earlier step has
    // count as zeros: no branch around a load, so that the loads in flight stay countable, and addresses are scalar but for
    // row_at and col_at (a minimum and a 64-bit product per lane and load before: 66.2 -> 64.9 us at 1024 samples, d = 4096, d_h =
    // 1024, which pays for most of what the small products' sums cost).
    static_assert(SPLIT_SAMPLES >= GradTile::STEP, "a step's worth of samples");
    __device__ __forceinline__ int first(int i) const { return min(i * GradTile::STEP, B - GradTile::STEP); }
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t from(const float *p)
    {
        return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, -1, 0x00020000);
    }
    __device__ __forceinline__ void load_rows(int i, int l, Rows &r) const
    {
        r.v[l] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(from(dact + first(i) * d_h), row_at, l * (int)d_h * 4, 0));
    }
    __device__ __forceinline__ void load_cols(int i, int l, Cols &r) const
    {
        r.v[l] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(from(x + (first(i) + 8 * wave) * d), col_at, l * (int)d * 16, 0));
    }
    __device__ __forceinline__ void clear_rows(int i, Rows &r) const
    {
        if ((i + 1) * GradTile::STEP <= B)
            return;
#pragma unroll
        for (int l = 0; l < 8; ++l)
            if (first(i) + 8 * kq + l < i * GradTile::STEP)
                r.v[l] = make_float2(0.f, 0.f);
    }
    __device__ __forceinline__ void clear_cols(int i, Cols &r) const
    {
        if ((i + 1) * GradTile::STEP <= B)
            return;
#pragma unroll
        for (int l = 0; l < 2; ++l)
            if (first(i) + 8 * wave + 4 * l + kq < i * GradTile::STEP)
                r.v[l] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // K elements 2 g and 2 g + 1 of eight are samples g and g + 4: a pair is what a lane loads of a column
    __device__ __forceinline__ float row_value(const Rows &r, int a, int e) const
    {
        const float2 v = r.v[e / 2 + e % 2 * 4];
        return a == 0 ? v.x : v.y;
    }
    __device__ __forceinline__ float col_value(const Cols &r, int, int e) const { return (&r.v[e % 2].x)[e / 2]; }
    __device__ __forceinline__ void write_col(unsigned char *buf, const split_u32x4 (&part)[1][3], int n) const
    {
        *(unsigned *)(buf + n % 3 * GradTile::PIECE + n / 3 * 1024 + (wave * 16 + l15) * 16 + kq * 4) = part[0][n % 3][n / 3];
    }
    __device__ __forceinline__ int slot() const { return threadIdx.x & 63; }
};

__device__ __forceinline__ void w1_update_split(int tile_k, int tile_j, const float *__restrict__ x,
                                                const float *__restrict__ dact, int B, int d, int d_h, const Adam &h,
                                                float *__restrict__ w1, float *__restrict__ m_w1, float *__restrict__ v_w1,
                                                float *__restrict__ g_w1, unsigned char *__restrict__ lds)
{
    using S = GradTile;
    constexpr int FA = S::FA, FB = S::FB;
    static_assert(FA == 2 && FB == 4 && S::SHARE == 1, "two neighbouring j, four neighbouring k to a lane");
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k0 = tile_k * S::COLS, j0 = tile_j * S::ROWS + 32 * wave;

    // d_h and d are multiples of 4: rows and columns that do not exist are others', computed and dropped
    GradSource src;
    src.d_h = d_h, src.d = d, src.B = B, src.wave = wave;
    src.l15 = tid & 15, src.kq = tid >> 4 & 3;
    src.dact = dact, src.row_at = (unsigned)(8 * src.kq * d_h + min(j0 + 2 * src.l15, d_h - 2)) * 4;
    src.x = x, src.col_at = (unsigned)(src.kq * d + min(k0 + 4 * src.l15, d - 4)) * 4;  // a wave stages eight samples
    split_f32x4 acc[FA][FB];
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int b = 0; b < FB; ++b)
            acc[a][b] = split_f32x4{0.f, 0.f, 0.f, 0.f};
    const int steps = (B + S::STEP - 1) / S::STEP;
    __builtin_assume(steps >= SPLIT_SAMPLES / S::STEP);
    split_contract<S>(lds, steps, acc, src);
    int again = tid;  // the lane's place, not held over the contraction (two registers that it does not have)
    asm("" : "+v"(again));
    const int l15 = again & 15, kq = again >> 4 & 3;
    const int j_at = min(j0 + 2 * l15, d_h - 2), k_at = min(k0 + 4 * l15, d - 4);
    if (__builtin_expect(!all_finite(acc), 0))
        redo_not_finite(B, acc, [&](int i, float (&av)[FA][4], float (&bv)[FB][4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int b = 16 * i + 4 * kq + e, sample = min(b, B - 1);
                const float2 dv = *(const float2 *)(dact + (long)sample * d_h + j_at);
                const float4 xv = *(const float4 *)(x + (long)sample * d + k_at);
                av[0][e] = b < B ? dv.x : 0.f, av[1][e] = b < B ? dv.y : 0.f;
                bv[0][e] = b < B ? xv.x : 0.f, bv[1][e] = b < B ? xv.y : 0.f;
                bv[2][e] = b < B ? xv.z : 0.f, bv[3][e] = b < B ? xv.w : 0.f;
            }
        });

    const int k = k0 + 4 * l15;
    if (k >= d)
        return;
    float4 w[FA][4], m[FA][4], v[FA][4];
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // rows that do not exist: a valid place, not used
            const long at = (long)min(j0 + 2 * (4 * kq + i) + a, d_h - 1) * d + k;
            w[a][i] = *(const float4 *)(w1 + at);
            m[a][i] = *(const float4 *)(m_w1 + at);
            v[a][i] = *(const float4 *)(v_w1 + at);
        }
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = j0 + 2 * (4 * kq + i) + a;
            if (j >= d_h)
                continue;
            const long at = (long)j * d + k;
            const float4 grad = make_float4(acc[a][0][i], acc[a][1][i], acc[a][2][i], acc[a][3][i]);
            adamw(h, grad.x, w[a][i].x, m[a][i].x, v[a][i].x);
            adamw(h, grad.y, w[a][i].y, m[a][i].y, v[a][i].y);
            adamw(h, grad.z, w[a][i].z, m[a][i].z, v[a][i].z);
            adamw(h, grad.w, w[a][i].w, m[a][i].w, v[a][i].w);
            *(float4 *)(w1 + at) = w[a][i];
            *(float4 *)(m_w1 + at) = m[a][i];
            *(float4 *)(v_w1 + at) = v[a][i];
            if (g_w1)
                *(float4 *)(g_w1 + at) = grad;
        }
}

// ---- 3. + 4. + 5. in one launch: all three need only what the per-sample kernel left behind and touch
// disjoint parameters, so they share a grid.  The W1 tiles come first in launch order (they carry the
// memory traffic of the step), then the workgroups of the small parameters, the loss last.
struct UpdateArgs {
    const float *x, *act, *dact, *dz, *loss_part;
    int B, d, d_h, K;
    int tiles_k, tiles_w1;
    int cols_h, blocks_w2, blocks_b2;  // 64-column blocks of d_h; workgroups of W2 and of b2 (b1 has cols_h)
    float lambda;
    Params w1, w2, b2, b1;
    float *loss;
};

template <bool SPLIT>
__global__ __launch_bounds__(256, SPLIT ? 2 : 1) void train_update_kernel(UpdateArgs a, Adam h)
{
    constexpr int LDS_FLOATS = SPLIT ? GradTile::LDS_BYTES / 4 : 2 * GRAD_STAGE_FLOATS;
    __shared__ __align__(16) float lds[LDS_FLOATS];
    static_assert(LDS_FLOATS >= 4 * W2_ROWS * 64, "LDS of the small-parameter part");
    const int small = (int)gridDim.x - a.tiles_w1;  // the other workgroups: behind the tiles, or (split) before them
    int id = blockIdx.x;
    if (SPLIT)
        id = id < small ? a.tiles_w1 + id : id - small;
    if (id < a.tiles_w1) {
        const int tk = id % a.tiles_k, tj = id / a.tiles_k;
        if constexpr (SPLIT)
            w1_update_split(tk, tj, a.x, a.dact, a.B, a.d, a.d_h, h, a.w1.w, a.w1.m, a.w1.v, a.w1.g, (unsigned char *)lds);
        else
            w1_update(tk, tj, a.x, a.dact, a.B, a.d, a.d_h, h, a.w1.w, a.w1.m, a.w1.v, a.w1.g, lds);
        return;
    }
    id -= a.tiles_w1;
    if (id < a.blocks_w2) {
        column_update<W2_ROWS>(a.act, a.d_h, a.d_h, (id % a.cols_h) * 64, a.dz, a.K, (id / a.cols_h) * W2_ROWS, a.B, h, a.w2,
                               lds);
        return;
    }
    id -= a.blocks_w2;
    if (id < a.cols_h) {
        column_update<0>(a.dact, a.d_h, a.d_h, id * 64, nullptr, 0, 0, a.B, h, a.b1, lds);
        return;
    }
    id -= a.cols_h;
    if (id < a.blocks_b2)
        column_update<0>(a.dz, a.K, a.K, id * 64, nullptr, 0, 0, a.B, h, a.b2, lds);
    else
        sum_loss(a.loss_part, a.B, a.lambda, a.loss);
}

}  // namespace

template <TailRow ROW, int NS>
static hipError_t launch_samples(const TrainArgs &a, int nks, size_t lds, hipStream_t st)
{
    static DeviceMask raised{0};
    hipError_t e = raise_dynamic_lds_limit((const void *)train_sample_kernel<ROW, NS>, (int)TAIL_LDS_LIMIT, raised);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((train_sample_kernel<ROW, NS>), dim3((a.B - 1) / NS + 1), dim3(TAIL_THREADS), NS * lds, st, a.act_part,
                       nks, a.B, a.d_h, a.K, a.b1, a.w2, a.b2, a.centers, a.bin, a.y, a.steps, a.n_seqs, a.lambda, a.act,
                       a.dact, a.dz, a.loss_part);
    return hipGetLastError();
}

static hipError_t launch_samples(const TrainArgs &a, int nks, size_t lds, hipStream_t st)
{
    return tail_launch(a.d_h, tail_sequences(a.B, lds), [&](auto row, auto ns) {
        return launch_samples<decltype(row)::value, decltype(ns)::value>(a, nks, lds, st);
    });
}

hipError_t head_train_step(const TrainArgs &a, hipStream_t st)
{
    if (a.B <= 0)
        return hipSuccess;
    if (a.d % 4 != 0)
        return hipErrorInvalidValue;
    const size_t lds = ((size_t)tail_row(a.d_h) + 2 * (size_t)a.K) * sizeof(float);
    if (lds > TAIL_LDS_LIMIT)
        return hipErrorInvalidValue;
    hipError_t e = head_layer1(a.x, nullptr, a.B, a.d, a.d_h, a.w1, DT_F32, a.act_part, st);
    if (e != hipSuccess)
        return e;
    e = launch_samples(a, head_k_splits(a.d, a.d_h, a.B, DT_F32), lds, st);
    if (e != hipSuccess)
        return e;
    Adam h;
    h.lr = a.lr;
    h.beta1 = a.beta1;
    h.beta2 = a.beta2;
    h.omb1 = a.omb1;
    h.omb2 = a.omb2;
    h.eps = a.eps;
    h.wd = a.weight_decay;
    h.corr1 = a.corr1;
    h.corr2 = a.corr2;
    h.step = (float)((double)a.lr / (double)a.corr1);
    h.inv_corr2 = (float)(1.0 / (double)a.corr2);
    h.decay = (float)((double)a.lr * (double)a.weight_decay);
    h.quick = a.eps >= QUICK_EPS;
    // the parameter updates come last: the forward and the backward pass above read the old W1 / W2
    UpdateArgs u;
    u.x = a.x, u.act = a.act, u.dact = a.dact, u.dz = a.dz, u.loss_part = a.loss_part;
    u.B = a.B, u.d = a.d, u.d_h = a.d_h, u.K = a.K;
    u.lambda = a.lambda;
    u.w1 = {a.w1, a.m_w1, a.v_w1, a.g_w1};
    u.w2 = {a.w2, a.m_w2, a.v_w2, a.g_w2};
    u.b2 = {a.b2, a.m_b2, a.v_b2, a.g_b2};
    u.b1 = {a.b1, a.m_b1, a.v_b1, a.g_b1};
    u.loss = a.loss;
    // (rows of dact start on 8-byte boundaries; the gradient's offsets from a step's first sample are 32-bit)
    const bool split = a.B >= SPLIT_SAMPLES && a.d_h % 4 == 0 && a.d <= (1 << 26) &&
                       (long)((a.d_h + GradTile::ROWS - 1) / GradTile::ROWS) * ((a.d + GradTile::COLS - 1) / GradTile::COLS) >=
                           SPLIT_TILES;
    const int tile_j = split ? GradTile::ROWS : GM, tile_k = split ? GradTile::COLS : GN;
    const long tiles_k = (a.d + tile_k - 1) / tile_k, tiles_j = (a.d_h + tile_j - 1) / tile_j;
    u.tiles_k = (int)tiles_k;
    u.tiles_w1 = (int)(tiles_k * tiles_j);
    u.cols_h = (a.d_h + 63) / 64;
    u.blocks_w2 = u.cols_h * ((a.K + W2_ROWS - 1) / W2_ROWS);
    u.blocks_b2 = (a.K + 63) / 64;
    const long wgs = tiles_k * tiles_j + u.blocks_w2 + u.cols_h + u.blocks_b2 + 1;
    if (wgs > 0x7fffffffL)
        return hipErrorInvalidValue;
    if (split)
        hipLaunchKernelGGL(train_update_kernel<true>, dim3((unsigned)wgs), dim3(256), 0, st, u, h);
    else
        hipLaunchKernelGGL(train_update_kernel<false>, dim3((unsigned)wgs), dim3(256), 0, st, u, h);
    return hipGetLastError();
}

}  // namespace egtp
