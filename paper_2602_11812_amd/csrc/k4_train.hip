// One optimisation step of a K-bin prediction head on frozen features (Section 3.2, 3.3):
// soft labels of Eq. 5, the joint loss of Eq. 7, the per-sequence step average of Eq. 9
// (as a per-sample weight), the backward pass through the head only, and AdamW.
//
// Master weights, moments, activations and sums are fp32.  For large batches (layer 1 from 65 samples and 2^24 products on, W1's
// gradient from 160 or 256 samples on) fp32 products are formed from bf16 pieces, six of the nine of a pair; what is left out is 2^-24 of a product at most
// (split_mfma.h).  Three launches:
//   1. layer 1 forward     partial pre-activations, split along d   (shared with scoring)
//   2. per-sample kernel   ReLU, logits, softmax, expected value, soft label, the two loss
//                          terms, d loss / d logits and d loss / d pre-activation (for large batches in pieces, too)
//   3. the updates, one grid of three kinds of workgroups that only need what 2. left behind:
//      W1                  gradient tile [64 x 64] of  dact^T . x  accumulated over the batch in
//                          registers and consumed by AdamW on the spot (128 x 64 for large
//                          batches) -- the d_h x d gradient is never written unless the
//                          caller asks for a copy.  With the
//                          paper's batch of 16 this part is a pure stream over W1 and its two
//                          moments (read and written once each).
//      small parameters    gradient of W2, b2 and b1, reduced over the batch in a fixed order and consumed by
//                          AdamW on the spot
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
    float step, step_rest, inv_corr2, inv_corr2_rest, decay;  // lr / corr1 and 1 / corr2, each the sum of two; lr wd
    bool quick;                                               // eps and the step are in the range of the quick arithmetic
};

// Decoupled weight decay: w <- w - lr wd w - lr mhat / (sqrt(vhat) + eps).
// With the divisions and the square root rounded correctly this is 59 vector instructions, 23 as it is, and no less exact.  In units of 2^-24 of the
// update the old form had at most 1 for each of mhat, vhat (half of which the root leaves), the root, the sum with eps, lr mhat and the quotient: 5.5.
// Here lr mhat and vhat are products with constants of two floats (1 and, under the root, 0.5), the sum is 1, and the quotient by the hardware's reciprocal
// is corrected (1) by its remainder, with that of the hardware's root, x - root^2, over 2 (root + eps) in place of 2 root (of the root's 2 it leaves
// the share that eps has in the sum, 0.5 at most): 4.  Root and reciprocal flush denormals, 1e-19 beside an eps of at least QUICK_EPS; an
// infinite root (second moments past fp32's range) leaves no update, as a division would.  Root mean square against fp64, the same units, Gaussian features, eps =
// 1e-8: old form 0.94, as it is 0.81.  Whole steps with the old form / as it is, us, d = 4096, d_h = 1024: 1 sample 30.6 / 29.6, 16
// 31.4 / 31.4, 64 40.5 / 37.7, 128 48.5 / 45.3.
constexpr float QUICK_EPS = 1e-10f, QUICK_MOST = 1e10f, MOST = 3.402823466e38f;
__device__ __forceinline__ void adamw(const Adam &h, float g, float &w, float &m, float &v)
{
    m = h.beta1 * m + h.omb1 * g;
    v = h.beta2 * v + h.omb2 * g * g;
    if (__builtin_expect(h.quick, 1)) {
        const float u = fmaf(h.step, m, h.step_rest * m);
        const float x = fmaf(h.inv_corr2, v, h.inv_corr2_rest * v);
        const float root = __builtin_amdgcn_sqrtf(x);
        const float below = __builtin_elementwise_minimum(root + h.eps, MOST);  // (keeps NaN)
        const float r = __builtin_amdgcn_rcpf(below);
        const float q = u * r;
        const float root_off = __builtin_amdgcn_fmed3f(fmaf(-root, root, x) * r, -MOST, MOST);  // twice; of an infinite root not NaN
        const float rest = fmaf(-0.5f * q, root_off, fmaf(-q, below, u));
        w = fmaf(-h.decay, w, w) - fmaf(rest, r, q);
    } else {
        const float mhat = m / h.corr1;
        const float vhat = v / h.corr2;
        w = w - h.lr * h.wd * w - h.lr * mhat / (sqrtf(vhat) + h.eps);
    }
}

typedef SplitTile<2, 4> GradTile;  // of W1's gradient (part 4 below)
// dact as it is multiplied: fragments of 16 rows j x 32 samples (1 KiB: lane l of a wave holds row l % 16, samples 8 (l / 16) .. + 8),
// [step of 32 samples][fragment][piece], zeros past the batch and past d_h.
constexpr int FRAGMENT_BYTES = 1024, FRAGMENT_ROWS = 16;
__host__ __device__ __forceinline__ int dact_fragments(int d_h) { return (d_h + GradTile::ROWS - 1) / GradTile::ROWS * (GradTile::ROWS / FRAGMENT_ROWS); }
__device__ __forceinline__ long fragment_at(long step, int fragments, int fragment, int piece)
{
    return ((step * fragments + fragment) * 3 + piece) * FRAGMENT_BYTES;
}

// row j of N neighbouring samples from b on (b a multiple of N)
template <int N>
__device__ __forceinline__ void store_pieces(const float (&v)[N], int b, int j, int fragments, unsigned char *__restrict__ pieces)
{
    typedef __attribute__((ext_vector_type(N > 1 ? N / 2 : 1))) unsigned Pairs;
    Pairs p[3];
#pragma unroll
    for (int n = 0; n < N; n += 2) {
        unsigned h, m, l;
        split3_pair_nearest(v[n], n + 1 < N ? v[n + 1 < N ? n + 1 : 0] : 0.f, h, m, l);
        p[0][n / 2] = h, p[1][n / 2] = m, p[2][n / 2] = l;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        unsigned char *to = pieces + fragment_at(b / GradTile::STEP, fragments, j / FRAGMENT_ROWS, i) +
                            (b % GradTile::STEP / 8 * FRAGMENT_ROWS + j % FRAGMENT_ROWS) * 16 + b % 8 * 2;
        if constexpr (N > 1)
            *(Pairs *)to = p[i];
        else
            *(unsigned short *)to = (unsigned short)p[i][0];
    }
}

// ---- 2. the samples, NS per workgroup (head_tail.h) ---------------------------------------
// LDS: a[NS][lda] | z[NS][K] | dz[NS][K]
constexpr int DACT_ROWS = 20;  // rows of W2 in flight per thread

template <TailRow ROW, int NS, bool PIECES>
__global__ __launch_bounds__(TAIL_THREADS) void train_sample_kernel(
    const float *__restrict__ act_part, int nks, int B, int d_h, int K, const float *__restrict__ b1,
    const float *__restrict__ w2, const float *__restrict__ b2, const float *__restrict__ centers,
    const int32_t *__restrict__ bin, const float *__restrict__ y, const int32_t *__restrict__ steps, int n_seqs,
    float lambda, float *__restrict__ act, float *__restrict__ dact, float *__restrict__ dz_out,
    float *__restrict__ loss_part, unsigned char *__restrict__ pieces)
{
    __shared__ float4 join[tail_joins<ROW, NS>];
    extern __shared__ __align__(16) float a[];
    // (with pieces, the workgroups that share their 16 bytes, eight samples', run on one XCD, i % 8, whose L2 puts the lines together:
    // 256 samples, d_h = 1024: 12.8 us where each sample of the eight is another XCD's, 10.8; without pieces 9.8)
    int b0 = blockIdx.x * NS;
    if (PIECES) {
        constexpr int SHARE = 8 / NS;
        const int x = blockIdx.x & 7, i = blockIdx.x >> 3;
        b0 = (i / SHARE * 8 + x) * 8 + i % SHARE * NS;
        if (b0 >= (B + GradTile::STEP - 1) / GradTile::STEP * GradTile::STEP)
            return;
    }
    const int lda = tail_row(d_h);
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
    // (with pieces: the zeros behind a row as well)
    const int fragments = dact_fragments(d_h), end = PIECES ? fragments * FRAGMENT_ROWS : d_h;
#pragma unroll 1
    for (int j = j0; j < end; j += TAIL_THREADS) {
        const bool unit = !PIECES || j < d_h;
        const int at = PIECES ? min(j, d_h - 1) : j;
        float s[PER] = {};
#pragma unroll 1
        for (int o0 = 0; o0 < K; o0 += DACT_ROWS) {
            if (j != j0 || o0 > 0)
                load_rows(o0, at);
#pragma unroll
            for (int o = 0; o < DACT_ROWS; ++o)
                if (o0 + o < K)
#pragma unroll
                    for (int n = 0; n < PER; ++n)
                        s[n] = fmaf(dz[(n0 + n) * K + o0 + o], w[o], s[n]);
        }
#pragma unroll
        for (int n = 0; n < PER; ++n) {
            const bool in = unit && b0 + n0 + n < B;
            s[n] = in && a[(n0 + n) * lda + hidden_place(at, d_h)] > 0.f ? s[n] : 0.f;
            if (in)
                dact[(long)(b0 + n0 + n) * d_h + j] = s[n];
        }
        if constexpr (PIECES)
            store_pieces(s, b0 + n0, j, fragments, pieces);
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
// Chains of cache latencies beside the tiles of W1: a workgroup's four waves share the samples, keep whole batches of loads in
// flight and join their sums in a fixed order.  Beside W1's gradient on the fp32 instructions they use FMAs and few registers, so that
// more workgroups of the W1 part, a stream there, stay on a compute unit; beside its gradient of bf16 pieces, which has the registers,
// the fp32 matrix instructions, behind the tiles: 1024 samples, d = 4096, d_h = 1024, 20 bins, 98 workgroups on FMAs ahead of the tiles
// took 20 us of a launch of 66, holding back as many tiles; 82 of them 14 us, beside the last tiles.
struct Params {
    float *w, *m, *v, *g;
};

__device__ __forceinline__ void update_one(const Adam &h, const Params &p, long e, float g)
{
    float w = p.w[e], m = p.m[e], v = p.v[e];
    adamw(h, g, w, m, v);
    p.w[e] = w;
    p.m[e] = m;
    p.v[e] = v;
    if (p.g)
        p.g[e] = g;
}

// Workgroup = 64 columns; wave q adds the samples b = q, q + 4, ... (each a coalesced load of 64 columns, SAMPLES_AHEAD in flight).
// NO > 0: the column is weighted with dz[b][o0 .. o0 + NO - 1] (rows of W2's gradient; a load of act serves all of
// them); NO = 0: a plain column sum (the biases).  Parameter (o, column) sits at base + o * ld + column.
constexpr int W2_ROWS = 4;  // rows of W2 per workgroup
constexpr int SAMPLES_AHEAD = 32;

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
        update_one(h, p, NO > 0 ? (o0 + r) * ld + col : col, g);
    }
}

// Beside the gradient of pieces.  W2: gradient[o][j] = sum over samples of dz[b][o] act[b][j], 32 rows o x 16 columns j a workgroup, on the fp32 matrix
// instructions (16x16x4; a chain of FMAs' precision).  Wave q takes the samples 16 s + 4 q + 0 .. 3 of step s; lane l holds row and
// column l % 16 of sample l / 16.  Rows past K and columns past d_h are others', computed and dropped.  `red`: 4 x 32 x 16 floats.
constexpr int W2_TILE_ROWS = 32, W2_TILE_COLS = 16, W2_AHEAD = 16;

__device__ __forceinline__ void w2_update(const float *__restrict__ act, const float *__restrict__ dz, int B, int d_h, int K, int col0,
                                          int o0, const Adam &h, const Params &p, float *__restrict__ red)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    const int tid = threadIdx.x, l15 = tid & 15, kq = tid >> 4 & 3, q = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sample = 4 * q + kq, steps = (B + 15) / 16;
    const float *pa = act + (long)min(sample, B - 1) * d_h + min(col0 + l15, d_h - 1);
    const float *pz = dz + (long)min(sample, B - 1) * K;
    const int row[2] = {min(o0 + l15, K - 1), min(o0 + 16 + l15, K - 1)};
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    struct Batch {
        float z[W2_AHEAD][2], a[W2_AHEAD];
    } now, next;
    auto load = [&](Batch &t, int s0) {
#pragma unroll
        for (int s = 0; s < W2_AHEAD; ++s) {
            t.a[s] = *pa, t.z[s][0] = pz[row[0]], t.z[s][1] = pz[row[1]];
            const bool more = 16 * (s0 + s + 1) + sample < B;  // past the end: the last sample, zeros of it
            pa += more ? 16L * d_h : 0, pz += more ? 16L * K : 0;
        }
    };
    load(now, 0);
#pragma unroll 1
    for (int s0 = 0; s0 < steps; s0 += W2_AHEAD) {
        if (s0 + W2_AHEAD < steps)
            load(next, s0 + W2_AHEAD);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < W2_AHEAD; ++s) {
            const bool in = 16 * (s0 + s) + sample < B;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? now.z[s][i] : 0.f, in ? now.a[s] : 0.f, acc[i], 0, 0, 0);
        }
        now = next;
    }
    constexpr int TILE = W2_TILE_ROWS * W2_TILE_COLS;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            red[q * TILE + (16 * i + 4 * kq + e) * W2_TILE_COLS + l15] = acc[i][e];
    __syncthreads();
#pragma unroll
    for (int e = tid; e < TILE; e += 256) {
        const int o = o0 + e / W2_TILE_COLS, j = col0 + e % W2_TILE_COLS;
        if (o >= K || j >= d_h)
            continue;
        const float g = ((red[e] + red[TILE + e]) + red[2 * TILE + e]) + red[3 * TILE + e];
        update_one(h, p, (long)o * d_h + j, g);
    }
}

// b1, b2: sums over the samples of columns of dact, dz: 64 columns (16 chunks of four, head_tail.h) a workgroup, lane l the samples
// 16 s + l / 16 of every step.  `red`: 16 x 64 floats.
constexpr int BIAS_COLS = 64, BIAS_AHEAD = 16;

template <bool TINY>
__device__ __forceinline__ void bias_update_of(const float *__restrict__ mat, int n, int col0, int B, const Adam &h, const Params &p,
                                            float *__restrict__ red)
{
    const int tid = threadIdx.x, l15 = tid & 15, sub = tid >> 4;
    const RowChunk<TINY> c(min(col0 / 4 + l15, (n - 1) / 4), n);  // chunks past the end are computed and dropped
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int s0 = sub; s0 < B; s0 += 16 * BIAS_AHEAD) {
        ChunkOf<float> v[BIAS_AHEAD];
#pragma unroll
        for (int s = 0; s < BIAS_AHEAD; ++s)  // past the end: the last sample, not used
            v[s] = load_chunk(mat + (long)min(s0 + 16 * s, B - 1) * n, c, n);
#pragma unroll
        for (int s = 0; s < BIAS_AHEAD; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                sum[e] += s0 + 16 * s < B ? v[s][e] : 0.f;
    }
    *(float4 *)(red + sub * BIAS_COLS + 4 * l15) = make_float4(sum[0], sum[1], sum[2], sum[3]);
    __syncthreads();
    const int j = col0 + tid;
    if (tid >= BIAS_COLS || j >= n)
        return;
    const float *r = red + hidden_place(j, n) - col0;
    float g = r[0];
#pragma unroll
    for (int k = 1; k < 16; ++k)
        g += r[k * BIAS_COLS];
    update_one(h, p, j, g);
}

__device__ __forceinline__ void bias_update(const float *__restrict__ mat, int n, int col0, int B, const Adam &h, const Params &p,
                                            float *__restrict__ red)
{
    if (n < 4)
        bias_update_of<true>(mat, n, col0, B, h, p, red);
    else
        bias_update_of<false>(mat, n, col0, B, h, p, red);
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
// rows of its own, two workgroups per compute unit.  The contraction runs over the samples, the slow index of x, of which a fragment
// wants eight in a lane: a lane loads four neighbouring k of two samples, a pair of K elements for each of four fragments, so that column c
// of fragment b is k = 4 c + b, and ends up with four neighbouring k of a row j, one 16-byte access each to W1 and the moments.
// dact comes as fragments of pieces from the samples' kernel: split here, by the 64 workgroups of d = 4096 that share a row, it was
// 88 of a step's 147 vector instructions a wave, and an MFMA 16x16x32 leaves a SIMD's issue to two others only (8 of its 16 cycles, measured in
// registers: with two vector instructions behind each MFMA a wave takes 16 cycles, with three 20, with six 32).
// Bound: loads and the 6 x 2 d d_h products a sample beside each other (33000 cycles of a wave's loop of 48000 with its loads taken out),
// at 2.0 GHz; then the stream of the parameters, 8 us.
// Whole steps, us: 1024 samples, d = 4096, d_h = 1024 128.5 -> 121.8; 512 77.6 -> 75.4; d = 1024, d_h = 384, 1024 samples 60.8 -> 53.8.  Tiles of 128 x 128, one
// workgroup to a compute unit: 116 -> 125.
// From SPLIT_SAMPLES samples on where the tiles are more than SPLIT_TILES, half a round of the compute units, elsewhere from
// SPLIT_SAMPLES_FEW_TILES.  Whole steps, us, fp32 instructions / pieces:
//   512 tiles (d = 4096, d_h = 1024)   128 samples 45.1 / 46.6   160 54.8 / 53.8   192 59.1 / 56.8   384 78.5 / 65.7   1024 162 / 113
//   144 tiles (d = 1024, d_h = 1100)   128 samples 35.6 / 35.7   160 37.5 / 36.6   256 43.4 / 39.7   512 62.3 / 51.8
//   128 tiles (d = 1024, d_h = 1024)   192 samples 33.3 / 33.6   256 34.8 / 34.2   384 43.5 / 42.2   1024 67.6 / 58.8
//   128 tiles (d = 2048, d_h = 512)    192 samples 32.6 / 33.6   256 36.2 / 35.5   384 43.6 / 42.2
//    48 tiles (d = 1024, d_h = 384)    192 samples 25.4 / 26.1   256 28.2 / 28.4   384 36.0 / 35.9   1024 59.6 / 53.8
//    16 tiles (d = 512, d_h = 256)     192 samples 22.4 / 22.7   256 24.3 / 24.2   384 30.2 / 28.7   1024 52.3 / 47.9
constexpr int SPLIT_SAMPLES = 160, SPLIT_SAMPLES_FEW_TILES = 256, SPLIT_TILES = 128;

struct GradSource {
    static constexpr int ROW_PIECES = 3, ROW_LOADS = 0, COL_LOADS = 2, COL_WRITES = 12;
    static constexpr bool ROWS_READY = true, ROWS_TURN = false;
    struct Rows {};
    struct Cols {
        float4 v[2];
    };
    const unsigned char *pieces;  // this wave's first fragment
    const float *x;
    unsigned lane_at, col_at[2];  // this lane's bytes of a fragment; of the columns, its two samples of the wave's eight
    long x_bytes, step_bytes, d;
    int steps, wave;

    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t from(const void *p, int bytes)
    {
        return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, bytes, 0x00020000);
    }
    // (steps that are only asked for: the last one again)
    __device__ __forceinline__ split_u32x4 load_rows(int i, int piece, int a) const
    {
        return __builtin_bit_cast(split_u32x4, __builtin_amdgcn_raw_buffer_load_b128(from(pieces + min(i, steps - 1) * step_bytes, 6 * FRAGMENT_BYTES),
                                                                                     lane_at, (a * 3 + piece) * FRAGMENT_BYTES, 0));
    }
    // Samples past the batch lie past the end of x: the hardware makes zeros of them.
    __device__ __forceinline__ void load_cols(int i, int l, Cols &r) const
    {
        const long at = (long)(i * GradTile::STEP + 8 * wave) * d * 4, left = x_bytes - at;
        const int bytes = left < 0 ? 0 : (int)min(left, 0x7fffffffL);
        r.v[l] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(from((const unsigned char *)x + at, bytes), col_at[l], 0, 0));
    }
    __device__ __forceinline__ void clear_rows(int, Rows &) const {}
    __device__ __forceinline__ void clear_cols(int, Cols &) const {}
    // a pair is what a lane loads of a column
    __device__ __forceinline__ float col_value(const Cols &r, int, int e) const { return (&r.v[e % 2].x)[e / 2]; }
    __device__ __forceinline__ void write_col(unsigned char *buf, const split_u32x4 (&part)[1][3], int n) const
    {
        const int lane = threadIdx.x & 63;
        *(unsigned *)(buf + n % 3 * GradTile::PIECE + n / 3 * 1024 + (wave * 16 + (lane & 15)) * 16 + (lane >> 4) * 4) = part[0][n % 3][n / 3];
    }
    __device__ __forceinline__ int slot() const { return threadIdx.x & 63; }
};

__device__ __forceinline__ void w1_update_split(int tile_k, int tile_j, const float *__restrict__ x,
                                                const float *__restrict__ dact, const unsigned char *__restrict__ pieces, int B, int d,
                                                int d_h, const Adam &h, float *__restrict__ w1, float *__restrict__ m_w1,
                                                float *__restrict__ v_w1, float *__restrict__ g_w1, unsigned char *__restrict__ lds)
{
    using S = GradTile;
    constexpr int FA = S::FA, FB = S::FB;
    static_assert(FB == 4 && S::SHARE == 1, "four neighbouring k to a lane");
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k0 = tile_k * S::COLS, j0 = tile_j * S::ROWS + 16 * FA * wave;

    // d is a multiple of 4: columns that do not exist are others', computed and dropped
    const int steps = (B + S::STEP - 1) / S::STEP;
    GradSource src;
    src.d = d, src.wave = wave, src.steps = steps, src.x = x, src.x_bytes = (long)B * d * 4;
    src.step_bytes = fragment_at(1, dact_fragments(d_h), 0, 0);
    src.pieces = pieces + fragment_at(0, 0, j0 / FRAGMENT_ROWS, 0), src.lane_at = (tid & 63) * 16;
#pragma unroll
    for (int l = 0; l < 2; ++l)
        src.col_at[l] = (unsigned)((2 * (tid >> 4 & 3) + l) * d + min(k0 + 4 * (tid & 15), d - 4)) * 4;
    split_f32x4 acc[FA][FB];
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int b = 0; b < FB; ++b)
            acc[a][b] = split_f32x4{0.f, 0.f, 0.f, 0.f};
    __builtin_assume(steps >= SPLIT_SAMPLES / S::STEP);
    split_contract<S>(lds, steps, acc, src);
    int again = tid;  // the lane's place, not held over the contraction (two registers that it does not have)
    asm("" : "+v"(again));
    const int l15 = again & 15, kq = again >> 4 & 3;
    const int k_at = min(k0 + 4 * l15, d - 4);
    if (__builtin_expect(!all_finite(acc), 0))
        redo_not_finite(B, acc, [&](int i, float (&av)[FA][4], float (&bv)[FB][4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int b = 16 * i + 4 * kq + e, sample = min(b, B - 1);
                const float4 xv = *(const float4 *)(x + (long)sample * d + k_at);
#pragma unroll
                for (int a = 0; a < FA; ++a) {
                    const float dv = dact[(long)sample * d_h + min(j0 + 16 * a + l15, d_h - 1)];
                    av[a][e] = b < B ? dv : 0.f;
                }
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
            const long at = (long)min(j0 + 16 * a + 4 * kq + i, d_h - 1) * d + k;
            w[a][i] = *(const float4 *)(w1 + at);
            m[a][i] = *(const float4 *)(m_w1 + at);
            v[a][i] = *(const float4 *)(v_w1 + at);
        }
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = j0 + 16 * a + 4 * kq + i;
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
    const unsigned char *pieces;  // of dact, for the tiles of bf16 pieces
    int B, d, d_h, K;
    int tiles_k, tiles_w1;
    int cols_w2, blocks_w2, blocks_b1, blocks_b2;  // tiles of a row of W2; workgroups of W2 and of the biases
    float lambda;
    Params w1, w2, b2, b1;
    float *loss;
};

template <bool SPLIT>
__global__ __launch_bounds__(256, SPLIT ? 2 : 1) void train_update_kernel(UpdateArgs a, Adam h)
{
    constexpr int LDS_FLOATS = SPLIT ? GradTile::LDS_BYTES / 4 : 2 * GRAD_STAGE_FLOATS;
    __shared__ __align__(16) float lds[LDS_FLOATS];
    static_assert(LDS_FLOATS >= 4 * W2_ROWS * 64 && LDS_FLOATS >= 4 * W2_TILE_ROWS * W2_TILE_COLS && LDS_FLOATS >= 16 * BIAS_COLS,
                  "LDS of the small-parameter part");
    int id = blockIdx.x;
    if (id < a.tiles_w1) {
        const int tk = id % a.tiles_k, tj = id / a.tiles_k;
        if constexpr (SPLIT)
            w1_update_split(tk, tj, a.x, a.dact, a.pieces, a.B, a.d, a.d_h, h, a.w1.w, a.w1.m, a.w1.v, a.w1.g, (unsigned char *)lds);
        else
            w1_update(tk, tj, a.x, a.dact, a.B, a.d, a.d_h, h, a.w1.w, a.w1.m, a.w1.v, a.w1.g, lds);
        return;
    }
    id -= a.tiles_w1;
    if (id < a.blocks_w2) {
        if constexpr (SPLIT)
            w2_update(a.act, a.dz, a.B, a.d_h, a.K, id % a.cols_w2 * W2_TILE_COLS, id / a.cols_w2 * W2_TILE_ROWS, h, a.w2, lds);
        else
            column_update<W2_ROWS>(a.act, a.d_h, a.d_h, (id % a.cols_w2) * 64, a.dz, a.K, (id / a.cols_w2) * W2_ROWS, a.B, h, a.w2, lds);
        return;
    }
    id -= a.blocks_w2;
    if (id < a.blocks_b1) {
        if constexpr (SPLIT)
            bias_update(a.dact, a.d_h, id * BIAS_COLS, a.B, h, a.b1, lds);
        else
            column_update<0>(a.dact, a.d_h, a.d_h, id * BIAS_COLS, nullptr, 0, 0, a.B, h, a.b1, lds);
        return;
    }
    id -= a.blocks_b1;
    if (id < a.blocks_b2) {
        if constexpr (SPLIT)
            bias_update(a.dz, a.K, id * BIAS_COLS, a.B, h, a.b2, lds);
        else
            column_update<0>(a.dz, a.K, a.K, id * BIAS_COLS, nullptr, 0, 0, a.B, h, a.b2, lds);
    } else
        sum_loss(a.loss_part, a.B, a.lambda, a.loss);
}

}  // namespace

template <TailRow ROW, int NS, bool PIECES>
static hipError_t launch_samples(const TrainArgs &a, int nks, size_t lds, hipStream_t st)
{
    static DeviceMask raised{0};
    hipError_t e = raise_dynamic_lds_limit((const void *)train_sample_kernel<ROW, NS, PIECES>, (int)TAIL_LDS_LIMIT, raised);
    if (e != hipSuccess)
        return e;
    // (with pieces: whole steps of samples, dealt to the XCDs in eights)
    constexpr int EIGHTS = 8 * 8;
    const int wgs = PIECES ? (a.B + EIGHTS - 1) / EIGHTS * (EIGHTS / NS) : (a.B - 1) / NS + 1;
    hipLaunchKernelGGL((train_sample_kernel<ROW, NS, PIECES>), dim3(wgs), dim3(TAIL_THREADS), NS * lds, st, a.act_part,
                       nks, a.B, a.d_h, a.K, a.b1, a.w2, a.b2, a.centers, a.bin, a.y, a.steps, a.n_seqs, a.lambda, a.act,
                       a.dact, a.dz, a.loss_part, a.dact_pieces);
    return hipGetLastError();
}

static hipError_t launch_samples(const TrainArgs &a, int nks, size_t lds, bool split, hipStream_t st)
{
    return tail_launch(a.d_h, tail_sequences(a.B, lds), [&](auto row, auto ns) {
        return split ? launch_samples<decltype(row)::value, decltype(ns)::value, true>(a, nks, lds, st)
                     : launch_samples<decltype(row)::value, decltype(ns)::value, false>(a, nks, lds, st);
    });
}

// (a lane's offset among the eight samples of a wave, up to 32 d bytes, and its 16 bytes lie inside a descriptor of 2^31 - 1 bytes:
// GradSource::load_cols)
static bool gradient_splits(int32_t B, int d, int d_h)
{
    const long tiles = (long)((d_h + GradTile::ROWS - 1) / GradTile::ROWS) * ((d + GradTile::COLS - 1) / GradTile::COLS);
    return B >= (tiles > SPLIT_TILES ? SPLIT_SAMPLES : SPLIT_SAMPLES_FEW_TILES) && d < (1 << 26);
}

size_t train_pieces_bytes(int32_t B, int d, int d_h)
{
    return gradient_splits(B, d, d_h) ? (size_t)((B + GradTile::STEP - 1) / GradTile::STEP) * dact_fragments(d_h) * 3 * FRAGMENT_BYTES : 0;
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
    const bool split = gradient_splits(a.B, a.d, a.d_h);
    e = launch_samples(a, head_k_splits(a.d, a.d_h, a.B, DT_F32), lds, split, st);
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
    // the first of the two below the value: their products with an infinite moment add up to infinity
    auto two_floats = [](double value, float &most, float &rest) {
        most = (float)value;
        if ((double)most >= value)
            most = nextafterf(most, 0.f);
        rest = (float)(value - (double)most);
    };
    const double step = (double)a.lr / (double)a.corr1;
    two_floats(step, h.step, h.step_rest);
    two_floats(1.0 / (double)a.corr2, h.inv_corr2, h.inv_corr2_rest);
    h.decay = (float)((double)a.lr * (double)a.weight_decay);
    h.quick = a.eps >= QUICK_EPS && a.eps <= QUICK_MOST && step <= (double)QUICK_MOST;
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
    u.pieces = a.dact_pieces;
    const int tile_j = split ? GradTile::ROWS : GM, tile_k = split ? GradTile::COLS : GN;
    const long tiles_k = (a.d + tile_k - 1) / tile_k, tiles_j = (a.d_h + tile_j - 1) / tile_j;
    u.tiles_k = (int)tiles_k;
    u.tiles_w1 = (int)(tiles_k * tiles_j);
    const int w2_cols = split ? W2_TILE_COLS : 64, w2_rows = split ? W2_TILE_ROWS : W2_ROWS;
    u.cols_w2 = (a.d_h + w2_cols - 1) / w2_cols;
    u.blocks_w2 = u.cols_w2 * ((a.K + w2_rows - 1) / w2_rows);
    u.blocks_b1 = (a.d_h + BIAS_COLS - 1) / BIAS_COLS;
    u.blocks_b2 = (a.K + BIAS_COLS - 1) / BIAS_COLS;
    const long wgs = tiles_k * tiles_j + u.blocks_w2 + u.blocks_b1 + u.blocks_b2 + 1;
    if (wgs > 0x7fffffffL)
        return hipErrorInvalidValue;
    if (split)
        hipLaunchKernelGGL(train_update_kernel<true>, dim3((unsigned)wgs), dim3(256), 0, st, u, h);
    else
        hipLaunchKernelGGL(train_update_kernel<false>, dim3((unsigned)wgs), dim3(256), 0, st, u, h);
    return hipGetLastError();
}

}  // namespace egtp
