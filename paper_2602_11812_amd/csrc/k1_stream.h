// Pieces shared by the three fused entropy kernels (Eq. 2): loads from memory straight into the LDS ring, the
// matching wait, and the fold of a tile's logits into a token's streaming statistics.  Device-side header.
#pragma once
#include "k1_common.h"

namespace egtp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

namespace {

// Pacing: workgroup i is placed on XCD i % 8; a cohort are the workgroups one XCD runs at a time (its compute units)
constexpr int COHORT = 32;
constexpr int PACE_SPINS = 24;     // bound of one wait: polls of the counter ...
constexpr int PACE_SLEEP = 4;      // ... each followed by a sleep of 64 * PACE_SLEEP cycles

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt in bits
// [3:0] and [15:14], export and LDS/scalar counters left at their maxima)
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// 16 bytes per lane from memory straight into LDS: lane i of the wave lands at lds_wave_base + 16 * i.
// A buffer load (descriptor + per-lane byte offset + scalar byte offset): the address of a K step is then one
// scalar add, with no 64-bit vector arithmetic in the main loop, and the hardware clamps every access to the
// descriptor's range.  Measured against the flat-address form of the same load: 0.5 % faster.
// STREAM: with the non-temporal hint, for data that is read once and does not fit the caches.
template <bool STREAM = false>
__device__ __forceinline__ void load16_to_lds(__amdgpu_buffer_rsrc_t rsrc, int lane_byte_offset, int scalar_byte_offset,
                                              unsigned char *lds_wave_base)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)lds_wave_base, 16,
                                             lane_byte_offset, scalar_byte_offset, 0, STREAM ? 2 : 0);
}
// raw buffer descriptor over `bytes` bytes at p (gfx9 family: 32-bit data format word, no swizzle)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const unsigned char *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, bytes, 0x00020000);
}

// Hidden states read where they are (row-major bf16, rows of 2 d bytes), two K steps at a time: 128 bytes of a row, a whole line, where the
// 64 of one step would ask for every line twice.  In the LDS a row of two steps has eight places of 16 bytes, keyed by the row so
// that the fragment reads meet all banks; a wave-wide load fills eight rows.  Rows past the batch lie past the descriptor, and K elements past d are
// given an offset that does: the hardware makes zeros of both, and asks no memory for them.
struct DirectRows {
    int at, chunk;  // this lane's bytes of the first eight rows of its wave: from the block's begin, and inside a row
    __device__ __forceinline__ DirectRows(int wave, int lane, int d) : chunk(((lane & 7) ^ (lane >> 3)) << 4) { at = (wave * 8 + (lane >> 3)) * 2 * d + chunk; }
    // load number q (32 rows each) of the pair of steps that begins with kt
    __device__ __forceinline__ int offset(int q, int kt, int d) const
    {
        return chunk < 2 * d - kt * ROW_BYTES ? at + q * 64 * d : (int)0x80000000;
    }
    // K step that the workgroups of vocabulary range `range` begin at (in turn to the last one, then from 0 on): where rows are a multiple
    // of 4 KiB apart, a step's lines lie in one channel of the L2 or a few, and all workgroups would be at the same step.
    static __device__ __forceinline__ int first_step(int range, int KT) { return (int)((unsigned)range * 4u % (unsigned)KT); }
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t block(const unsigned char *hidden, long tok0, int tokens, long T, int d)
    {
        return raw_buffer(hidden + tok0 * 2 * d, (int)min((long)tokens, T - tok0) * 2 * d);
    }
    // this lane's 16 bytes of a fragment of 16 rows, even step; odd: ^ ODD
    static __device__ __forceinline__ unsigned fragment(int lane) { return (lane & 15) * 2 * ROW_BYTES + (((lane >> 4) ^ (lane & 7)) << 4); }
    static constexpr unsigned ODD = 64;
};

// Fold N logits of one token: zin[4*q+i] is vocabulary row row0 + 16*q + i.  MASK: rows from V on do not exist.
// Whether a lane has any row at all follows from the row numbers: its maximum cannot tell, fmaxf passes over NaN.
template <bool MASK, int N>
__device__ __forceinline__ void fold(const float (&zin)[N], Stats &st, int row0, int V)
{
    if (MASK && row0 >= V)
        return;  // nothing to add (and perhaps no reference maximum yet)
    float z[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        float v = zin[i];
        if (MASK)
            v = (row0 + 16 * (i >> 2) + (i & 3)) < V ? v : NEG_BIG;
        z[i] = v;
    }
    float mx = z[0];
#pragma unroll
    for (int i = 1; i < N; ++i)
        mx = fmaxf(mx, z[i]);
    // The reference lives in log2 units, r = fl(max z * log2 e): every exponent is then ONE fused
    // multiply-add z * log2 e - r (exact product, one rounding of a small result) and re-referencing is an
    // exact difference of two r, so the precision does not degrade with the magnitude of the logits.
    const float r = mx * LOG2E;
    if (r > st.m) {  // new running reference: rescale what has been summed so far
        float dl = st.m - r;
        float sc = fast_exp2(dl);
        st.U = (st.U + dl * st.S) * sc;
        st.S = st.S * sc;
        st.m = r;
    }
    const float mc = -st.m;
    float S0 = 0.f, S1 = 0.f, U0 = 0.f, U1 = 0.f;
#pragma unroll
    for (int i = 0; i < N; i += 2) {
        float t0 = fmaf(z[i], LOG2E, mc);
        float t1 = fmaf(z[i + 1], LOG2E, mc);
        float e0 = fast_exp2(t0);
        float e1 = fast_exp2(t1);
        S0 += e0;
        S1 += e1;
        U0 = fmaf(e0, t0, U0);
        U1 = fmaf(e1, t1, U1);
    }
    st.S += S0 + S1;
    st.U += U0 + U1;
}

}  // namespace
}  // namespace egtp
