// Bodies of the V quantizer (Section 4.3: psi_V per channel; Section 3.2 gives the per-channel quantizer) --
// HBM-bound.  They take their workgroup coordinates as arguments, so that they can share launches with the K side
// (sage_prepass.hip) or have their own (sage_prepass_v.hip).
//
//   per-channel absolute maximum over all tokens of a (batch, head) slab  -> delta_V[c] = amax / 127
//   V^[t,c] = clamp(rne(V[t,c] * fl32(127 / amax_c)), -127, 127)          -> stored TRANSPOSED,
//   channel-major [D][Np] with Np = 64 * ceil(N / 64), tokens past N as code 0
//
// Channel-major is what the attention kernel wants: the A operand of the INT8 matrix instruction
// of O^T = V^^T P^^T is 16 consecutive TOKENS of one channel, i.e. one 16-byte read of a row of V^^T.
// Maxima are taken on fp16 pairs and pass over NaN, so that a token that holds one leaves the other tokens' codes as
// they are; they do not depend on how the tokens are split.
#pragma once
#include "sage_device.h"

namespace sage {

struct Max8 {          // maxima of 8 channels
    half2v m[4] = {};
    __device__ __forceinline__ void take(const half8& x) {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        const u4 w = __builtin_bit_cast(u4, x);
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] = max_abs(m[e], w[e]);
    }
    // over the lanes VPR, 2 VPR, ... apart, which hold the same channels of other rows
    template <int VPR> __device__ __forceinline__ void fold() {
#pragma unroll
        for (int off = VPR; off < 64; off <<= 1)
#pragma unroll
            for (int e = 0; e < 4; ++e) m[e] = max_abs(m[e], (unsigned)__shfl_xor(__builtin_bit_cast(int, m[e]), off, 64));
    }
};

// Per-channel maxima of the rows row_begin .. row_end - 1 of a slab, as fp16 patterns (no NaN among them: they order like
// their bits); thread c < D returns channel c's.
// s_part: NT / 64 rows of D patterns.
template <int D, int NT>
__device__ __forceinline__ unsigned short v_absmax_rows(const _Float16* __restrict__ base, int row_begin, int row_end,
                                                        unsigned short (*s_part)[D]) {
    constexpr int VPR = D / 8, RG = NT / VPR, BATCH = 16;
    const int t = threadIdx.x, c8 = t % VPR, rg = t / VPR;
    Max8 m;
    for (int r0 = row_begin; r0 < row_end; r0 += BATCH * RG) {
        // all loads of a batch are issued before the first is used; a row past the end is fetched from
        // the last row instead, which leaves the maximum unchanged
        half8 x[BATCH];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            const int r = r0 + rg + i * RG;
            x[i] = *(const half8*)(base + (size_t)(r < row_end ? r : row_end - 1) * D + c8 * 8);
        }
        __builtin_amdgcn_sched_barrier(0);       // the fence that keeps the compiler from sinking each load to its use
#pragma unroll
        for (int i = 0; i < BATCH; ++i) m.take(x[i]);
    }
    m.fold<VPR>();
    if ((t & 63) < VPR) {
#pragma unroll
        for (int e = 0; e < 4; ++e) *(half2v*)&s_part[t >> 6][c8 * 8 + 2 * e] = m.m[e];
    }
    __syncthreads();
    unsigned short most = 0;
    if (t < D) {
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) most = s_part[w][t] > most ? s_part[w][t] : most;
    }
    return most;
}

__device__ __forceinline__ float f16_pattern(unsigned short p) { return (float)__builtin_bit_cast(_Float16, p); }

// Codes of 4 consecutive tokens of 8 channels, into the transposed tile tr (rows of PITCH bytes): the four codes of a
// channel leave as one 32-bit LDS store.  Rows of the tile are padded by one word, which spreads those stores over the banks.
template <int PITCH>
__device__ __forceinline__ void v_codes4x8(int8_t* tr, int c0, int token, const half8 (&x)[4], const float (&r)[8], int live) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float f[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = i < live ? (float)x[i][e] : 0.0f;
        *(unsigned*)(tr + (c0 + e) * PITCH + token) = quantize4(f[0], f[1], f[2], f[3], r[e]);
    }
}

// Quantizes tiles of ROWS = 128 tokens (tile tile0, tile0 + stride, ...) of a slab and writes them transposed, whole
// 128-byte lines of a channel row.  amax: P sets of D maxima (fp32 bits) to take the largest of; the workgroup of tile 0
// writes the scales.
template <int D, int NT>
__device__ __forceinline__ void v_transpose_body(const _Float16* __restrict__ v, const unsigned* __restrict__ amax, int P,
                                                 int8_t* __restrict__ vt, float* __restrict__ vscale, int N, int Np,
                                                 int tile0, int stride, int bh) {
    constexpr int VPR = D / 8, G = NT / VPR, ROWS = 128, PITCH = ROWS + 4, SETS = ROWS / (4 * G);
    static_assert(SETS >= 1, "a thread owns whole groups of 4 tokens");
    const int t = threadIdx.x, c8 = t % VPR, g = t / VPR;
    const _Float16* base = v + ((size_t)bh * N) * D + c8 * 8;
    __shared__ __attribute__((aligned(16))) int8_t tr[D * PITCH];
    __shared__ __attribute__((aligned(16))) float s_r[D];
    half8 x[SETS][4];
    auto fetch = [&](int tile) {
#pragma unroll
        for (int s = 0; s < SETS; ++s)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = tile * ROWS + 4 * (g + s * G) + i;
                x[s][i] = *(const half8*)(base + (size_t)(row < N ? row : N - 1) * D);      // (past the end: code 0 below)
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(tile0);              // in flight while the maxima are collected
    if (t < D) {
        unsigned most = 0u;
#pragma unroll 8
        for (int p = 0; p < P; ++p) {
            const unsigned b = amax[((size_t)bh * P + p) * D + t];
            most = b > most ? b : most;
        }
        const float a = __uint_as_float(most);
        s_r[t] = a > 0.0f ? 127.0f / a : 0.0f;
        if (tile0 == 0) vscale[(size_t)bh * D + t] = a / 127.0f;
    }
    __syncthreads();
    float r[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = s_r[c8 * 8 + e];
    const int tiles = (Np + ROWS - 1) / ROWS;
    for (int tile = tile0; tile < tiles; tile += stride) {
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const int token = 4 * (g + s * G);
            v_codes4x8<PITCH>(tr, c8 * 8, token, x[s], r, N - (tile * ROWS + token));
        }
        if (tile + stride < tiles) fetch(tile + stride);
        __syncthreads();
        constexpr int CPR = ROWS / 16;          // 16-byte chunks per channel row
        int8_t* out = vt + ((size_t)bh * D) * Np + (size_t)tile * ROWS;
#pragma unroll
        for (int i = 0; i < D * CPR / NT; ++i) {
            const int idx = t + NT * i, c = idx / CPR, part = idx % CPR;
            if (tile * ROWS + part * 16 < Np) {          // the last tile may be half outside
                const unsigned* src = (const unsigned*)(tr + c * PITCH + part * 16);
                *(int4*)(out + (size_t)c * Np + part * 16) = make_int4((int)src[0], (int)src[1], (int)src[2], (int)src[3]);
            }
        }
        if (tile + stride < tiles) __syncthreads();       // the tile is written again
    }
}

// Short sequences (N <= 512): the whole V pre-pass of a slab in one workgroup of 1024 threads; the slab is read once and
// stays in registers (at most 8 rows per thread).
template <int D>
__device__ __forceinline__ void v_small_body(const _Float16* __restrict__ v, int8_t* __restrict__ vt, float* __restrict__ vscale,
                                             int N, int Np, int bh) {
    constexpr int NT = 1024, VPR = D / 8, G = NT / VPR, ROWS = 4 * G, PITCH = ROWS + 4, SETS = 512 / ROWS;
    const int t = threadIdx.x, c8 = t % VPR, g = t / VPR;
    const _Float16* base = v + ((size_t)bh * N) * D + c8 * 8;
    __shared__ __attribute__((aligned(16))) int8_t tr[D * PITCH];
    __shared__ unsigned short s_part[NT / 64][D];
    __shared__ float s_r[D];
    half8 x[SETS][4];
    Max8 m;
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        if (s * ROWS >= N) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = s * ROWS + 4 * g + i;
            x[s][i] = *(const half8*)(base + (size_t)(row < N ? row : N - 1) * D);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        if (s * ROWS >= N) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) m.take(x[s][i]);
    }
    m.fold<VPR>();
    if ((t & 63) < VPR) {
#pragma unroll
        for (int e = 0; e < 4; ++e) *(half2v*)&s_part[t >> 6][c8 * 8 + 2 * e] = m.m[e];
    }
    __syncthreads();
    if (t < D) {
        unsigned short most = 0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) most = s_part[w][t] > most ? s_part[w][t] : most;
        const float a = f16_pattern(most);
        s_r[t] = a > 0.0f ? 127.0f / a : 0.0f;
        vscale[(size_t)bh * D + t] = a / 127.0f;
    }
    __syncthreads();
    float r[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = s_r[c8 * 8 + e];
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        if (s * ROWS >= Np) continue;
        v_codes4x8<PITCH>(tr, c8 * 8, 4 * g, x[s], r, N - (s * ROWS + 4 * g));
        __syncthreads();
        constexpr int CPR = ROWS / 16;
        int8_t* out = vt + ((size_t)bh * D) * Np + (size_t)s * ROWS;
#pragma unroll
        for (int i = 0; i < D * CPR / NT; ++i) {
            const int idx = t + NT * i, c = idx / CPR, part = idx % CPR;
            if (s * ROWS + part * 16 < Np) {
                const unsigned* src = (const unsigned*)(tr + c * PITCH + part * 16);
                *(int4*)(out + (size_t)c * Np + part * 16) = make_int4((int)src[0], (int)src[1], (int)src[2], (int)src[3]);
            }
        }
        if (s + 1 < SETS) __syncthreads();
    }
}

}  // namespace sage
