// Device code shared by the kernels that quantize.
#pragma once
#include <hip/hip_runtime.h>

namespace sage {

// Four INT8 codes round_half_even(clamp(x * rcp)) of Section 3.2, byte i from x[i].  Adding 1.5 * 2^23 rounds
// the (once rounded) product to an integer, ties to even, and leaves it in the low byte of the bit pattern in
// two's complement; a byte permute per pair packs them: 3.75 VALU instructions per code instead of 7 with a
// rounding, a conversion, a mask and a shift.  The same bits as rintf and a conversion: |product| <= 127 after
// the clamp.
__device__ __forceinline__ unsigned quantize4(float x0, float x1, float x2, float x3, float rcp) {
    auto code = [rcp](float x) {
        const float p = __builtin_fminf(__builtin_fmaxf(x * rcp, -127.0f), 127.0f);
        return __builtin_bit_cast(unsigned, p + 12582912.0f);
    };
    const unsigned lo = __builtin_amdgcn_perm(code(x1), code(x0), 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm(code(x3), code(x2), 0x04000c0cu);
    return lo | hi;
}

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

// The fp16 rows of a wavefront's 32 queries quantized where they are used (Section 4.6: the quantizer fused
// into the operator's neighbour): lane l holds half of row l % 32, the channels 32 ks + 16 (l / 32) .. + 15, as the
// INT8 matrix instruction's operand wants them.  amax of a row: both lanes of it; of a block of 32, 64 or 128
// rows: the wavefronts that share the block, through one LDS word each.
// The workgroup's rows start at a multiple of every block size.  Same arithmetic as the pre-pass kernel.
template <int KS>
struct QueryRows {
    half8 raw[KS][2];
    __device__ __forceinline__ void fetch(const _Float16* row, int half, bool live) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                raw[ks][j] = (half8){0, 0, 0, 0, 0, 0, 0, 0};
                if (live) raw[ks][j] = *(const half8*)(row + 32 * ks + 16 * half + 8 * j);
            }
    }
    // largest |x * sm_scale| of the lane's quantization block; every wavefront of the workgroup calls it.
    // red: one float of LDS per wavefront, not used for anything else before the next barrier.
    __device__ __forceinline__ float block_amax(float sm_scale, int shift_q, int wave, float* red) const {
        float m = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) m = __builtin_fmaxf(m, __builtin_fabsf((float)raw[ks][j][e] * sm_scale));
        m = __builtin_fmaxf(m, __shfl_xor(m, 32, 64));
        if (shift_q == 0) return m;
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, off, 64));
        if (shift_q == 5) return m;
        if ((threadIdx.x & 63) == 0) red[wave] = m;
        __syncthreads();
        const int first = shift_q == 6 ? wave & ~1 : wave & ~3;
        m = __builtin_fmaxf(red[first], red[first + 1]);
        if (shift_q == 7) m = __builtin_fmaxf(m, __builtin_fmaxf(red[first + 2], red[first + 3]));
        return m;
    }
    // word i of contraction step ks: channels 4 i .. 4 i + 3 of the lane's 16
    __device__ __forceinline__ unsigned word(int ks, int i, float sm_scale, float rcp) const {
        const half8& h = raw[ks][i >> 1];
        const int e = 4 * (i & 1);
        return quantize4((float)h[e] * sm_scale, (float)h[e + 1] * sm_scale, (float)h[e + 2] * sm_scale, (float)h[e + 3] * sm_scale, rcp);
    }
};

}  // namespace sage
