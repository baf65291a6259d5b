// The V quantizer by itself (sage_quant_v): launches of the bodies in sage_prepass_v.h.
#include "sage_internal.h"
#include "sage_prepass_v.h"

namespace sage {

__global__ void __launch_bounds__(256) zero_words_kernel(unsigned* w, int n) {
    int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) w[i] = 0u;
}

// grid (chunks, BH): the caller's workspace has room for one set of maxima per slab, so the chunks merge there (atomicMax
// on the bits: order-free)
template <int D>
__global__ void __launch_bounds__(256) v_absmax_kernel(const _Float16* __restrict__ v, unsigned* __restrict__ amax_bits, int N, int chunk) {
    __shared__ unsigned short s_part[4][D];
    const int bh = blockIdx.y, begin = blockIdx.x * chunk;
    const unsigned short m = v_absmax_rows<D, 256>(v + ((size_t)bh * N) * D, begin, begin + chunk < N ? begin + chunk : N, s_part);
    if (threadIdx.x < D) atomicMax(amax_bits + (size_t)bh * D + threadIdx.x, __float_as_uint(f16_pattern(m)));
}
template <int D>
__global__ void __launch_bounds__(256) v_quant_transpose_kernel(const _Float16* __restrict__ v, const unsigned* __restrict__ amax_bits,
                                                                int8_t* __restrict__ vt, float* __restrict__ vscale, int N, int Np) {
    v_transpose_body<D, 256>(v, amax_bits, 1, vt, vscale, N, Np, blockIdx.x, gridDim.x, blockIdx.y);
}
template <int D>
__global__ void __launch_bounds__(1024) v_small_kernel(const _Float16* __restrict__ v, int8_t* __restrict__ vt, float* __restrict__ vscale,
                                                       int N, int Np) {
    v_small_body<D>(v, vt, vscale, N, Np, blockIdx.x);
}

template <int D>
static hipError_t launch_quant_v_d(const _Float16* v, int8_t* vt, float* vscale, unsigned* amax_bits, int BH, int N, hipStream_t st) {
    const int n = BH * D, Np = 64 * ((N + 63) / 64);
    if (N <= 512) {
        v_small_kernel<D><<<BH, 1024, 0, st>>>(v, vt, vscale, N, Np);
        return hipGetLastError();
    }
    zero_words_kernel<<<(n + 255) / 256, 256, 0, st>>>(amax_bits, n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int CHUNK = 256 / (D / 8) * 16;          // one batch of rows
    v_absmax_kernel<D><<<dim3((N + CHUNK - 1) / CHUNK, BH), 256, 0, st>>>(v, amax_bits, N, CHUNK);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int tiles = (Np + 127) / 128;
    v_quant_transpose_kernel<D><<<dim3(quant_groups(BH, tiles), BH), 256, 0, st>>>(v, amax_bits, vt, vscale, N, Np);
    return hipGetLastError();
}
hipError_t launch_quant_v(const void* v, int8_t* vt, float* vscale, unsigned* amax_bits,
                          int BH, int N, int D, hipStream_t st) {
    return D == 64 ? launch_quant_v_d<64>((const _Float16*)v, vt, vscale, amax_bits, BH, N, st)
                   : launch_quant_v_d<128>((const _Float16*)v, vt, vscale, amax_bits, BH, N, st);
}

}  // namespace sage
