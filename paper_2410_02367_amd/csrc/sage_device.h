// Device code shared by the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>

namespace sage {

// Four INT8 codes round_half_even(clamp(x * rcp)) of Section 3.2, byte i from x[i].  Adding 1.5 * 2^23 rounds
// the (once rounded) product to an integer, ties to even, and leaves it in the low byte of the bit pattern in
// two's complement; a byte permute per pair packs them: 3.75 VALU instructions per code instead of 8 with a
// rounding, two-sided clamp, conversion, mask and shift.  The same bits as rintf and a conversion: |product| <= 127
// after the clamp, and a product that is not a number (0 * infinity: amax below 2^-121) is -127 either way.
__device__ __forceinline__ unsigned quantize4(float x0, float x1, float x2, float x3, float rcp) {
    auto code = [rcp](float x) {
        return __builtin_bit_cast(unsigned, __builtin_amdgcn_fmed3f(x * rcp, -127.0f, 127.0f) + 12582912.0f);
    };
    const unsigned lo = __builtin_amdgcn_perm(code(x1), code(x0), 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm(code(x3), code(x2), 0x04000c0cu);
    return lo | hi;
}

// a word as a float, by value (a bit_cast of a vector's element in place takes element 0 whatever its index)
__device__ __forceinline__ float word_f32(unsigned v) { return __builtin_bit_cast(float, v); }
// max / sum of a lane's value and that of the lane 32 away
__device__ __forceinline__ float pair32_max(float m) {
    const unsigned v = __builtin_bit_cast(unsigned, m);
    auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return __builtin_fmaxf(word_f32(r[0]), word_f32(r[1]));
}
__device__ __forceinline__ float pair32_sum(float x) {
    const unsigned v = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return word_f32(r[0]) + word_f32(r[1]);
}

// Maximum over groups of LANES adjacent lanes (4, 8, 16, 32 or 64), in every lane; passes over NaN as fmaxf does.  Lane
// permutations of the vector unit, about 8 clocks a step: __shfl_xor goes through the LDS, 60 or more, and the steps are a chain.
template <int CTRL>
__device__ __forceinline__ float dpp_max(float m) {
    const int v = __builtin_bit_cast(int, m);
    return __builtin_fmaxf(m, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false)));
}
template <int LANES>
__device__ __forceinline__ float lanes_max(float m) {
    m = dpp_max<0xB1>(m);                        // lane ^ 1
    m = dpp_max<0x4E>(m);                        // lane ^ 2
    if (LANES >= 8) m = dpp_max<0x141>(m);       // the other half of 8, mirrored
    if (LANES >= 16) m = dpp_max<0x140>(m);      // the other half of 16, mirrored
    if (LANES >= 32) {
        const unsigned v = __builtin_bit_cast(unsigned, m);
        auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        m = __builtin_fmaxf(word_f32(r[0]), word_f32(r[1]));
    }
    return LANES >= 64 ? pair32_max(m) : m;
}
// x + the value of the lane 32 (16) away, of two values at once: lanes of the lower half (even rows of 16) end with
// the sum of a, the others with the sum of b
__device__ __forceinline__ double fold32(double a, double b) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
    auto lo = __builtin_amdgcn_permlane32_swap(x[0], y[0], false, false), hi = __builtin_amdgcn_permlane32_swap(x[1], y[1], false, false);
    return __builtin_bit_cast(double, (u2){lo[0], hi[0]}) + __builtin_bit_cast(double, (u2){lo[1], hi[1]});
}
__device__ __forceinline__ double fold16(double a, double b) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
    auto lo = __builtin_amdgcn_permlane16_swap(x[0], y[0], false, false), hi = __builtin_amdgcn_permlane16_swap(x[1], y[1], false, false);
    return __builtin_bit_cast(double, (u2){lo[0], hi[0]}) + __builtin_bit_cast(double, (u2){lo[1], hi[1]});
}

// ---- tiles of K^ and V in LDS (the attention kernels)
// Rows are unpadded (K^ of D bytes, V of 2 D); their 16-byte chunks are XOR-swizzled so that the operand reads of 16
// consecutive rows touch every bank once.
template <int D> __device__ __forceinline__ int k_swz(int row) { return D == 128 ? ((row >> 1) & 7) : ((row >> 2) & 3); }
template <int D> __device__ __forceinline__ int v_swz(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }

// Raw-buffer descriptor of `bytes` bytes at `base` (wave-uniform; readfirstlane pins it to scalar registers): the hardware
// checks every lane's offset against the size, and a lane beyond it does not touch memory.  The ragged last tile
// needs no clamping code: its rows are masked or multiplied by P~ = 0 anyway.
typedef int buffer4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ buffer4 buffer_descriptor(const void* base, unsigned bytes) {
    const unsigned long long p = (unsigned long long)base;
    // dword 0-1: 48-bit base, stride 0 (raw buffer); dword 2: size in bytes; dword 3: 32-bit data format
    return (buffer4){__builtin_amdgcn_readfirstlane((int)(unsigned)p),
                     __builtin_amdgcn_readfirstlane((int)((unsigned)(p >> 32) & 0xffffu)),
                     __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
}
// 16 (4) bytes per lane from global memory straight into LDS: lane l lands at LDS byte address lds_addr + 16 l (4 l), with
// lds_addr in a scalar register.  Written as assembly because the compiler, which cannot tell which LDS bytes such a
// load writes, makes every later LDS read wait for it (vmcnt(0)) and so turns the asynchronous load into a synchronous
// one.  Completion is tracked by hand: the issuing wavefront waits with s_waitcnt vmcnt before it reads the bytes, or
// before the barrier that publishes them.  m0 is set without being declared; the build checks that the compiler does not
// use it itself.
__device__ __forceinline__ void load_to_lds16(const buffer4& rsrc, unsigned goff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
                 : : "v"(goff), "s"(rsrc), "s"(lds_addr) : "memory");
}
__device__ __forceinline__ void load_to_lds4(const buffer4& rsrc, unsigned goff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dword %0, %1, 0 offen lds"
                 : : "v"(goff), "s"(rsrc), "s"(lds_addr) : "memory");
}
// an address that is the same in every lane, pinned to a scalar register
__device__ __forceinline__ unsigned uniform(unsigned addr) { return (unsigned)__builtin_amdgcn_readfirstlane((int)addr); }

// Causal launches: item `slot` of an XCD -> (unit, query tile).  A unit is a (batch, head) slab or a key chunk of one; a
// tile's weight grows with qt, so the order is heaviest tile first over `group` units of the XCD at a time (one pass),
// whose K^ and V the WGs on the XCD then walk together; see causal_order().  Units left over after the passes of 8 *
// group are shared by all XCDs: with U of them, query tile number r (from the heaviest) of unit s goes to XCD
// (8 s + e) / U, where e runs through 0 .. 7 as r does, in bit-reversed order -- every XCD gets U / 8 of the tiles of every
// weight, and a unit's tiles stay on as few XCDs as that allows.  Returns false where the XCD has no such item.
struct CausalOrder {
    int group, full, rest;      // units per XCD and pass; passes; units left over
};
__host__ __device__ __forceinline__ int causal_share(int xcd, int rest, int e, int& first) {
    const int lo = xcd * rest - e, hi = lo + rest;         // units s with lo <= 8 s < hi
    first = (lo + 7) >> 3;
    return ((hi + 7) >> 3) - first;
}
__device__ __forceinline__ bool causal_item(int xcd, int slot, int tiles_q, const CausalOrder& o, int& unit, int& qt) {
    const int pass_items = o.group * tiles_q;
    const int pass = slot / pass_items;
    if (pass < o.full) {
        const int i = slot - pass * pass_items, r = i / o.group;
        unit = (pass * 8 + xcd) * o.group + (i - r * o.group);
        qt = tiles_q - 1 - r;
        return true;
    }
    if (o.rest == 0) return false;
    const int i = slot - o.full * pass_items, block = i / o.rest;
    int at = i - block * o.rest, r = 8 * block;
    for (int k = 0; k < 8; ++k, ++r) {
        int first;
        const int n = causal_share(xcd, o.rest, ((k & 1) << 2) | (k & 2) | (k >> 2), first);
        if (at < n) {
            unit = o.full * 8 * o.group + first + at;
            qt = tiles_q - 1 - r;
            return qt >= 0;
        }
        at -= n;
    }
    return false;
}

// The same without the clamp: where 127 / amax and every value are finite, and for K, where no product exceeds 127 (1 + 2^-22)
// and none overflows -- the smallest non-zero |K - mean| is far above 2^-121 (K is a multiple of 2^-24, the mean at least 2^-47).
__device__ __forceinline__ unsigned quantize4_k(float x0, float x1, float x2, float x3, float rcp) {
    auto code = [rcp](float x) { return __builtin_bit_cast(unsigned, x * rcp + 12582912.0f); };
    const unsigned lo = __builtin_amdgcn_perm(code(x1), code(x0), 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm(code(x3), code(x2), 0x04000c0cu);
    return lo | hi;
}

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
// max(m, |x|) of two fp16 values at once, x as a word; of half2v the other operand where one is NaN, of ushort2v the larger
// bit pattern: the order of the numbers, infinity and then NaN above them
template <class T>
__device__ __forceinline__ T max_abs(T m, unsigned x) {
    return __builtin_elementwise_max(m, __builtin_bit_cast(T, x & 0x7fff7fffu));
}

// The fp16 rows of a wavefront's 32 queries quantized where they are used (Section 4.6: the quantizer fused
// into the operator's neighbour): lane l holds half of row l % 32, the channels 32 ks + 16 (l / 32) .. + 15, as the
// INT8 matrix instruction's operand wants them.  amax of a row: both lanes of it; of a block of 32, 64 or 128
// rows: the wavefronts that share the block, through one LDS word each.
// The workgroup's rows start at a multiple of every block size.  Same arithmetic as the pre-pass kernel.
template <int KS>
struct QueryRows {
    half8 raw[KS][2];
    bool special;           // wave-uniform, set by block_amax(): some query of the wavefront is NaN or infinite
    // row: the lane's row; lanes past the last row fetch that row again, which changes no maximum they share with a
    // row that exists (a condition around the loads would make them wait for each other)
    __device__ __forceinline__ void fetch(const _Float16* row, int half) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < 2; ++j) raw[ks][j] = *(const half8*)(row + 32 * ks + 16 * half + 8 * j);
        __builtin_amdgcn_sched_barrier(0);
    }
    // largest |x * sm_scale| of the lane's quantization block; every wavefront of the workgroup calls it.
    // red: one float of LDS per wavefront, not used for anything else before the next barrier.
    __device__ __forceinline__ float block_amax(float sm_scale, int shift_q, int wave, float* red) {
        // max |x * sm_scale| = max |x| * sm_scale, rounded once either way (rounding is monotonic): the maximum is
        // taken on fp16 pairs, of the bit patterns, which shows a NaN at no cost.  Where there is one it is taken again and
        // passes over NaN, as fmaxf does: a row that holds one leaves the other rows of its block as they are.
        auto over_all = [&](auto start) {
            typedef unsigned u4 __attribute__((ext_vector_type(4)));
            auto m = start;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const u4 w = __builtin_bit_cast(u4, raw[ks][j]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) m = max_abs(m, w[e]);
                }
            return m;
        };
        const ushort2v pattern = over_all(ushort2v{});
        special = __builtin_amdgcn_ballot_w64(pattern[0] >= 0x7C00 || pattern[1] >= 0x7C00) != 0ull;
        half2v top = __builtin_bit_cast(half2v, pattern);
        if (__builtin_expect(special, 0)) top = over_all(half2v{});
        float m = __builtin_fmaxf((float)top[0], (float)top[1]) * sm_scale;
        m = pair32_max(m);
        if (shift_q == 0) return m;
        m = lanes_max<32>(m);
        if (shift_q == 5) return m;
        if ((threadIdx.x & 63) == 0) red[wave] = m;
        __syncthreads();
        const int first = shift_q == 6 ? wave & ~1 : wave & ~3;
        m = __builtin_fmaxf(red[first], red[first + 1]);
        if (shift_q == 7) m = __builtin_fmaxf(m, __builtin_fmaxf(red[first + 2], red[first + 3]));
        return m;
    }
    // put(ks, i, word): word i of contraction step ks, channels 4 i .. 4 i + 3 of the lane's 16.  rcp = 127 / amax, or 0.
    // The clamp matters only where 127 / amax overflows (amax below 2^-121), elsewhere no product exceeds 127 (1 + 2^-22), and
    // for a product that is not a number, whose code is -127.  Without it a code is 3.75 vector instructions instead of 4.75.
    template <class F>
    __device__ __forceinline__ void codes(float sm_scale, float rcp, F&& put) const {
        auto all = [&](auto clamp) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int i = 0; i < 4; ++i) put(ks, i, word<decltype(clamp)::value>(ks, i, sm_scale, rcp));
        };
        if (__builtin_expect(special || __builtin_amdgcn_ballot_w64(rcp == __builtin_inff()) != 0ull, 0)) all(std::true_type{});
        else all(std::false_type{});
    }
    template <bool CLAMP>
    __device__ __forceinline__ unsigned word(int ks, int i, float sm_scale, float rcp) const {
        const half8& h = raw[ks][i >> 1];
        const int e = 4 * (i & 1);
        // x * sm_scale rounded once: the FMA takes the fp16 operand as it is (no conversion), the 0 changes no code
        auto scaled = [sm_scale](_Float16 x) { return __builtin_fmaf((float)x, sm_scale, 0.0f); };
        return CLAMP ? quantize4(scaled(h[e]), scaled(h[e + 1]), scaled(h[e + 2]), scaled(h[e + 3]), rcp)
                     : quantize4_k(scaled(h[e]), scaled(h[e + 1]), scaled(h[e + 2]), scaled(h[e + 3]), rcp);
    }
};

// Stores a wavefront's 32 output rows (fp16, D channels).  As the matrix instructions leave O^T, a lane owns one row
// and holds 4 consecutive channels (8 bytes) at a time; stored like that, an instruction writes 16 bytes to each of 32
// rows, and the stores of a workgroup were 11 % of the time of a 1536-token sequence.  Two register swaps with the
// lanes 32 and 16 away collect 16 bytes per lane and 64 bytes per row: half the store instructions, a quarter of the
// row segments.
// value(dt, r): register r of the lane's block of channels 32 dt ..: row lane % 32, channel 8 (r / 4) + 4 (lane / 32) + r % 4.
// rows: how many of the 32 rows exist.  final: the output itself, which nobody on this XCD reads again, goes past the
// L2 that holds K^ and V (1-3 % up to 4K tokens); partial results, which a merge reads next, stay in it.
template <int D, class F>
__device__ __forceinline__ void store_rows(_Float16* out, int rows, int lane, bool final, F&& value) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef int i4 __attribute__((ext_vector_type(4)));
    const int row = lane & 15, chunk = 2 * ((lane >> 4) & 1) + (lane >> 5);
    _Float16* const at = out + (size_t)row * D + 8 * chunk;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
        i4 c[2];                // chunk 2 k + lane / 32 of the lane's row, 8 channels
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const f2 x = {value(dt, 8 * k + 2 * i), value(dt, 8 * k + 2 * i + 1)};
                const f2 y = {value(dt, 8 * k + 4 + 2 * i), value(dt, 8 * k + 4 + 2 * i + 1)};
                auto s = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, __builtin_convertvector(x, h2)),
                                                          __builtin_bit_cast(int, __builtin_convertvector(y, h2)), false, false);
                c[k][i] = s[0];
                c[k][2 + i] = s[1];
            }
        i4 w[2];                // rows 0 .. 15 and 16 .. 31: chunk `chunk` of row `row`
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            auto s = __builtin_amdgcn_permlane16_swap(c[0][m], c[1][m], false, false);
            w[0][m] = s[0];
            w[1][m] = s[1];
        }
        if (final) {
            if (row < rows) __builtin_nontemporal_store(w[0], (i4*)(at + 32 * dt));
            if (row + 16 < rows) __builtin_nontemporal_store(w[1], (i4*)(at + 16 * D + 32 * dt));
        } else {
            if (row < rows) *(i4*)(at + 32 * dt) = w[0];
            if (row + 16 < rows) *(i4*)(at + 16 * D + 32 * dt) = w[1];
        }
    }
}

}  // namespace sage
