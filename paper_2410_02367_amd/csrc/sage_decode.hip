// The attention loop for at most 32 query rows per (batch, head) slab (decoding, short tails of a prompt), FP16
// second product: Algorithm 1 with the keys dealt out to the wavefronts instead of the query rows.
//
// The call reads K^ and V once and does next to no arithmetic for them, so it is bound by memory -- if the rest keeps out
// of the way.  In the general kernel (sage_attn.hip) a workgroup has 128 query rows: of its four wavefronts one
// had real rows here, and all of them met at a barrier for every 64 keys.  Here a workgroup takes one slab, or one
// chunk of its keys; its wavefronts take 32-key tiles in turn, each with its own running maximum, sum and O, its own
// LDS buffers and no barrier, and their results are added at the end as chunks of a split launch are.
// Tiles come in by asynchronous loads straight to LDS, NBUF tiles per wavefront deep.
#include "sage_internal.h"
#include "sage_device.h"

namespace sage {

typedef int d4i __attribute__((ext_vector_type(4)));
typedef int d16i __attribute__((ext_vector_type(16)));
typedef float d16f __attribute__((ext_vector_type(16)));
typedef float d4f __attribute__((ext_vector_type(4)));
typedef float d2f __attribute__((ext_vector_type(2)));
typedef short d4s __attribute__((ext_vector_type(4)));
typedef _Float16 d2h __attribute__((ext_vector_type(2)));
typedef _Float16 d4h __attribute__((ext_vector_type(4)));

namespace {
constexpr float DEC_LOG2E = 1.4426950408889634f;
constexpr float DEC_SLACK = 8.0f;           // log2 of the largest P~ tolerated before the running maximum is raised
}  // namespace

// grid: one workgroup per (slab, key chunk), chunk fastest.  lse != nullptr: a partial result per chunk, as in sage_attn.hip.
// NW wavefronts: 4 while every workgroup has a compute unit to itself; with more workgroups than that and 24 KB of LDS per
// wavefront (D = 128), 2, so that three fit, unless the workgroups are long: see launch_decode_d().
template <int D, bool KTOK, int NBUF, int NW>
__global__ void __launch_bounds__(NW * 64, 1)
sage_decode_kernel(const int8_t* __restrict__ qi, const float* __restrict__ qsc, const int8_t* __restrict__ ki,
                   const float* __restrict__ ksc, const _Float16* __restrict__ vg, _Float16* __restrict__ og, float* __restrict__ lse,
                   int Nq, int Nkv, int shift_q, int shift_k, int causal, int BH, int n_splits, int chunk,
                   const _Float16* __restrict__ qf, float sm_scale) {
    constexpr int KS = D / 32, DT = D / 32, VROW = 2 * D;
    constexpr int KB = 32 * D, VB = 32 * VROW, SB = KTOK ? 256 : 0;       // bytes of a 32-key tile: K^, V, key scales (64 floats)
    constexpr int BUF = KB + VB + SB, WBUF = NBUF * BUF;
    constexpr int KL = KB / 1024, VL = VB / 1024, LOADS = KL + VL + (KTOK ? 1 : 0);
    constexpr int KCH = D / 16, VCH = VROW / 16;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NW * WBUF];
    __shared__ float s_m[NW][32], s_l[NW][32];
    static_assert(64 * DT * 16 * 4 <= WBUF, "the four O blocks fit where the tiles were");

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int ql = lane & 31, g = lane >> 5;
    const int bh = blockIdx.x / n_splits, split = blockIdx.x - bh * n_splits;
    const int k0 = split * chunk, N = split == n_splits - 1 ? Nkv - k0 : chunk;
    const size_t slab = (size_t)bh * Nkv + k0, slab_q = (size_t)bh * Nq;
    const int coff = Nkv - Nq - k0;
    const int nbq = (Nq + (1 << shift_q) - 1) >> shift_q, nbk = (Nkv + (1 << shift_k) - 1) >> shift_k;
    const float* __restrict__ ksc_bh = ksc + (size_t)bh * nbk + (k0 >> shift_k);
    const int tiles = (N + 31) / 32;

    // ---- tile loads of this wavefront.  Rows past the end lie beyond the descriptors: their K^ is masked, their V must
    // be finite, so the V buffers start as zeros (a load may leave them untouched).
    const unsigned base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)lds + wave * WBUF;
    const d4i k_rsrc = buffer_descriptor(ki + slab * D, (unsigned)N * D);
    const d4i v_rsrc = buffer_descriptor(vg + slab * D, (unsigned)N * VROW);
    const d4i s_rsrc = buffer_descriptor(ksc_bh, (unsigned)N * 4u);
    unsigned k_goff[KL], v_goff[VL];
#pragma unroll
    for (int i = 0; i < KL; ++i) {
        const int vi = 64 * i + lane, row = vi / KCH;
        k_goff[i] = (unsigned)(row * D + ((vi % KCH) ^ k_swz<D>(row)) * 16);
    }
#pragma unroll
    for (int i = 0; i < VL; ++i) {
        const int vi = 64 * i + lane, row = vi / VCH;
        v_goff[i] = (unsigned)(row * VROW + ((vi % VCH) ^ v_swz<D>(row)) * 16);
    }
    auto request = [&](int j, int buf) {
        const unsigned at = __builtin_amdgcn_readfirstlane((int)(base + buf * BUF));
#pragma unroll
        for (int i = 0; i < KL; ++i) load_to_lds16(k_rsrc, k_goff[i] + (unsigned)j * KB, at + 1024 * i);
#pragma unroll
        for (int i = 0; i < VL; ++i) load_to_lds16(v_rsrc, v_goff[i] + (unsigned)j * VB, at + KB + 1024 * i);
        if (KTOK) load_to_lds4(s_rsrc, (unsigned)(j * 32 + lane) * 4u, at + KB + VB);
    };
    unsigned char* const mine = lds + wave * WBUF;
    if (tiles * 32 > N) {
#pragma unroll
        for (int b = 0; b < NBUF; ++b)
#pragma unroll
            for (int i = 0; i < VL; ++i) *(d4i*)(mine + b * BUF + KB + 1024 * i + 16 * lane) = (d4i){0, 0, 0, 0};
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    // this wavefront's tiles: wave, wave + NW, ...
    const int mine_n = tiles > wave ? (tiles - wave + NW - 1) / NW : 0;
#pragma unroll
    for (int b = 0; b < NBUF; ++b)
        if (b < mine_n) request(wave + NW * b, b);

    // ---- queries: codes as they are, or made here from fp16 rows (with at most 32 rows a block of them is the wavefront's)
    d4i q[KS];
    float dq;
    const int qc = ql < Nq ? ql : Nq - 1;
    if (qf != nullptr) {
        QueryRows<KS> rows;
        rows.fetch(qf + (slab_q + qc) * D, g);
        const float amax = rows.block_amax(sm_scale, shift_q == 0 ? 0 : 5, wave, nullptr);
        const float rcp = amax > 0.0f ? 127.0f / amax : 0.0f;
        dq = amax / 127.0f * DEC_LOG2E;
        rows.codes(sm_scale, rcp, [&](int ks, int i, unsigned w) { q[ks][i] = (int)w; });
    } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) q[ks] = *(const d4i*)(qi + (slab_q + qc) * D + ks * 32 + g * 16);
        dq = qsc[(size_t)bh * nbq + (qc >> shift_q)] * DEC_LOG2E;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(q[ks]));        // loaded before the loop counts its own loads
    asm volatile("" : "+v"(dq));

    // ---- operand read offsets, as in sage_attn.hip
    int k_off[KS], v_off[DT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k_off[ks] = ql * D + (((2 * ks + g) ^ k_swz<D>(ql)) * 16);
    const int grp = lane >> 4, li = lane & 15, v_row = 4 * (grp >> 1) + (li >> 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        v_off[dt] = KB + v_row * VROW + (((4 * dt + 2 * (grp & 1) + ((li & 3) >> 1)) ^ v_swz<D>(v_row)) * 16) + (li & 1) * 8;

    d16f o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;
    float m_run = -__builtin_inff(), l = 0.0f;

    for (int n = 0, buf = 0; n < mine_n; ++n, buf = buf + 1 == NBUF ? 0 : buf + 1) {
        const int j = wave + NW * n, kv0 = 32 * j;
        const float dk = KTOK ? 1.0f : ksc_bh[kv0 >> shift_k];
        // tile n has landed; up to NBUF - 1 later ones stay in flight
        if (n + NBUF <= mine_n) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NBUF - 1) * LOADS) : "memory");
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        const unsigned char* tb = mine + buf * BUF;
        d16i s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const d4i*)(tb + k_off[ks]), q[ks], s, 0, 0, 0);
        // register r: key kv0 + 8 (r / 4) + 4 g + r % 4
        const float sc = __builtin_fmaxf(dq * dk, 1e-30f);
        float y[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) y[r] = (float)s[r];
        if (KTOK) {
            const float* ks_t = (const float*)(tb + KB + VB) + 4 * g;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const d4f a = *(const d4f*)(ks_t + 8 * c);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[4 * c + e] *= a[e];
            }
        }
        if (kv0 + 32 > N || (causal && kv0 + 31 > coff)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = kv0 + 8 * (r >> 2) + 4 * g + (r & 3);
                if (key >= N || (causal && key > ql + coff)) y[r] = -__builtin_inff();
            }
        }
        float top = y[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) top = __builtin_fmaxf(top, y[r]);
        top = pair32_max(top) * sc;
        if (__builtin_amdgcn_ballot_w64(top > m_run + DEC_SLACK) != 0ull) {
            const float m_new = __builtin_fmaxf(m_run, top);
            // (a row that has seen no key yet: nothing to rescale, and no difference of infinities)
            const float alpha = m_run == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        }
        const float m_sub = m_run == -__builtin_inff() ? 0.0f : m_run;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            d4i p;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(y[8 * u + 2 * e], sc, -m_sub));
                const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(y[8 * u + 2 * e + 1], sc, -m_sub));
                const d2h h = __builtin_convertvector((d2f){p0, p1}, d2h);
                p[e] = __builtin_bit_cast(int, h);
                l += (float)h[0] + (float)h[1];         // of the weights as the product takes them: their rounding cancels in O / l
            }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const unsigned char* va = tb + (16 * u) * VROW + v_off[dt];
                const d4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) d4s*)va);
                const d4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) d4s*)(va + 8 * VROW));
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                    __builtin_bit_cast(half8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)), __builtin_bit_cast(half8, p),
                    o[dt], 0, 0, 0);
            }
        }
        if (n + NBUF < mine_n) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // this tile has been read
            request(j + NW * NBUF, buf);
        }
    }

    // ---- the wavefronts' results: O = sum_w f_w O_w / sum_w f_w l_w, f_w = 2^(m_w - max m)
    l = pair32_sum(l);
    if (g == 0) {
        s_m[wave][ql] = m_run;
        s_l[wave][ql] = l;
    }
    __syncthreads();
    float m_all = s_m[0][ql];
#pragma unroll
    for (int w = 1; w < NW; ++w) m_all = __builtin_fmaxf(m_all, s_m[w][ql]);
    float l_all = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) l_all = __builtin_fmaf(s_l[w][ql], __builtin_amdgcn_exp2f(s_m[w][ql] - m_all), l_all);
    const float f = __builtin_amdgcn_exp2f(m_run - m_all);
    if (ql < Nq) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                d4f x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = o[dt][4 * c + e] * f;
                *(d4f*)(lds + ((wave * DT * 4 + dt * 4 + c) * 64 + lane) * 16) = x;
            }
    }
    __syncthreads();
    if (ql < Nq) {
        // each wavefront adds up its share of the 4 * DT register groups (4 channels each)
        const float inv = 1.0f / l_all;
        const size_t row = (lse != nullptr ? ((size_t)split * BH + bh) * Nq : slab_q) + ql;
        if (lse != nullptr && wave == 0 && g == 0) lse[row] = m_all + __builtin_amdgcn_logf(l_all);
#pragma unroll
        for (int i = 0; i < 4 * DT / NW; ++i) {
            const int c = wave * (4 * DT / NW) + i;
            d4f x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int w = 0; w < NW; ++w) x += *(const d4f*)(lds + ((w * DT * 4 + c) * 64 + lane) * 16);
            d4h h;
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = (_Float16)(x[e] * inv);
            *(d4h*)(og + row * D + 8 * c + 4 * g) = h;
        }
    }
}

// At D = 128 this kernel has one or three workgroups on a CU, the general one (sage_attn.hip) three of one 64-key tile at a
// time.  Where the workgroups do not go evenly into the 256 CUs -- more than one each, fewer than one and a half -- and are
// long, three small ones in flight read the memory better: us here / there, each pass on other inputs, 100 slabs of 5000
// keys (3 chunks) 50 / 47, of 16384 133 / 123; 130 of 8192 (2 chunks) 100 / 86; 300 of 1436 40 / 38, of 4096 101 / 92; 350 of
// 4096 105 / 100; 380 of 4096 108 / 107; from there on this one (400: 110 / 111, 600: 170 / 204); short ones too (130 of
// 1436, 718 a workgroup: 24.0 / 24.1; 300 of 700 21.7 / 22.6).  With one scale per key there is no such case (300 of
// 4096 102 / 105).
bool decode_takes(long workgroups, int Nq, int keys, int D, int block_k) {
    if (Nq > 32) return false;
    return !(D == 128 && block_k != 1 && workgroups > 256 && workgroups < 384 && keys >= 1280);
}

template <int D>
static hipError_t launch_decode_d(const Queries& q, const int8_t* kq, const float* kscale, const void* v, void* o, int BH, int Nq,
                                  int N, int causal, int block_q, int block_k, const SplitPlan& sp, hipStream_t st) {
    const int shift_q = __builtin_ctz((unsigned)block_q), shift_k = __builtin_ctz((unsigned)block_k);
    const dim3 grid((unsigned)(BH * sp.n_splits));
#define SAGE_DECODE(KT, NW) sage_decode_kernel<D, KT, 2, NW><<<grid, NW * 64, 0, st>>>(q.i8, q.scale, kq, kscale, (const _Float16*)v, \
        (_Float16*)o, sp.lse, Nq, N, shift_q, shift_k, causal, BH, sp.n_splits, sp.chunk, (const _Float16*)q.f16, q.sm_scale)
    // D = 128: 2 wavefronts while the second round of workgroups would be what counts (us with 2 / 4, each pass on other inputs: 600
    // slabs of 1436 keys 66 / 70, 800 of 700 46 / 53); for long ones the deeper queue of 4 (400 of 4096: 115 / 110, 200 of
    // 12000 in 2 chunks 169 / 162; 700 of 2000 97 / 96)
    if constexpr (D == 128) {
        if (grid.x > 256 && (sp.lse != nullptr ? sp.chunk : N) <= 2048) {
            if (block_k == 1) SAGE_DECODE(true, 2); else SAGE_DECODE(false, 2);
            return hipGetLastError();
        }
    }
    if (block_k == 1) SAGE_DECODE(true, 4); else SAGE_DECODE(false, 4);
#undef SAGE_DECODE
    return hipGetLastError();
}

hipError_t launch_decode(const Queries& q, const int8_t* kq, const float* kscale, const void* v, void* o, int BH, int Nq, int N,
                         int D, int causal, int block_q, int block_k, const SplitPlan& sp, hipStream_t st) {
    if (D == 64) return launch_decode_d<64>(q, kq, kscale, v, o, BH, Nq, N, causal, block_q, block_k, sp, st);
    return launch_decode_d<128>(q, kq, kscale, v, o, BH, Nq, N, causal, block_q, block_k, sp, st);
}

// ---- merge of the partial results of a split launch: O = sum_s w_s O_s / sum_s w_s, w_s = 2^(lse_s - max_s lse_s)
// A lane holds 8 channels of a row and takes every S-th chunk, BATCH of them requested before the first is used; the S
// lanes of the same channels add up at the end.  Few rows (a decode step): S as large as a wavefront allows, so that up
// to 16 (D = 128) or 32 chunks are one memory round trip (5.3 -> 3.5 us at 32 rows and 8 chunks); many rows: S = 1, the
// launch is bound by memory.
template <int D, int S, int BATCH>
__global__ void __launch_bounds__(256) merge_splits_kernel(const _Float16* __restrict__ part, const float* __restrict__ lse,
                                                           _Float16* __restrict__ og, long rows, int n_splits) {
    constexpr int TPR = D / 8, RPW = 64 / (TPR * S);
    const int lane = threadIdx.x & 63, c8 = lane % TPR, s0 = lane / TPR % S;
    const long row = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * RPW + lane / (TPR * S);
    if (row >= rows) return;           // (whole groups of TPR * S lanes)
    float top = -__builtin_inff(), wsum = 0.0f, acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
    for (int sb = 0; sb < n_splits; sb += S * BATCH) {
        float ls[BATCH];
        half8 x[BATCH];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            // (past the last chunk: the last one again, with weight 0)
            const int s = sb + b * S + s0, sc = s < n_splits ? s : n_splits - 1;
            const float v = lse[(size_t)sc * rows + row];
            x[b] = *(const half8*)(part + ((size_t)sc * rows + row) * D + c8 * 8);
            ls[b] = s < n_splits ? v : -__builtin_inff();
        }
        __builtin_amdgcn_sched_barrier(0);
        float most = top;
#pragma unroll
        for (int b = 0; b < BATCH; ++b) most = __builtin_fmaxf(most, ls[b]);
#pragma unroll
        for (int off = TPR; off < TPR * S; off <<= 1) most = __builtin_fmaxf(most, __shfl_xor(most, off, 64));
        const float keep = __builtin_amdgcn_exp2f(top - most);         // (0 on the first batch: top is -inf, most is not)
        top = most;
        wsum *= keep;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= keep;
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            const float w = __builtin_amdgcn_exp2f(ls[b] - top);
            wsum += w;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = __builtin_fmaf(w, (float)x[b][e], acc[e]);
        }
    }
#pragma unroll
    for (int off = TPR; off < TPR * S; off <<= 1) {
        wsum += __shfl_xor(wsum, off, 64);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], off, 64);
    }
    if (s0 == 0) {
        const float inv = 1.0f / wsum;
        half8 y;
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = (_Float16)(acc[e] * inv);
        *(half8*)(og + (size_t)row * D + c8 * 8) = y;
    }
}

template <int D>
static hipError_t launch_merge_d(const void* part, const float* lse, void* o, long rows, int n_splits, hipStream_t st) {
    constexpr int S = 64 / (D / 8);
    const _Float16* pp = (const _Float16*)part;
    _Float16* op = (_Float16*)o;
    const unsigned few = (unsigned)((rows + 3) / 4), many = (unsigned)((rows + 4 * S - 1) / (4 * S));
    if (rows <= 4096 && n_splits > 4) merge_splits_kernel<D, S, 4><<<few, 256, 0, st>>>(pp, lse, op, rows, n_splits);
    else if (rows <= 4096) merge_splits_kernel<D, S, 1><<<few, 256, 0, st>>>(pp, lse, op, rows, n_splits);
    else if (n_splits > 2) merge_splits_kernel<D, 1, 4><<<many, 256, 0, st>>>(pp, lse, op, rows, n_splits);
    else merge_splits_kernel<D, 1, 2><<<many, 256, 0, st>>>(pp, lse, op, rows, n_splits);
    return hipGetLastError();
}
hipError_t launch_merge_splits(const void* part, const float* lse, void* o, long rows, int D, int n_splits, hipStream_t st) {
    return D == 64 ? launch_merge_d<64>(part, lse, o, rows, n_splits, st) : launch_merge_d<128>(part, lse, o, rows, n_splits, st);
}

}  // namespace sage
