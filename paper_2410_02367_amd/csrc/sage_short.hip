// The whole pass of Algorithm 1 in one launch for key sequences that fit the LDS of a compute unit: smoothing and
// quantization of K (Sections 4.2, 3.2), quantization of Q (Section 4.6) and the attention loop (Sections 3.1, 4.4).
//
// A workgroup of 4 wavefronts reads the keys of one (batch, head) slab once, into registers: exact column sums,
// mean, block maxima and codes all come from there, K^ stays in LDS, V goes to LDS while that happens, and the
// wavefronts then walk 32-row query tiles without another barrier.  Nothing but Q, K and V is read from memory and
// nothing but O is written.
//
// Several workgroups can share a slab (each takes its part of the query tiles and makes K^ for itself); see
// short_groups() for how many, and short_fits() for which launches come here.
//
// Measured against the launches of the separate calls, us for the whole call: 12 x 64 slabs of 197 keys at D = 64: 44 ->
// 24.4; 1 x 2 of 256: 32 -> 7.8; 129 of 512: 36 -> 25; 256 of 256 at D = 128: 39 -> 17.5; 128 x (4096 queries against 77
// keys): 133 -> 67.  (26.5 and 8.6 before maxima went through lane permutations instead of the LDS, masks took one comparison
// per score and the first tile's rescaling of an empty accumulator was left out; 667 x 468, causal: 66.1 -> 60.5, 616 x 84 x
// 128, causal: 18.0 -> 15.9.)  Bounds: launch latency for few slabs; for many, a memory phase (Q, K, V in, at the copy rate)
// and a VALU phase (codes of K^ and Q^, softmax) of about equal length, which overlap only between workgroups.
#include "sage_internal.h"
#include "sage_device.h"
#include <type_traits>

namespace sage {

typedef int s4i __attribute__((ext_vector_type(4)));
typedef int s16i __attribute__((ext_vector_type(16)));
typedef float s16f __attribute__((ext_vector_type(16)));
typedef short s4s __attribute__((ext_vector_type(4)));
typedef float s2f __attribute__((ext_vector_type(2)));
typedef _Float16 s2h __attribute__((ext_vector_type(2)));

namespace {
constexpr float SHORT_LOG2E = 1.4426950408889634f;
constexpr float SHORT_SLACK = 8.0f;         // log2 of the largest P~ tolerated before the running maximum is raised
constexpr int SHORT_MAGIC_I = 0x4B400000;    // 12582912.0f = 1.5 * 2^23
constexpr float SHORT_MAGIC = 12582912.0f;
typedef float s4f __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float as_f(unsigned v) { return __builtin_bit_cast(float, v); }
__device__ __forceinline__ unsigned as_u(float v) { return __builtin_bit_cast(unsigned, v); }
}  // namespace

// D channels, NTILE tiles of 64 keys at most, NW wavefronts; KTOK: one scale per key.  grid: groups workgroups per
// slab.  48 KB of K^ and V (NTILE * D = 256): 4 wavefronts, two or three workgroups per CU; 96 KB: 8 wavefronts, one.
// KSP = 2: launches that leave CUs empty, where a workgroup's chain is all there is.  Two wavefronts share a query tile, each
// takes every other key tile, and their results are added up in LDS; a workgroup makes one round (NW / 2 query tiles).
template <int D, int NTILE, int NW, int KSP, bool KTOK>
__device__ __forceinline__ void short_pass(const _Float16* __restrict__ qf, const _Float16* __restrict__ kf,
                                           const _Float16* __restrict__ vf, _Float16* __restrict__ og, int Nq, int N,
                                           int shift_q, int shift_k, int causal, float sm_scale, int groups) {
    constexpr int KMAX = NTILE * 64;            // keys that fit
    constexpr int VPR = D / 8;                  // 16-byte vectors (8 channels) of a K row
    constexpr int RPI = 64 / VPR;               // K rows per load instruction of a wavefront
    constexpr int LPG = 32 / RPI;               // load instructions per group of 32 rows
    constexpr int GPW = NTILE * 2 / NW;         // groups of 32 rows per wavefront
    constexpr int NT = NW * 64;
    constexpr int KS = D / 32, DT = D / 32;
    constexpr int VROW = 2 * D;
    constexpr int VCH = VROW / 16;              // 16-byte chunks of a V row
    static_assert(GPW >= 1, "every wavefront owns at least one group of 32 keys");
    constexpr int RT = NW / KSP;                // query tiles of a round
    static_assert(KSP == 1 || RT == 4, "a round is a multiple of every block_q");
    constexpr int MERGE = KSP == 1 ? 0 : RT * 32 * D * 4, TILES = KMAX * D + KMAX * VROW;      // bytes
    __shared__ __attribute__((aligned(1024))) unsigned char pool[TILES > MERGE ? TILES : MERGE];
    unsigned char* const kl = pool;
    unsigned char* const vl = pool + KMAX * D;
    __shared__ __attribute__((aligned(16))) float s_mean[D];
    __shared__ __attribute__((aligned(16))) float s_max[KMAX / 32];
    __shared__ __attribute__((aligned(16))) float s_scale[KTOK ? KMAX : KMAX / 64];
    __shared__ __attribute__((aligned(16))) float s_bias[KTOK ? KMAX : 4];       // -12582912 * s_scale
    __shared__ float s_q[2][RT];
    __shared__ float s_ml[KSP == 1 ? 1 : 2 * RT][64];
    static_assert(NW * D * 8 <= KMAX * D, "the partial column sums fit where K^ will be");
    double (*const s_part)[D] = (double (*)[D])kl;       // [wavefront][channel]; read before the codes are written

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int ql = lane & 31, g = lane >> 5;
    const int own = KSP == 1 ? wave : wave % RT, kpart = KSP == 1 ? 0 : wave / RT;      // query tile of a round; share of the key tiles
    const int bh = blockIdx.x / groups, part = blockIdx.x - bh * groups;
    const size_t slab = (size_t)bh * N, slab_q = (size_t)bh * Nq;
    const int tiles = (N + 63) / 64;
    const int coff = Nq <= N ? N - Nq : 0;       // (only read when causal, where Nq <= N)

    // ---- keys into registers; groups of 32 rows past the end are skipped, rows past the end repeat the last one
    half8 x[GPW][LPG];
    const int c8 = lane % VPR, r0 = wave * (GPW * 32) + lane / VPR;
    const _Float16* kbase = kf + slab * D + c8 * 8;
#pragma unroll
    for (int gr = 0; gr < GPW; ++gr) {
        if (wave * (GPW * 32) + gr * 32 >= N) continue;
#pragma unroll
        for (int i = 0; i < LPG; ++i) {
            const int r = r0 + gr * 32 + i * RPI;
            x[gr][i] = *(const half8*)(kbase + (size_t)(r < N ? r : N - 1) * D);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- values into LDS, asynchronously.  Chunks of rows past the end are zeroed first (P~ is 0 there, but 0 * NaN
    // would not be); their loads lie beyond the descriptor.
    {
        const s4i rsrc = buffer_descriptor(vf + slab * D, (unsigned)N * VROW);
        const unsigned base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)vl;
        const int vecs = tiles * (64 * VCH);
        for (int i = wave * 64; i < vecs; i += NT) {
            const int vi = i + lane, row = vi / VCH, c = (vi % VCH) ^ v_swz<D>(row);
            if (i / VCH + 64 / VCH > N) {
                *(s4i*)(vl + vi * 16) = (s4i){0, 0, 0, 0};
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            load_to_lds16(rsrc, (unsigned)(row * VROW + c * 16), uniform(base + i * 16));
        }
    }
    const int rtiles = (Nq + 31) / 32;
    // the workgroup's query tiles: RT at a time (128 or 256 rows, a multiple of every block_q)
    QueryRows<KS> rows;
    {
        const int row = (part * RT + own) * 32 + ql;
        rows.fetch(qf + (slab_q + (row < Nq ? row : Nq - 1)) * D, g);
    }

    // ---- exact column sums (fp64: multiples of 2^-24 below 2^25), folded over the wavefront's rows.  The keys stay in
    // registers as fp32 from here on: every conversion is made once.
    float xs[GPW][LPG][8];
    double sum[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] = 0.0;
#pragma unroll
    for (int gr = 0; gr < GPW; ++gr) {
        if (wave * (GPW * 32) + gr * 32 >= N) continue;
        const bool whole = wave * (GPW * 32) + gr * 32 + 32 <= N;
#pragma unroll
        for (int i = 0; i < LPG; ++i) {
            const double live = whole || r0 + gr * 32 + i * RPI < N ? 1.0 : 0.0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                xs[gr][i][e] = (float)x[gr][i][e];
                sum[e] = __builtin_fma(live, (double)xs[gr][i][e], sum[e]);
            }
        }
    }
    {
        // lanes 32 apart, then 16 apart (then 8, where a row is 8 lanes) hold the same channels of other rows
        double a[4], b[2];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = fold32(sum[e], sum[e + 4]);
#pragma unroll
        for (int e = 0; e < 2; ++e) b[e] = fold16(a[e], a[e + 2]);
        if (VPR == 8) {
#pragma unroll
            for (int e = 0; e < 2; ++e) b[e] += __shfl_xor(b[e], 8, 64);
        }
        const int ch = c8 * 8 + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1);
        s_part[wave][ch] = b[0];
        s_part[wave][ch + 1] = b[1];
    }
    __syncthreads();
    if (t < D) {
        double total = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) total += s_part[w][t];
        s_mean[t] = (float)(total / (double)N);
    }
    __syncthreads();
    float mean[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) mean[e] = s_mean[c8 * 8 + e];

    // ---- codes of K^ into LDS (rows of D bytes, 16-byte chunks swizzled)
#pragma unroll
    for (int gr = 0; gr < GPW; ++gr) {
        if (wave * (GPW * 32) + gr * 32 >= N) continue;
#pragma unroll
        for (int i = 0; i < LPG; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) xs[gr][i][e] -= mean[e];
    }
    auto store_codes = [&](const float (&f)[8], int r, float rcp) {
        const uint2 w = make_uint2(quantize4_k(f[0], f[1], f[2], f[3], rcp), quantize4_k(f[4], f[5], f[6], f[7], rcp));
        *(uint2*)(kl + r * D + (((c8 >> 1) ^ k_swz<D>(r)) * 16) + (c8 & 1) * 8) = w;
    };
    auto row_max = [&](float m, const float (&f)[8]) {
#pragma unroll
        for (int e = 0; e < 8; e += 2) m = __builtin_fmaxf(__builtin_fmaxf(m, __builtin_fabsf(f[e])), __builtin_fabsf(f[e + 1]));
        return m;
    };
    float k_top = 0.0f;              // one scale per block: the largest key of all
    if (KTOK) {
#pragma unroll
        for (int gr = 0; gr < GPW; ++gr) {
            if (wave * (GPW * 32) + gr * 32 >= N) continue;
#pragma unroll
            for (int i = 0; i < LPG; ++i) {
                const int r = r0 + gr * 32 + i * RPI;
                float m = row_max(0.0f, xs[gr][i]);
                m = lanes_max<VPR>(m);
                if (c8 == 0) {
                    // 22 significant bits, so that 12582912 * a is exact; not 0, so that -inf * a is not NaN
                    const float a = as_f(as_u(__builtin_fmaxf(m / 127.0f, 1e-30f)) & ~3u);
                    s_scale[r] = a;
                    s_bias[r] = -SHORT_MAGIC * a;
                }
                store_codes(xs[gr][i], r, m > 0.0f ? 127.0f / m : 0.0f);
            }
        }
    } else {
        float gm[GPW];
#pragma unroll
        for (int gr = 0; gr < GPW; ++gr) {
            gm[gr] = 0.0f;
            if (wave * (GPW * 32) + gr * 32 >= N) continue;
#pragma unroll
            for (int i = 0; i < LPG; ++i) gm[gr] = row_max(gm[gr], xs[gr][i]);      // a repeated row changes no maximum
        }
#pragma unroll
        for (int gr = 0; gr < GPW; ++gr) {
            gm[gr] = lanes_max<64>(gm[gr]);
            if (lane == 0) s_max[wave * GPW + gr] = gm[gr];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < KMAX / 32; ++i) k_top = __builtin_fmaxf(k_top, s_max[i]);       // (a group past the end has 0)
#pragma unroll
        for (int gr = 0; gr < GPW; ++gr) {
            const int row = wave * (GPW * 32) + gr * 32;
            if (row >= N) continue;
            const int blk = (row >> shift_k) << (shift_k - 5);       // first 32-row group of the quantization block (64 or 128 rows)
            float m = __builtin_fmaxf(s_max[blk], s_max[blk + 1]);
            if (shift_k == 7 && NTILE > 1) m = __builtin_fmaxf(m, __builtin_fmaxf(s_max[blk + 2], s_max[blk + 3]));
            if (lane == 0) s_scale[row >> 6] = m / 127.0f;           // (both groups of a tile write the same value)
            const float rcp = m > 0.0f ? 127.0f / m : 0.0f;
#pragma unroll
            for (int i = 0; i < LPG; ++i) store_codes(xs[gr][i], r0 + gr * 32 + i * RPI, rcp);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // this wavefront's part of V has landed
    __syncthreads();

    // ---- operand read offsets, as in sage_attn.hip
    int k_off[KS], v_off[DT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k_off[ks] = ql * D + (((2 * ks + g) ^ k_swz<D>(ql)) * 16);
    const int grp = lane >> 4, li = lane & 15, v_row = 4 * (grp >> 1) + (li >> 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        v_off[dt] = v_row * VROW + (((4 * dt + 2 * (grp & 1) + ((li & 3) >> 1)) ^ v_swz<D>(v_row)) * 16) + (li & 1) * 8;

    // seed of the scores and selector of the row sums, as in sage_attn.hip
    s16i magic;
#pragma unroll
    for (int r = 0; r < 16; ++r) magic[r] = SHORT_MAGIC_I;
    const int sel_word = (((lane >> 4) ^ lane) & 1) ? 0 : 0x3C003C00;
    const s4i sel = {sel_word, sel_word, sel_word, sel_word};

    for (int set = part, turn = 0; set * RT < rtiles; set += groups, turn ^= 1) {
        const int row0 = (set * RT + own) * 32;
        const float qmax = rows.block_amax(sm_scale, shift_q, own, s_q[turn]);
        const float qrcp = qmax > 0.0f ? 127.0f / qmax : 0.0f;
        const float dq = qmax / 127.0f * SHORT_LOG2E;
        s4i q[KS];
        rows.codes(sm_scale, qrcp, [&](int ks, int i, unsigned w) { q[ks][i] = (int)w; });
        if (KSP == 1 && (set + groups) * RT < rtiles) {          // the next rows are requested before this tile's loop
            const int row = ((set + groups) * RT + own) * 32 + ql;
            rows.fetch(qf + (slab_q + (row < Nq ? row : Nq - 1)) * D, g);
        }
        if (KSP == 1 && row0 >= Nq) continue;

        s16f o[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;
        s4f lsum = {0.0f, 0.0f, 0.0f, 0.0f};       // registers 0, 1: sums of the queries lane % 16, 16 + lane % 16
        // Below every score.  With KSP = 2 a row may see none of its wavefront's keys, and the start is finite: the row's weights
        // are then exp2(-inf + 3.4e38) = 0, where an infinity would make them NaN.  (The second lowest number, since rounding
        // the lowest to the grid of a huge scale could leave the range.)
        float m_run = KSP == 1 ? -__builtin_inff() : -0x1.fffffcp127f;
        bool fresh = true;                           // O and l are 0
        // keys this wavefront sees; a tile of which it sees only the first half is done by halves
        int seen = causal ? row0 + 32 + coff : N;
        seen = seen < N ? seen : N;
        // COARSE: the scales make the grid of the maximum wider than 1 (coarse_dk in sage_attn.hip); the scores lose their seed,
        // which is exact, and need no grid.
        auto tile = [&](int j, auto HALVES, auto COARSE) {
            constexpr int NH = HALVES.value;
            constexpr bool seeded = !KTOK && COARSE.value == 0;
            const unsigned char* kt = kl + j * (64 * D);
            s16i s[NH];
#pragma unroll
            for (int h = 0; h < NH; ++h) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    s[h] = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const s4i*)(kt + h * (32 * D) + k_off[ks]), q[ks], ks == 0 ? magic : s[h], 0, 0, 0);
            }
            if (COARSE.value != 0) {
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[h][r] = (int)as_u(as_f((unsigned)s[h][r]) - SHORT_MAGIC);
            }
            // register r of half h: key 64 j + 32 h + 8 (r / 4) + 4 g + r % 4
            const float sc = KTOK ? __builtin_fmaxf(dq, 1e-30f) : as_f(as_u(__builtin_fmaxf(dq * s_scale[j], 1e-30f)) & ~3u);
            if (j * 64 + 32 * NH > N || (causal && j * 64 + 32 * NH - 1 > row0 + coff)) {
                // keys of the lane's half that the row sees, counted from the tile's first: one comparison per score
                // (formed here and not ahead of the loop, where it would cost a register of the 168)
                int ln = t & 63;
                asm volatile("" : "+v"(ln));
                int last = N;
                if (causal && last > row0 + (ln & 31) + coff + 1) last = row0 + (ln & 31) + coff + 1;
                last -= 64 * j + 4 * (ln >> 5);
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int r = 0; r < 16; ++r)        // -inf, and below every score
                        s[h][r] = 32 * h + 8 * (r >> 2) + (r & 3) < last ? (int)s[h][r] : (int)0xFF800000;
            }
            // the argument of exp2 is y * sc + bias, y the seeded score (KTOK: the score times delta_K); see sage_attn.hip
            // for why it is rounded once, and why that needs the running maximum on the grid of 12582912 * sc
            float y[NH][16], bias;
            bool off_grid = false, want;
            float mf = 0.0f;
            int mi = 0;
            if (KTOK) {
                const float* ka = s_scale + 64 * j + 4 * g;
                const float* kb = s_bias + 64 * j + 4 * g;
                mf = -__builtin_inff();
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const s4f a = *(const s4f*)(ka + 32 * h + 8 * c), b = *(const s4f*)(kb + 32 * h + 8 * c);
#pragma unroll
                        for (int e = 0; e < 4; ++e) y[h][4 * c + e] = __builtin_fmaf(as_f((unsigned)s[h][4 * c + e]), a[e], b[e]);
                        mf = __builtin_fmaxf(__builtin_fmaxf(mf, y[h][4 * c]), y[h][4 * c + 1]);
                        mf = __builtin_fmaxf(__builtin_fmaxf(mf, y[h][4 * c + 2]), y[h][4 * c + 3]);
                    }
                bias = -m_run;
                want = __builtin_fmaf(mf, sc, bias) > SHORT_SLACK;
            } else if (!seeded) {
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int r = 0; r < 16; ++r) y[h][r] = as_f((unsigned)s[h][r]);
                mf = y[0][0];
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int r = 0; r < 16; ++r) mf = __builtin_fmaxf(mf, y[h][r]);
                bias = -m_run;
                want = __builtin_fmaf(mf, sc, bias) > SHORT_SLACK;
            } else {
                mi = s[0][0];
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int r = 0; r < 16; r += 2) mi = max(max(mi, (int)s[h][r]), (int)s[h][r + 1]);
#pragma unroll
                for (int h = 0; h < NH; ++h)
#pragma unroll
                    for (int r = 0; r < 16; ++r) y[h][r] = as_f((unsigned)s[h][r]);
                const float at = __builtin_fmaf(SHORT_MAGIC, sc, m_run);
                bias = -at;
                off_grid = __builtin_fmaf(-SHORT_MAGIC, sc, at) != m_run;
                want = off_grid || __builtin_fmaf(as_f((unsigned)mi), sc, bias) > SHORT_SLACK;
            }
            if (__builtin_amdgcn_ballot_w64(want) != 0ull) {
                // (on the first tile every row that sees a key is here)
                float top;
                if (!seeded) {
                    auto x = __builtin_amdgcn_permlane32_swap(as_u(mf), as_u(mf), false, false);
                    top = __builtin_fmaxf(as_f(x[0]), as_f(x[1])) * sc;
                } else {
                    auto x = __builtin_amdgcn_permlane32_swap((unsigned)mi, (unsigned)mi, false, false);
                    top = (as_f((unsigned)max((int)x[0], (int)x[1])) - SHORT_MAGIC) * sc;
                }
                float m_new = __builtin_fmaxf(m_run, top);
                if (seeded) m_new = __builtin_fmaf(-SHORT_MAGIC, sc, __builtin_fmaf(SHORT_MAGIC, sc, m_new));
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
                m_run = m_new;
                bias = !seeded ? -m_run : -__builtin_fmaf(SHORT_MAGIC, sc, m_run);
                if (!fresh) {
                    lsum *= alpha;
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
                }
            }
            fresh = false;
            const unsigned char* vt = vl + j * (64 * VROW);
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    s4i p;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(y[h][8 * u + 2 * e], sc, bias));
                        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(y[h][8 * u + 2 * e + 1], sc, bias));
                        p[e] = __builtin_bit_cast(int, __builtin_convertvector((s2f){p0, p1}, s2h));
                    }
                    // row sums on the matrix pipe (l_mfma of sage_attn.hip)
                    lsum = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, sel), __builtin_bit_cast(half8, p), lsum, 0, 0, 0);
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) {
                        const unsigned char* va = vt + (32 * h + 16 * u) * VROW + v_off[dt];
                        const s4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4s*)va);
                        const s4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4s*)(va + 8 * VROW));
                        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                            __builtin_bit_cast(half8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)),
                            __builtin_bit_cast(half8, p), o[dt], 0, 0, 0);
                    }
                }
        };
        const int whole = (seen + 31) / 64;
        auto tiles_seen = [&](auto COARSE) {
            for (int j = kpart; j < whole; j += KSP) tile(j, std::integral_constant<int, 2>{}, COARSE);
            if (whole * 64 < seen && (KSP == 1 || whole % KSP == kpart)) tile(whole, std::integral_constant<int, 1>{}, COARSE);
        };
        if (KSP == 1 || row0 < Nq) {
            if (!KTOK && __builtin_expect(__builtin_amdgcn_ballot_w64(qmax * k_top > 127.0f * 127.0f / SHORT_LOG2E) != 0ull, 0))
                tiles_seen(std::integral_constant<int, 1>{});
            else
                tiles_seen(std::integral_constant<int, 0>{});
        }
        float l = (lane & 16) ? lsum[1] : lsum[0];
        if constexpr (KSP == 2) {
            // the other wavefront's result, relative to its own maximum, through the LDS that held the key tiles
            float* const other = (float*)pool + own * (32 * D) + lane;
            __syncthreads();
            if (kpart == 1) {
                s_ml[own][lane] = m_run;
                s_ml[RT + own][lane] = l;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) other[(16 * dt + r) * 64] = o[dt][r];
            }
            __syncthreads();
            if (kpart == 1 || row0 >= Nq) return;
            const float m1 = s_ml[own][lane], top = __builtin_fmaxf(m_run, m1);
            const float f0 = __builtin_amdgcn_exp2f(m_run - top), f1 = __builtin_amdgcn_exp2f(m1 - top);
            l = __builtin_fmaf(l, f0, s_ml[RT + own][lane] * f1);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] = __builtin_fmaf(o[dt][r], f0, other[(16 * dt + r) * 64] * f1);
        }
        const float inv = 1.0f / l;
        store_rows<D>(og + (slab_q + row0) * D, Nq - row0, lane, true, [&](int dt, int r) { return o[dt][r] * inv; });
        if (KSP == 2) return;
    }
}

template <int D, int NTILE, int NW, bool KTOK>
__global__ void __launch_bounds__(NW * 64, NW == 8 || D == 128 ? 2 : 3)
sage_short_kernel(const _Float16* __restrict__ qf, const _Float16* __restrict__ kf, const _Float16* __restrict__ vf,
                  _Float16* __restrict__ og, int Nq, int N, int shift_q, int shift_k, int causal, float sm_scale, int groups) {
    short_pass<D, NTILE, NW, 1, KTOK>(qf, kf, vf, og, Nq, N, shift_q, shift_k, causal, sm_scale, groups);
}
template <int D, int NTILE, int NW, bool KTOK>
__global__ void __launch_bounds__(NW * 64, 2)
sage_short_pair_kernel(const _Float16* __restrict__ qf, const _Float16* __restrict__ kf, const _Float16* __restrict__ vf,
                       _Float16* __restrict__ og, int Nq, int N, int shift_q, int shift_k, int causal, float sm_scale, int groups) {
    short_pass<D, NTILE, NW, 2, KTOK>(qf, kf, vf, og, Nq, N, shift_q, shift_k, causal, sm_scale, groups);
}

// Key sequences whose K^ and V fit the LDS beside a second workgroup's, or nearly: 512 keys of 64 channels, 256 of 128.
bool short_fits(int N, int D) { return N <= (D == 64 ? 512 : 256); }

// Workgroups per slab: up to one per round of the wavefronts while the chip has room for more workgroups.  (Rounded down:
// 129 to 255 slabs of 256-row workgroups get one each, and leave the CUs between; 129 of 512 keys at D = 64 take 25 us,
// 256 of them 28.)
static int short_groups(int BH, int Nq, int rows, int per_cu) {
    const int most = (Nq + rows - 1) / rows;
    const int room = 256 * per_cu / BH;
    return room < 1 ? 1 : (room < most ? room : most);
}

template <int D, int NTILE, int NW, int KSP = 1>
static hipError_t launch_short_t(const void* q, const void* k, const void* v, void* o, int BH, int Nq, int N, int causal,
                                 float sm_scale, int block_q, int block_k, hipStream_t st) {
    const int groups = KSP == 2 ? (Nq + 127) / 128 : short_groups(BH, Nq, NW * 32, NW == 8 ? 1 : D == 64 ? 3 : 2);
    const int shift_q = __builtin_ctz((unsigned)block_q), shift_k = __builtin_ctz((unsigned)block_k);
    const dim3 grid((unsigned)(BH * groups));
#define SAGE_SHORT(NAME, KT) NAME<D, NTILE, NW, KT><<<grid, NW * 64, 0, st>>>((const _Float16*)q, (const _Float16*)k, (const _Float16*)v, \
        (_Float16*)o, Nq, N, shift_q, shift_k, causal, sm_scale, groups)
    if constexpr (KSP == 2) {
        if (block_k == 1) SAGE_SHORT(sage_short_pair_kernel, true); else SAGE_SHORT(sage_short_pair_kernel, false);
    } else {
        if (block_k == 1) SAGE_SHORT(sage_short_kernel, true); else SAGE_SHORT(sage_short_kernel, false);
    }
#undef SAGE_SHORT
    return hipGetLastError();
}

hipError_t launch_short(const void* q, const void* k, const void* v, void* o, int BH, int Nq, int N, int D, int causal,
                        float sm_scale, int block_q, int block_k, hipStream_t st) {
#define SAGE_SHORT_N(DD, NT, NW) return launch_short_t<DD, NT, NW>(q, k, v, o, BH, Nq, N, causal, sm_scale, block_q, block_k, st)
    if (D == 64) {
        // Two wavefronts per query tile (KSP = 2) where there is a CU for every 128 rows and the chain of key tiles is long
        // enough.  us with one / two: 2 slabs of 300 keys 11.4 / 9.2, 85 of 330 12.6 / 10.7, 60 of 500 14.9 / 13.0, 40 of 230,
        // per token, 9.5 / 8.6, 2 of 256 7.9 / 7.8; with a mask, where half the tiles are left out anyway, 2 of 488 13.2 / 11.0,
        // but 64 of 512 (256 workgroups) 14.0 / 14.5 and 128 of 256 8.2 / 8.7.  Not at D = 128, at most 4 tiles and twice the
        // results to exchange: 64 of 126 8.7 / 10.0, 128 of 256 13.9 / 15.3.
        // The sums are made in another order, each half's weights relative to its own maximum.  Relative error against 64 bits
        // over the same codes, 1e-4, with one / two: 2 slabs of 256 2.78 / 2.71, 60 of 500 2.80 / 2.76, 20 of 400 causal, per
        // token, 2.44 / 2.41; smaller in all of 17 shapes from 197 to 512 keys, six inputs each.
        if (N > 192 && (long)BH * ((Nq + 127) / 128) <= (causal ? 128 : 256)) {
            if (N <= 256) return launch_short_t<64, 4, 8, 2>(q, k, v, o, BH, Nq, N, causal, sm_scale, block_q, block_k, st);
            return launch_short_t<64, 8, 8, 2>(q, k, v, o, BH, Nq, N, causal, sm_scale, block_q, block_k, st);
        }
        if (N <= 128) SAGE_SHORT_N(64, 2, 4);
        if (N <= 256) SAGE_SHORT_N(64, 4, 4);
        SAGE_SHORT_N(64, 8, 8);
    }
    if (N <= 128) SAGE_SHORT_N(128, 2, 4);
    SAGE_SHORT_N(128, 4, 8);
#undef SAGE_SHORT_N
}

}  // namespace sage
