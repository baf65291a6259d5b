// Which workgroups a launch of the attention kernel (sage_attn.hip) is made of.  Host code without HIP, so that a test can ask it.
#pragma once

namespace sage {

// D = 64: 128-row workgroups, three per CU.  D = 128: 128-row ones, two per CU, or 256-row ones (8 wavefronts sharing one
// set of LDS tiles), one per CU; a row's bits do not depend on which.  us below are with 128 / 256 rows.
// Short sequences, to 2048 keys, 4096 with a mask: 128 rows.  A workgroup visits few tiles, and the independent progress of
// the small ones and the finer causal staircase matter more than the sharing.  No mask: 4096 queries of 128 slabs against
// 200 keys 83 / 98, against 800 196 / 208; 90 slabs of 1000 47 / 56, 60 of 2000 106 / 103.  Causal: 128 slabs of 1536 keys
// 77 / 81, of 3000 259 / 264, of 4096 441 / 449, 64 of 4096 219 / 217; with one scale per key 83 / 88, 287 / 288,
// 494 / 499, 244 / 243.
// Longer, causal: 256 rows where there are two of them per CU; with fewer the launch is the chain of its heaviest tile (16
// slabs of 5000 93 / 104).
// Longer, no mask: a 256-row workgroup takes 3-5 % less than two 128-row ones side by side, but a 128-row one that has its
// CU to itself 0.74 of that time.  So the smaller ones where their last round over the 512 places is at most half full
// and no more than five full ones are before it (12 slabs of 6000, 564 of them: 207 / 245; 30 of 3000, 720: 115 / 132;
// 86 of 4096, 2752: 567 / 579) and where rows that are no multiple of 256 cost the larger ones a round more (480 against
// 288 for 96 chunks of 2816 keys and 640 queries: 92 / 117), the larger ones elsewhere (12 of 3000, 288: 64 / 58; 46 of
// 3800, 1380: 281 / 268; one scale per key, 20 of 6000, 940: 328 / 315).
// Chunks of the keys under a mask (a chunk of a prompt, where the mask takes little of any workgroup): as without one, if the
// rows fill as many halves of 256-row tiles as 128-row ones: 32 slabs of 512 rows against 16384 keys 111.9 / 107.6, 20 of
// 1000 against 20000 167 / 159, 13 of 130 against 40000 56.5 / 53.7, with one scale per key 50 of 500 against 6000 84.1 / 78.0;
// 40 of 640 against 12000 (5 tiles or 3) 137 / 139.
// BH slabs of Nq queries; N keys per slab, walked whole (n_splits = 1) or in n_splits chunks.  True: 128 rows.
inline bool small_workgroups(int D, int BH, int Nq, int N, bool causal, int n_splits, int chunk) {
    const bool staircase = causal && n_splits == 1;
    const int n_seen = n_splits > 1 ? chunk : N;           // keys a workgroup walks
    if (D != 128 || n_seen <= (staircase ? 4096 : 2048)) return true;
    const int small_tiles = (Nq + 127) / 128, large_tiles = (Nq + 255) / 256;
    const long units = (long)BH * n_splits;
    if (staircase) return units * large_tiles < 2 * 256;
    if (causal && 2 * large_tiles != small_tiles) return true;
    const long rounds = (units * small_tiles + 511) / 512, last = units * small_tiles - 512 * (rounds - 1);
    return (last <= 256 && rounds <= 6) || (units * large_tiles + 255) / 256 > rounds;
}

// Whether the 128-row workgroups of a launch are made of two sets of 4 wavefronts, each with half of the keys (HALVES in
// sage_attn.hip): where a CU has one of them at most, and with it one wavefront per SIMD.  us of the attention call with one /
// two sets, D = 64: 1 slab of 1024 11.9 / 11.1, 32 of 1024 13.9 / 13.8, causal 13.4 / 13.2, 16 of 2048 22.9 / 21.7, causal 21.9 /
// 19.9, 8 of 4096 39.4 / 36.2, causal 38.4 / 32.3, 1 of 6000 54.3 / 43.0; with one scale per key 32 of 1024 16.4 / 14.9; whole
// pass, 1 slab of 20000 183 / 154.  With fewer keys the merge and the rows that see the first set's keys alone cost more than the
// shorter chain saves: 36 of 800 12.3 / 12.3, 51 of 600 causal 10.2 / 12.2, 85 of 300 7.5 / 8.3.
// The sums of two sets are added in another order than one set's: at D = 64 the last bits of a row depend on whether the call
// has few slabs.  Not so at D = 128, where the rule above counts on it that a row's bits do not depend on the shape.
inline bool two_halves(int D, int BH, int Nq, int N, int n_splits) {
    return D == 64 && n_splits == 1 && N >= 1024 && (long)BH * ((Nq + 127) / 128) <= 256;
}

}  // namespace sage
