// Which passes of small models run in one launch (kernels_small.h), and how long their workgroups wait: host code only, no HIP.
#pragma once
#include <stddef.h>

namespace ks {

constexpr int SM_NT = 512, SM_NW = SM_NT / 64;   // threads, wavefronts of a workgroup
constexpr int SM_G = 64;                         // workgroups
constexpr int SM_ITEMS = SM_NT / 256 * SM_G;     // (row, head) items of the attention worked on side by side

inline size_t small_stage_floats(int d, int qd, int F, int hd, int mr, int score_len) {
    size_t n = (size_t)mr * (qd > F ? qd : F);
    const size_t attn = SM_NT / 256 * ((size_t)hd + 2 * (size_t)mr * hd + score_len), head = (size_t)3 * SM_G * mr;
    if ((size_t)mr * d > n) n = (size_t)mr * d;
    if (attn > n) n = attn;
    return head > n ? head : n;
}
inline size_t small_lds_bytes(int d, int qd, int F, int hd, int mr, int score_len) {
    return ((size_t)mr * d + small_stage_floats(d, qd, F, hd, mr, score_len)) * 4;
}

// How long a workgroup waits for a word before it gives the launch up, in ticks of the 100 MHz clock. The products of a step are
// bounded by the size of a small model's matrices, some tens of microseconds at most; 360 us are far beyond. The attention is
// bounded by the context: an item is a chain of dependent rounds over the keys and as many over the values, 256 threads at four
// positions each a round, and where there are more items than SM_ITEMS a workgroup takes several of them one after the other
// while the others wait. A round takes 0.9-1.1 us (reductions, LDS, loads out of the L2 or from memory); 2.5 are allowed for it. (Counted
// in looks, the wait was no bound on time: a look takes 0.7 us or less than 0.2, and a head of 128 over 6000 positions, 0.4 ms,
// broke up every pass of one or two rows with nobody else on the GPU.)
inline int small_wait(int n_heads, int head_dim, int n_rows, int len) {
    const int per_round = 4 * 256 / (head_dim / 4), rounds = 2 * ((len + per_round - 1) / per_round);
    return 36000 + 250 * rounds * ((n_heads * n_rows + SM_ITEMS - 1) / SM_ITEMS);
}

}  // namespace ks
