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

// A workgroup takes its (row, head) items in turns, and an item is a chain of dependent rounds over the keys and as many over the values,
// 256 threads at four positions each a round.
inline int small_rounds(int head_dim, int len) {
    const int per_round = 4 * 256 / (head_dim / 4);
    return 2 * ((len + per_round - 1) / per_round);
}

// Is a pass faster in one launch? It saves what launches cost, five per block and six around them, but its attention is slower: items
// are spread over SM_G workgroups, a launch of their own spreads them over the chip, and a round takes 0.9-1.1 us here and
// 0.6-0.8 there. So the context decides, by the rounds that follow one another in a block, against a limit that the launches around the
// blocks raise where few of them hold attention. The form was fitted to 1840 pairs of timings (1 to 12 blocks, 2 to 32 heads of 64 and
// 128, 1 to 16 rows, contexts 30 to 1400; draft steps and verifications as calls and inside generations): the way chosen
// is 0.9 % slower than the better one in the mean; one launch always 8.7 % (twice the time at worst), never 15 %. For instance, launches / one
// launch, GPU us: four blocks, fp32, four heads of 64, a draft step 87 / 55 at context 30, 96 / 74 at 250, 115 / 116 at
// 600, 179 / 215 at 1400; 5 rows 89 / 75, 101 / 96, 130 / 142, 191 / 235; sixteen heads, 5 rows 95 / 87, 107 / 115. bf16 with 12
// rows, which take the build for 16, is never faster: 126 / 127, 144 / 146, 97 / 110.
inline bool small_faster(int n_heads, int head_dim, bool bf16, int n_attn, int n_rows, int len) {
    if (bf16 && n_rows == 12) return false;
    const int groups = (n_heads * n_rows + SM_G - 1) / SM_G;                // items a workgroup has, two of them side by side
    const long weight = 40 + (n_rows - 1) + 60 * (groups - 1);              // of a round, in fortieths
    return (long)small_rounds(head_dim, len) * weight * n_attn <= 40L * ((bf16 ? 20 : 12) * n_attn + 32);
}

// One launch, or launches for a while because one was broken up? On a GPU that others keep busy the next one would be broken up too, and
// that costs the wait and a pass on one workgroup: 1.0 ms for a draft step of the fp32 configuration and 1.4 ms for 5 rows, where launches
// take 0.09-0.12 ms and one whole launch 0.03-0.07. So the next SM_HOLD passes run as launches, and each time that the first
// one-launch passes afterwards are broken up again, twice as many, up to SM_HOLD_MAX. (Never going back would give up a third to a
// half of each pass for one disturbance.)
constexpr int SM_HOLD = 64, SM_HOLD_MAX = 1024;
struct SmallHold {
    int seen = 0;       // broken launches known of
    int length = 0;     // passes held back the last time
    int left = 0;       // ... still to come
    int whole = 0;      // one-launch passes since then
    // asked once per pass; broken: launches broken up so far
    bool hold(int broken) {
        if (broken != seen) {
            seen = broken;
            if (left == 0) {           // (those enqueued with it tell nothing new)
                length = length == 0 || whole > length ? SM_HOLD : (2 * length < SM_HOLD_MAX ? 2 * length : SM_HOLD_MAX);
                left = length;
                whole = 0;
            }
        }
        if (left > 0) { --left; return true; }
        ++whole;
        return false;
    }
};

// How long a workgroup waits for a word before it gives the launch up, in ticks of the 100 MHz clock. The products of a step are
// bounded by the size of a small model's matrices, some tens of microseconds at most; 360 us are far beyond. The attention is
// bounded by the context: where there are more items than SM_ITEMS a workgroup takes several of them one after the other while the
// others wait. A round takes 0.9-1.1 us (reductions, LDS, loads out of the L2 or from memory); 2.5 are allowed for it. (Counted
// in looks, the wait was no bound on time: a look takes 0.7 us or less than 0.2, and a head of 128 over 6000 positions, 0.4 ms,
// broke up every pass of one or two rows with nobody else on the GPU.)
inline int small_wait(int n_heads, int head_dim, int n_rows, int len) {
    return 36000 + 250 * small_rounds(head_dim, len) * ((n_heads * n_rows + SM_ITEMS - 1) / SM_ITEMS);
}

}  // namespace ks
