// A whole pass of a small model (any shape, fp32 or bf16 storage) in ONE launch, for gfx950.
//
// What bounds it: a small model's pass is a chain of dependent products, each far smaller than what a launch costs: 4-5 us
// per step as launches (two or three round trips to the L2, 1 us between kernels), five steps per block. Here SM_G
// workgroups stay for the whole pass and hand the vectors over themselves. A value travels as an 8-byte word {value, tag of the
// step}, written and read with agent-scope accesses of that size: whoever reads the word with the right tag has the
// value, so a step costs one store and one load through memory (0.7-0.8 us), no counter, no barrier, no fence.
// Measured: a draft step of the fp32 configuration (two of four blocks of d = 256) 62 us as launches, 31-32 us here, its 5-row
// verification 118 -> 74 us, the whole generation (prompt 32, 32 tokens, rounds of four drafts) 9.7-10.3 -> 7.0-7.1 ms. A step of a block is
// now 0.7 us of hand-over and 1.1-1.8 us of products or attention, bound by dependent latencies: the operands' way from the
// L2, the reduction, square root and division. (32 workgroups: 25 % slower, 48: 4 %; 128: no faster. 1024 threads: spills.)
//
// Nobody may overwrite a word that somebody has yet to read. A step's words are written again one block later at the
// earliest, and its writers have then read outputs of steps in between to which EVERY workgroup contributes at least
// one value after it has read the words in question (small_ok: no more workgroups than rotary pairs and value pairs or
// SwiGLU features, dealt to workgroups first, wavefronts second). Tags differ between all steps of all launches
// (knnssd_ctx::small_tag).
//
// Workgroups that wait for each other have to be resident together. Nothing guarantees that where many launches share the
// GPU, so nothing relies on it: a workgroup that has waited for a word for SmallArgs::wait declares the launch broken up
// (SmallMeet::state) and leaves; the last one to leave then runs the whole pass by itself, as a launch of one workgroup, which waits
// for nobody. Once the first workgroup has declared the pass done, nobody can break it up.
// What a broken launch leaves behind is what the workgroup that stayed has stored: its own die's L2 holds those lines, and the L2 of
// another die may hold lines of the same cache entries, logits or hidden state that a departed workgroup wrote earlier;
// which of the two reaches memory last is not defined. So a workgroup that has given up stores nothing but handed-over words, and
// those marked (SM_BAD_TAG). Whatever was stored before has been worked out from sound inputs and is the same bytes.
//
// The arithmetic is that of gemm_rows_kernel, attention_kernel and rmsnorm_kernel, operation for operation (the same
// device code), and that of argmax_classes_kernel, so a row's logits and probability do not depend on which of the two ways a pass
// takes, nor on whether a launch was broken up.
#pragma once
#include "kernels_generic.h"
#include "small_plan.h"

namespace ks {

typedef unsigned long long u64;

constexpr int SM_MAX_BLOCKS = 64;                // skip masks travel as launch arguments
constexpr unsigned int SM_BAD_TAG = 0x80000000u; // marks the words of a workgroup that has given up
constexpr int SM_MEETS = 8;                      // launches whose SmallMeet are kept apart
enum { MEET_OPEN = 0, MEET_BROKEN, MEET_DONE };
struct SmallMeet { int state, left; };           // how a launch stands, workgroups that have left it

struct SmallBlock {              // addresses as numbers: see as_global
    uint64_t attn_norm, mlp_norm, wqkv, wo, wgu, wdown;
};

struct SmallArgs {
    PassCtl *ctl;
    PassEnds ends;
    const SmallBlock *blocks;
    int n_blocks;
    u64 skip_attn, skip_mlp;     // bit b: block b's sublayer is skipped
    const void *embed, *lm_head;
    const float *final_norm;
    char *kv;
    size_t kv_block_bytes;
    u64 *w_qkv, *w_att, *w_xo, *w_u, *w_xd, *w_head;     // handed-over vectors: [row][feature]
    float *xn, *logits;
    HeadResult *head;
    SmallMeet *meets;            // [SM_MEETS]
    int launch;                  // which of them is this launch's
    const float *cos_t, *sin_t;
    int d, H, Hkv, hd, F, V, max_seq;
    float eps;
    unsigned int tag;            // first tag of the launch
    int one_head;                // the LM head sees one row at most
    int score_len;               // attention scores: floats per item
    int *flags;                  // host words, [3]: launches that were broken up, [4]: a workgroup has waited in vain for its own words
    int wait;                    // small_wait
    int quit_wg, quit_block;     // for tests: this workgroup (SM_G: every one, SM_G + 1: also the one left alone) gives up at its first wait from this block on
};

// weight pieces of an output product requested ahead, 1 KB of a row each
constexpr int small_pieces(int mr) { return mr <= 6 ? 3 : 1; }
// tags a pass takes: five steps per block and the head
inline unsigned int small_tags(int n_blocks) { return 5u * (unsigned int)n_blocks + 1u; }
// gave_up: the value is worth nothing
__device__ __forceinline__ void word_put(u64 *p, float v, unsigned int tag, int gave_up) {
    if (gave_up) tag |= SM_BAD_TAG;
    __hip_atomic_store(p, ((u64)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 word_get(const u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Words 0..n-1 by threads tid of nt: at(i) is a word's address, put(i, value) receives its value. U words per thread are
// looked at together. A wait that is given up, after `wait` ticks of the 100 MHz clock, leaves a mark (gave_up, in LDS), after which the
// workgroup waits no more. wait = 0: it is given up whatever is there.
template <int U, typename FA, typename FP>
__device__ __forceinline__ void words_read(int n, int tid, int nt, unsigned int tag, int &gave_up, int wait, FA at, FP put) {
    const int limit = gave_up ? 0 : wait;     // (after that it goes through the motions)
    for (int i0 = tid; i0 < n; i0 += nt * U) {
        u64 v[U], until = 0;
        int look = 0;
        bool all, more = limit > 0;
        do {
            all = true;
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = word_get(at((unsigned int)min(i0 + u * nt, n - 1)));
#pragma unroll
            for (int u = 0; u < U; ++u) all = all && (unsigned int)(v[u] >> 32) == tag;
            if (!all && (++look & 15) == 0) {             // the clock, now and then
                const u64 now = wall_clock64();
                if (until == 0) until = now + limit;
                more = more && now < until;
            }
        } while (!all && more);
        if (!all || wait == 0) gave_up = 1;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u == 0 || i0 + u * nt < n) put(i0 + u * nt, __uint_as_float((unsigned int)v[u]));
    }
}

// An address that was read from memory as a pointer the compiler knows to be a global one (of a plain pointer out of memory it
// does not know that, and takes loads that wait for the LDS unit as well).
template <typename T> __device__ __forceinline__ const T *as_global(uint64_t address) {
    return (const T *)(const __attribute__((address_space(1))) T *)address;
}

__device__ __forceinline__ float as_stored(float v, float) { return v; }
__device__ __forceinline__ float as_stored(float v, bf16_t) { return bf16_to_float(float_to_bf16_rne(v)); }

struct SmallLds {
    AttnItemLds att[SM_NT / 256];
    float part[SM_NT / 256][4];
    float hm[SM_NW][KS_MAX_ROWS], hs[SM_NW][KS_MAX_ROWS];
    int hi[SM_NW][KS_MAX_ROWS];
    PassCtl ctl;
    HeadResult head;
    int gave_up, done, alone;
};

// The workgroup takes (row, head) items side by side, 256 threads each.
template <typename T, int MR, int HD>
__device__ __forceinline__ void small_attention(const SmallArgs &a, SmallLds &sl, float *st, const T *kvb, int n_rows, int start, int n_wg, int wg,
                                                unsigned int tag, int wait) {
    int thread = threadIdx.x;
    asm volatile("" : "+v"(thread));
    const int part = thread >> 8, tid = thread & 255, d0 = (tid % (HD / 4)) * 4;
    const u64 *const w_qkv = a.w_qkv;
    u64 *const w_att = a.w_att;
    const int H = a.H, Hkv = a.Hkv, items = H * n_rows;
    float *q = st + part * (HD + 2 * MR * HD + a.score_len), *kn = q + HD, *vn = kn + MR * HD, *scores = vn + MR * HD;
    for (int base = wg; base < items; base += SM_NT / 256 * n_wg) {
        const int it = min(base + part * n_wg, items - 1);
        const bool live = base + part * n_wg < items;
        const int h = it / n_rows, r = it - h * n_rows, kvh = h / (H / Hkv), len = start + r + 1;
        // what the cache holds is requested before the pass's own rows are waited for
        const T *kc = kvb + (size_t)kvh * a.max_seq * HD + d0, *vc = kvb + ((size_t)Hkv + kvh) * a.max_seq * HD + d0;
        auto old = [&](const T *cache, int t) { return load4_as_float(cache + (size_t)min(t, max(start - 1, 0)) * HD); };
        auto now = [&](const float *fresh, float4 o, int t) {      // the pass's own row, if position t is one
            const float4 n = *reinterpret_cast<const float4 *>(fresh + max(t - start, 0) * HD + d0);
            return t < start ? o : n;
        };
        float4 k0[ATI_U], v0[ATI_U];
#pragma unroll
        for (int u = 0; u < ATI_U; ++u) k0[u] = old(kc, attention_position<HD>(tid, u, len));
#pragma unroll
        for (int u = 0; u < ATI_U; ++u) v0[u] = old(vc, attention_position<HD>(tid, u, len));
        // the query, and the keys and values of the pass's own rows
        const int qkvd = (H + 2 * Hkv) * HD, own = HD * (r + 1);
        const unsigned int qo = r * qkvd + h * HD, ko = (H + kvh) * HD, vo = ko + Hkv * HD;
        words_read<4>(HD + 2 * own, tid, 256, tag, sl.gave_up, wait,
                   [=](unsigned int i) {
                       const unsigned int j = i < HD ? i : (i < HD + own ? i - HD : i - HD - own);
                       const unsigned int kv = i < HD + own ? +ko : +vo;       // (values: a choice between the captured variables would put them in memory)
                       return w_qkv + ((i < HD ? +qo : kv + j / HD * qkvd) + j % HD);
                   },
                   [&](int i, float v) {
                       if (i < HD) q[i] = v;
                       else if (i < HD + own) kn[i - HD] = v;
                       else vn[i - HD - own] = v;
                   });
        __syncthreads();
#pragma unroll
        for (int u = 0; u < ATI_U; ++u) {
            k0[u] = now(kn, k0[u], attention_position<HD>(tid, u, len));
            v0[u] = now(vn, v0[u], attention_position<HD>(tid, u, len));
        }
        attention_item<HD>(*reinterpret_cast<const float4 *>(q + d0), len, tid, scores, sl.att[part], k0, v0, [&](int t) { return now(kn, old(kc, t), t); },
                           [&](int t) { return now(vn, old(vc, t), t); },
                           [&](int dim, float v) { if (live) word_put(w_att + (size_t)r * H * HD + h * HD + dim, v, tag + 1, sl.gave_up); });
        __syncthreads();       // the next item's operands may overwrite this one's
    }
}

// The end of a pass that ran alone. One that has given up (it reads nothing but its own words, so this means that something is badly wrong)
// has no result: the host finds the word and fails the call.
// It is counted before the pass tells the host that it is over (pass_end): a host that sees a pass's number holds the next ones back.
__device__ __forceinline__ void small_alone(const SmallArgs &a, int gave_up) {
    ++a.flags[3];
    if (gave_up) a.flags[4] = 1;
    __threadfence_system();
}

// T: storage type of weights and cache; MR: rows the build holds (the pass has n_rows <= MR)
template <typename T, int MR>
__global__ __launch_bounds__(SM_NT) void small_pass_kernel(SmallArgs a) {
    extern __shared__ __align__(16) char lds_bytes[];
    float *lds = reinterpret_cast<float *>(lds_bytes);
    __shared__ SmallLds sl;
    int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wg = blockIdx.x;
    if (wg == 0 && tid == 0) a.meets[(a.launch + SM_MEETS / 2) % SM_MEETS] = SmallMeet{MEET_OPEN, 0};     // for a later launch
    SmallMeet *const meet = a.meets + a.launch;
    // (the state that a verification is taken from changes when the whole pass is over)
    const PassCtl *ctl = pass_begin(a.ends, a.ctl, &sl.ctl);
    if (!ctl->active) {
        if (wg == 0 && tid == 0) pass_end(a.ends, a.ctl, ctl, a.head);
        return;
    }
    const int n_rows = min(ctl->n_rows, MR), start = ctl->start, head_from = ctl->head_from;
    int n_wg = SM_G;                                   // 1: the pass of a launch that was broken up
    for (;;) {
    int gw = wave * n_wg + wg;                         // workgroups first: see above
    const int NW = n_wg * SM_NW;
    int wait = n_wg == 1 ? 100000000 : a.wait;         // (alone, only its own words can be on their way)
    const int quit_from = (n_wg == 1 ? a.quit_wg > SM_G : a.quit_wg >= SM_G || a.quit_wg == wg) ? a.quit_block : SM_MAX_BLOCKS + 1;
    const int d = a.d, hd = a.hd, half = hd >> 1, qd = a.H * hd, qkvd = (a.H + 2 * a.Hkv) * hd;
    float *xs = lds, *st = lds + (size_t)MR * d;       // residual stream; the input of a step
    if (tid == 0) sl.gave_up = 0;
    for (int i = tid; i < n_rows * d; i += SM_NT) {
        const int r = i / d, c = i - r * d;
        xs[i] = load_as_float(reinterpret_cast<const T *>(a.embed) + (size_t)ctl->tok[r] * d, c);
    }
    __syncthreads();

    // a handed-over vector of n features per row into LDS rows of n floats
    auto gather = [&](const u64 *w, int n, float *to, unsigned int tag) {
        __syncthreads();                               // everybody is done with what lies there
        const int count = n * n_rows;
        auto at = [&](unsigned int i) { return w + i; };
        auto put = [&](int i, float v) { to[i] = v; };
        if (count <= SM_NT) words_read<1>(count, tid, SM_NT, tag, sl.gave_up, wait, at, put);
        else words_read<4>(count, tid, SM_NT, tag, sl.gave_up, wait, at, put);
        __syncthreads();
    };
    // A step's first weights are requested before its input is waited for, an item's while the item before is computed.
    static_assert(SM_G == HEAD_GROUPS && SM_NW == HEAD_WAVES, "the head's classes");
    constexpr int NP = small_pieces(MR), IT = MR <= 6 ? 2 : 1;     // items a wavefront works on side by side
    // output product + residual
    auto residual = [&](const T *W, const u64 *in, int K, unsigned int tag_in, u64 *out) {
        if (wg < d) {                                  // this workgroup owns features
            RowsPieces<T, false, NP> next;
            next.load(W + (size_t)min(gw, d - 1) * K, nullptr, nullptr, K);
            gather(in, K, st, tag_in);
            for (int o = gw; o < d; o += NW) {
                float v, unused;
                const RowsPieces<T, false, NP> p = next;
                if (o + NW < d) next.load(W + (size_t)(o + NW) * K, nullptr, nullptr, K);
                rows_product<T, MR, false, false, NP>(p, W + (size_t)o * K, nullptr, st, K, n_rows, K, nullptr, a.eps, v, unused);
                if (lane < n_rows) word_put(out + (size_t)lane * d + o, xs[(size_t)lane * d + o] + v, tag_in + 1, sl.gave_up);
            }
        }
    };
    const u64 *x_words = a.w_xo;                       // the residual stream, where it has moved on to
    unsigned int x_tag = 0;                            // 0: xs holds it
    const int P = (a.H + a.Hkv) * half, items = P + a.Hkv * half, head_shift = hd == 128 ? 7 : 6, half_shift = head_shift - 1;
    for (int b = 0; b < a.n_blocks; ++b) {
        const SmallBlock blk = a.blocks[b];
        asm volatile("" : "+v"(tid), "+v"(lane), "+v"(gw));       // addresses are worked out where they are used, not kept over the blocks
        if (b >= quit_from) wait = 0;
        const float *attn_norm = as_global<float>(blk.attn_norm), *mlp_norm = as_global<float>(blk.mlp_norm);
        const unsigned int tag = a.tag + 5u * b;
        if (!((a.skip_attn >> b) & 1)) {
            T *kvb = reinterpret_cast<T *>(a.kv + (size_t)b * a.kv_block_bytes), *kc = kvb, *vc = kvb + (size_t)a.Hkv * a.max_seq * hd;
            const T *W = as_global<T>(blk.wqkv);
            // rotary pairs, then pairs of value rows
            auto row0 = [&](int o) { return o < P ? ((o >> half_shift) << head_shift) + (o & (half - 1)) : ((a.H + a.Hkv) << head_shift) + (o - P) * 2; };
            auto row1 = [&](int o) { return row0(o) + (o < P ? half : 1); };
            RowsPieces<T, true, 1> next;
            const int o0 = min(gw, items - 1);
            next.load(W + (size_t)row0(o0) * d, W + (size_t)row1(o0) * d, attn_norm, d);
            if (x_tag) gather(x_words, d, xs, x_tag);
            const int pos = start + min(lane, n_rows - 1);
            float rope_c = a.cos_t[(size_t)pos * half + (gw & (half - 1))], rope_s = a.sin_t[(size_t)pos * half + (gw & (half - 1))];
            for (int o = gw; o < items; o += NW) {
                const int r0 = row0(o), r1 = row1(o), i = o & (half - 1);
                const RowsPieces<T, true, 1> p = next;
                if (o + NW < items) next.load(W + (size_t)row0(o + NW) * d, W + (size_t)row1(o + NW) * d, attn_norm, d);
                if (o != gw) { rope_c = a.cos_t[(size_t)pos * half + i]; rope_s = a.sin_t[(size_t)pos * half + i]; }
                const float c = rope_c, s = rope_s;
                float v0, v1;
                rows_product<T, MR, true, true, 1>(p, W + (size_t)r0 * d, W + (size_t)r1 * d, xs, d, n_rows, d, attn_norm, a.eps, v0, v1);
                if (lane < n_rows) {
                    if (o < P) {
                        const int head = o >> half_shift;
                        float ra, rb;
                        rotate_pair(v0, v1, c, s, ra, rb);
                        if (head >= a.H) {
                            const size_t base = ((size_t)(head - a.H) * a.max_seq + pos) * hd;
                            if (!sl.gave_up) {         // what a workgroup that has given up works out is stored nowhere
                                store_rounded(kc, base + i, ra);
                                store_rounded(kc, base + i + half, rb);
                            }
                            ra = as_stored(ra, T()); rb = as_stored(rb, T());
                        }
                        v0 = ra; v1 = rb;
                    } else {
                        const int v = (o - P) * 2;
                        const size_t base = ((size_t)(v >> head_shift) * a.max_seq + pos) * hd + (v & (hd - 1));
                        if (!sl.gave_up) {
                            store_rounded(vc, base, v0);
                            store_rounded(vc, base + 1, v1);
                        }
                        v0 = as_stored(v0, T()); v1 = as_stored(v1, T());
                    }
                    word_put(a.w_qkv + (size_t)lane * qkvd + r0, v0, tag, sl.gave_up);
                    word_put(a.w_qkv + (size_t)lane * qkvd + r1, v1, tag, sl.gave_up);
                }
            }
            if (hd == 128) small_attention<T, MR, 128>(a, sl, st, kvb, n_rows, start, n_wg, wg, tag, wait);
            else small_attention<T, MR, 64>(a, sl, st, kvb, n_rows, start, n_wg, wg, tag, wait);
            residual(as_global<T>(blk.wo), a.w_att, qd, tag + 1, a.w_xo);
            x_words = a.w_xo;
            x_tag = tag + 2;
        }
        if (!((a.skip_mlp >> b) & 1)) {
            const T *W = as_global<T>(blk.wgu), *W2 = W + (size_t)a.F * d;
            RowsPieces<T, true, 1> p[IT];
#pragma unroll
            for (int j = 0; j < IT; ++j) p[j].load(W + (size_t)min(gw + j * NW, a.F - 1) * d, W2 + (size_t)min(gw + j * NW, a.F - 1) * d, mlp_norm, d);
            if (x_tag) gather(x_words, d, xs, x_tag);
            for (int o = gw; o < a.F; o += IT * NW) {
                float g[IT], u[IT];
#pragma unroll
                for (int j = 0; j < IT; ++j) {
                    const size_t f = (size_t)min(o + j * NW, a.F - 1) * d;
                    if (o != gw) p[j].load(W + f, W2 + f, mlp_norm, d);
                    rows_product<T, MR, true, true, 1>(p[j], W + f, W2 + f, xs, d, n_rows, d, mlp_norm, a.eps, g[j], u[j]);
                }
#pragma unroll
                for (int j = 0; j < IT; ++j)
                    if (lane < n_rows && o + j * NW < a.F) word_put(a.w_u + (size_t)lane * a.F + o + j * NW, (g[j] / (1.0f + expf(-g[j]))) * u[j], tag + 3, sl.gave_up);
            }
            residual(as_global<T>(blk.wdown), a.w_u, a.F, tag + 3, a.w_xd);
            x_words = a.w_xd;
            x_tag = tag + 4;
        }
    }
    asm volatile("" : "+v"(tid), "+v"(lane), "+v"(gw), "+v"(wave));
    const int n_head = n_rows - head_from;
    if (a.n_blocks >= quit_from) wait = 0;
    if (n_head > 0) {
    const T *W = reinterpret_cast<const T *>(a.lm_head);
    RowsPieces<T, false, 1> p[IT];
    const int c0 = wave * SM_G + wg;                   // the wavefront's (first) class of tokens
#pragma unroll
    for (int j = 0; j < IT; ++j) p[j].load(W + (size_t)min(c0 + j * HEAD_CLASSES, a.V - 1) * d, nullptr, nullptr, d);
    if (x_tag) gather(x_words, d, xs, x_tag);
    // final norm, a row per 256 threads
    {
        const int hf = tid >> 8, t = tid & 255;
        for (int base = 0; base < n_head; base += SM_NT / 256) {
            const int rr = min(base + hf, n_head - 1);
            const float *xr = xs + (size_t)(head_from + rr) * d;
            float ss = 0.f;
            for (int i = t; i < d; i += 256) ss = fmaf(xr[i], xr[i], ss);
            ss = wave_sum(ss);
            if (lane == 0) sl.part[hf][wave & 3] = ss;
            __syncthreads();
            const float tot = (sl.part[hf][0] + sl.part[hf][1]) + (sl.part[hf][2] + sl.part[hf][3]);
            const float rs = 1.0f / sqrtf(tot / (float)d + a.eps);
            for (int i = t; i < d; i += 256) {
                const float v = xr[i] * rs * a.final_norm[i];
                st[(size_t)rr * d + i] = v;
                if (wg == 0 && !sl.gave_up) a.xn[(size_t)(head_from + rr) * d + i] = v;
            }
            __syncthreads();
        }
    }
    // LM head: lane r keeps row r's largest logit so far and its sum of exponentials. Alone, the workgroup takes the others' classes one
    // after the other, so that the sums are formed as everybody together forms them.
    const unsigned int tag = a.tag + 5u * a.n_blocks;
    for (int g = wg; g < SM_G; g += n_wg) {
    const int c = wave * SM_G + g;
    float m = -INFINITY, s = 0.f;
    int mi = 0x7fffffff;
    for (int o0 = c; o0 < a.V; o0 += IT * HEAD_CLASSES) {
        float v[IT], unused;
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const T *w = W + (size_t)min(o0 + j * HEAD_CLASSES, a.V - 1) * d;
            if (o0 != c0) p[j].load(w, nullptr, nullptr, d);
            if (a.one_head) rows_product<T, 1, false, false, 1>(p[j], w, nullptr, st, d, 1, d, nullptr, a.eps, v[j], unused);
            else rows_product<T, MR, false, false, 1>(p[j], w, nullptr, st, d, n_head, d, nullptr, a.eps, v[j], unused);
        }
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int o = o0 + j * HEAD_CLASSES;
            if (lane < n_head && o < a.V) {
                if (!sl.gave_up) a.logits[(size_t)(head_from + lane) * a.V + o] = v[j];
                head_fold(v[j], o, m, s, mi);
            }
        }
    }
    if (lane < n_head) { sl.hm[wave][lane] = m; sl.hs[wave][lane] = s; sl.hi[wave][lane] = mi; }
    __syncthreads();
    if (tid < n_head) {
        float bm, sum;
        int bi;
        head_join(&sl.hm[0][tid], &sl.hs[0][tid], &sl.hi[0][tid], KS_MAX_ROWS, bm, bi, sum);
        u64 *o = a.w_head + ((size_t)tid * SM_G + g) * 3;      // [row][workgroup]
        word_put(o, bm, tag, sl.gave_up);
        word_put(o + 1, __uint_as_float((unsigned int)bi), tag, sl.gave_up);
        word_put(o + 2, sum, tag, sl.gave_up);
    }
    if (n_wg == 1) __syncthreads();                    // the next classes overwrite these
    }
    if (wg == 0) {
    // the workgroups' shares, a lane each
    static_assert(SM_G == 64, "a lane per workgroup");
    words_read<4>(3 * SM_G * n_head, tid, SM_NT, tag, sl.gave_up, wait, [&](unsigned int i) { return a.w_head + i; }, [&](int i, float v) { st[i] = v; });
    __syncthreads();
    if (tid == 0) {
        // from here on the launch cannot be broken up (alone it is not: nobody else is left)
        int open = MEET_OPEN;
        sl.done = n_wg == 1 || (!sl.gave_up && __hip_atomic_compare_exchange_strong(&meet->state, &open, MEET_DONE, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    __syncthreads();
    if (sl.done) {
        for (int r = wave; r < n_head; r += SM_NW) {
            const float *p = st + ((size_t)r * SM_G + lane) * 3;
            int token;
            float prob;
            head_merge(p[0], (int)__float_as_uint(p[1]), p[2], token, prob);
            if (lane == 0) {
                a.head->tok[head_from + r] = sl.head.tok[head_from + r] = token;
                a.head->prob[head_from + r] = sl.head.prob[head_from + r] = prob;
            }
        }
        __syncthreads();
        if (tid == 0) {
            if (n_wg == 1) small_alone(a, sl.gave_up);
            if (!sl.gave_up) pass_end(a.ends, a.ctl, ctl, &sl.head);
            if (n_wg != 1) __hip_atomic_fetch_add(&meet->left, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    }
    }
    if (n_wg == 1) {                                   // (a pass without a head)
        if (tid == 0) small_alone(a, sl.gave_up);
        return;
    }
    // leave; the last one of a launch that was broken up stays for the whole pass
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the words this workgroup has handed over are where everybody looks for them
    __syncthreads();
    if (tid == 0) {
        int open = MEET_OPEN;
        if (sl.gave_up) __hip_atomic_compare_exchange_strong(&meet->state, &open, MEET_BROKEN, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // in this order
        const bool last = __hip_atomic_fetch_add(&meet->left, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == SM_G - 1;
        sl.alone = last && __hip_atomic_load(&meet->state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == MEET_BROKEN;
        sl.gave_up = 0;
    }
    __syncthreads();
    if (!sl.alone) return;
    n_wg = 1;
    wg = 0;
    }
}

}  // namespace ks
