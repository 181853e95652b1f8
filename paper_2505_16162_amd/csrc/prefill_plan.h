// How the prompt prefill cuts its products into workgroups: plain code, no HIP.
#pragma once
#include <stddef.h>

#include "../../include/knnssd.h"
#include "device_types.h"

#ifdef __HIPCC__
#define KS_HD __host__ __device__
#else
#define KS_HD
#endif

namespace ks {

enum { PF_QKV = 0, PF_O, PF_GU, PF_DOWN, PF_OPS };     // the four matrices of a block

// What becomes of the sums: stored as they are (a K part, or a row kernel finishes them anyway), SwiGLU, or RoPE + cache.
// (A build per kind: a workgroup's fixed cost is largely its instructions in front of the first load and the fetch of those
// behind the loop, 4-5 us with everything in one build.)
enum { PF_PARTS = 0, PF_SWIGLU, PF_ROPE };

// Equal runs of n units for G workgroups: the first unit of run w (w = G: n), and the run that unit u belongs to
KS_HD inline int pf_share(int n, int G, int w) { return (int)((unsigned int)n * (unsigned int)w / (unsigned int)G); }
KS_HD inline int pf_share_owner(int n, int G, int u) { return (int)((((unsigned int)u + 1u) * (unsigned int)G - 1u) / (unsigned int)n); }

// How the prefill GEMM covers one matrix for a prompt of tt token tiles (16 rows each)
struct PfPlan {
    int tb;                  // token tiles per workgroup: 16, 12, 8 (256 weight rows) or 4 (128 weight rows)
    int n_mt, n_mr, n_tt;    // row tiles, those of them with rotary pairs (OP_QKV), workgroup tiles along the tokens
    int rows;                // rows of the prompt's token tiles
    int S;                   // parts K is split into (G > 0: the most parts of a tile)
    bool fused = false;      // workgroups of 256 rows that walk all of K finish their rows themselves, whatever tb is
    int G = 0;               // > 0: a thin launch of so many workgroups (prefill_thin_kernel), tiles of 256 weight rows x all tokens
    int tiles() const { return n_mt * n_tt; }
    // sums through memory to a row kernel? (residual rows always; the others unless one large workgroup finishes them)
    bool parts(int which) const { return G > 0 || S > 1 || (tb != 16 && !fused) || which == PF_O || which == PF_DOWN; }
    int epilogue(int which) const { return parts(which) ? PF_PARTS : (which == PF_GU ? PF_SWIGLU : PF_ROPE); }
    bool own_sums(int which) const { return which == PF_QKV || tb == 4; }       // sums of their own per step: see the kernel
    int tm() const { return tb == 4 && G == 0 ? 128 : 256; }
    int out_rows() const { return rows; }
    size_t part_bytes() const { return (size_t)S * out_rows() * n_mt * tm() * 4; }       // K parts of the product
};

// row tiles of tm rows that cover a matrix (n_mr: those of rotary pairs)
inline int pf_row_tiles(const knnssd_model_cfg &g, int which, int tm, int *n_mr = nullptr) {
    const int P = (g.n_heads + g.n_kv_heads) * (g.head_dim / 2), VR = g.n_kv_heads * g.head_dim;
    const int mr = which == PF_QKV ? (P + tm / 2 - 1) / (tm / 2) : 0;
    if (n_mr) *n_mr = mr;
    if (which == PF_QKV) return mr + (VR + tm - 1) / tm;
    return which == PF_GU ? (g.d_ffn + tm / 2 - 1) / (tm / 2) : (g.d_model + tm - 1) / tm;
}

// The plan with the lowest estimated time: rounds of workgroups over the chip x (steps x ns of a step + what a workgroup
// pays once), plus the K parts' way through memory. The constants come from kernel traces (those of 128 x 64 from before its wavefronts
// had roles); what counts is the choice. With one matrix's plan varied at a time over 7B, 13B and Qwen widths, whole prompts, us per
// block against the choice: 20 to 130 rows (blocks of 170-410 us, all crossings of 128 x 64 and 256 x 128) no plan is better by
// more than 5, half of which is noise. 7B, 45 rows: QKV in five parts of 128 x 64 (chosen), in two +1, in four +3; gate+up in four (chosen),
// unsplit +5, in five +7; 13B, 80 rows: QKV in four parts of 256 x 128 (chosen), of 128 x 64 +14; gate+up in two (chosen), four +8.
// 200 to 400 rows: within 13 but for gate+up at 260 and 300 rows (256 x 256, where two or three parts of 256 x 128 take 14-28 less of
// 500-700) and 13B's QKV there (-15). 13B, 1024 rows: QKV unsplit 256 x 256 (chosen), 256 x 128 +31 us, in two parts +60; O in three
// parts of 256 x 256 (chosen), of 256 x 128 -7, in two +17; gate+up unsplit (chosen), 256 x 128 +86.
// least > 0 (pf_choose): also tiles of 256 x 192, and 256 x 128 ones that finish their rows themselves where K is whole; at least so many parts,
// of at most `room` bytes together.
inline PfPlan pf_plan(const knnssd_model_cfg &g, int which, int tt, int least = 0, size_t room = 0) {
    const int K = which == PF_O ? g.n_heads * g.head_dim : (which == PF_DOWN ? g.d_ffn : g.d_model), KS = K / 32;
    PfPlan best{};
    double best_cost = 0;
    for (int tb = 4; tb <= 16; tb += 4) {
        if (tb == 12 && least == 0) continue;
        PfPlan p{};
        p.tb = tb;
        p.fused = least > 0 && tb >= 8;
        const int tm = p.tm();
        p.n_mt = pf_row_tiles(g, which, tm, &p.n_mr);
        p.n_tt = (tt + tb - 1) / tb;
        p.rows = tt * 16;
        // 256 x 256 to 256 x 128: one workgroup per unit, bound by the matrix cores. 128 x 64: the two workgroups a unit holds
        // take turns at its LDS, but pay their fixed cost together
        const double step = tb == 16 ? (which == PF_QKV ? 2340 : 1930) : tb == 12 ? (which == PF_QKV ? 1660 : 1380) : tb == 8 ? (which == PF_QKV ? 1290 : 1040) : 540;
        const double fixed = tb == 16 ? 14000 : tb == 12 ? 12000 : tb == 8 ? 10000 : 6000;
        for (int S = least > 0 ? least : 1; S <= 16; ++S) {
            if (S > 1 && S * 4 > KS) break;
            p.S = S;
            const int rounds = (p.tiles() * S + KS_NWG - 1) / KS_NWG;
            if (S > 1 && rounds > 8) break;
            if (least > 0 && p.parts(which) && p.part_bytes() > room) break;
            const double moved = p.parts(which) ? 2.0 * S * tt * 16 * p.n_mt * tm * 4 : 0;
            if (best_cost > 0 && moved / 3000 >= best_cost) break;     // (only grows with S)
            const double cost = rounds * ((KS + S - 1) / S * step) + (tb == 4 ? (rounds + 1) / 2 : rounds) * fixed + moved / 3000;
            if (best_cost == 0 || cost < best_cost) { best = p; best_cost = cost; }
        }
    }
    return best;
}

// The tiles a product takes: the best of pf_plan's and of the wide ones with no fewer parts, so that no sum has more roundings in a row than
// it would have without them (256 x 192 tiles of two parts instead of 256 x 256 ones of three for the O projection, and QKV rows of one part
// instead of two: 0.72 % of a Qwen-shaped prompt's cache entries on another bf16 value than in 64 bits, 777 rows, instead of 0.62). Gate+up rows may have
// fewer (in the shipped widths one part instead of two, 13B and Qwen with 257 to 288 and 577 to 640 rows, 7B with 641 to 784): they reach the cache through the down
// product alone. Measured against pf_plan alone over 96 prompts each: the next block's cache entries lie on another bf16 value 0.1 to 0.3 % more often (13B 257
// and 600 rows +0.13 and +0.12 % of 1.3-1.4 %, Qwen +0.34 and +0.23 %, 7B 777 +0.19 %), hidden states' error +0.5, -0.8, -0.1, -0.4, +0.7 % with a standard error
// of 0.5 to 0.8. With no fewer parts these prompts take 4-6 % longer (13B 257 rows, two blocks, 1096 -> 1166 us, 608 2076 -> 2168, Qwen 257 983 -> 1045, 7B 777 1772 ->
// 1859) and up to 31 % more workspace (7B, 576 positions); with sums of their own per step as long (1167, 2216, 1037, 1872).
// 128 x 64 tiles add up each step's planes on their own (own_sums), which the residual and SwiGLU rows do nowhere else: those stay.
// Measured against pf_plan alone, whole prompts, two blocks, us: 7B 180 rows 738 -> 660, 257 1110 -> 983, 777 2201 -> 2005, 13B 257 1474 -> 1255, 600
// 2575 -> 2313, 2200 7776 -> 7066, Qwen 513 2280 -> 2003, 777 2919 -> 2845; where the plan stays (100, 400, 1024 rows) 0.997-1.003.
// Room for the parts of a product: what pf_plan's take in the shipped widths at the lengths where they take most. The workspace grows where a context's
// max_seq does not reach those lengths (four blocks, pf_plan alone -> with these: 13B up to 256 positions 83 -> 115 MB, 1024 288 -> 322,
// Qwen 256 92 -> 119) and shrinks where other tiles need fewer parts (7B 576 287 -> 233, 1024 320 -> 244, 13B 512 182 -> 128); from 4608 positions
// on it is the same. A context over a buffer that is too small for it takes pf_plan's tiles.
constexpr size_t PF_PART_ROOM = (size_t)128 << 20;
inline PfPlan pf_tiles(const knnssd_model_cfg &g, int which, int tt) {
    const PfPlan p = pf_plan(g, which, tt);
    if (p.tb == 4 && which != PF_QKV) return p;
    const size_t room = p.parts(which) ? p.part_bytes() : 0;
    return pf_plan(g, which, tt, which == PF_GU ? 1 : p.S, room > PF_PART_ROOM ? room : PF_PART_ROOM);
}

// Prompts of up to PF_THIN token tiles take prefill_thin_kernel for matrices of at least PF_THIN_PAIRS pairs of steps a workgroup: with fewer
// its fixed cost shows (7B's O projection, four pairs: 14.9 us against 14.5; models of 256 to 2000 columns with all products
// this way 12-20 % slower), 13B's O projection with six and a quarter takes 18 against 20.
constexpr int PF_THIN = 3, PF_THIN_PAIRS = 6, PF_THIN_TILES = 4;        // PF_THIN_TILES: row tiles a workgroup's run may touch
constexpr int PF_THIN_FOLD = 8;                        // pairs of steps that are summed on their own
inline PfPlan pf_choose(const knnssd_model_cfg &g, int which, int tt) {
    const int K = which == PF_O ? g.n_heads * g.head_dim : (which == PF_DOWN ? g.d_ffn : g.d_model), KP = (K / 32 + 1) / 2;
    PfPlan p{};
    p.tb = 4;
    p.G = KS_NWG;
    p.n_mt = pf_row_tiles(g, which, p.tm(), &p.n_mr);
    p.n_tt = 1;
    p.rows = tt * 16;
    const int units = p.n_mt * KP;
    if (tt > PF_THIN || units < PF_THIN_PAIRS * KS_NWG || units > (PF_THIN_TILES - 2) * KP * KS_NWG) return pf_tiles(g, which, tt);
    for (int t = 0; t < p.n_mt; ++t) {
        const int n = pf_share_owner(units, p.G, (t + 1) * KP - 1) - pf_share_owner(units, p.G, t * KP) + 1;
        if (n > p.S) p.S = n;
    }
    if (p.S > 32) return pf_tiles(g, which, tt);        // few rows, many columns: a row kernel would read them all
    return p;
}

// plain: the workspace has room for pf_plan's parts only
inline PfPlan pf_tiles_of(const knnssd_model_cfg &g, int which, int tt, bool plain) { return plain ? pf_plan(g, which, tt) : pf_choose(g, which, tt); }

}  // namespace ks
