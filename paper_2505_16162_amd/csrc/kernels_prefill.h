// Prompt prefill for the tuned bf16 path (gfx950): the full model over hundreds to thousands of rows.
//
// Unlike a decode pass this is bound by the matrix cores, so it has kernels of its own. They read the
// SAME stream-order weights as the decode kernels (a unit = <= 16 rows x 32 columns is one MFMA A operand).
//
// Arithmetic, the same as in the decode kernels: activations are fp32 and stay exact, as three bf16 planes (hi + mid + lo by
// truncation = the value, whatever it is), weights are bf16 as they are. So a product takes three matrix instructions per 32
// columns, exact up to the sums in fp32.
//
// Activations of all rows live in "fragment order": [plane][32-column step][16-row tile][lane][8],
// lane = 16*kg + r holding row r of the tile and columns 8*kg..8*kg+7 of the step, i.e. the MFMA B
// operand of v_mfma_f32_16x16x32_bf16 as stored, so staging a tile is a linear copy. RMSNorm: the planes hold gain (.) x, the
// row's rsqrt lies beside them and multiplies the product's sums.
//
// prefill_gemm_kernel: a workgroup owns TA tiles of 16 weight rows x TB tiles of 16 tokens and walks K (or one of S parts
// of it) in steps of 32 columns. Activations and weights go from memory straight to LDS (16-byte loads whose LDS side is
// linear and whose memory side is free). A tile is filled with whatever rows suit it, wherever they lie in the decode
// layout: no dead rows from the decode layout's short tiles (20 rows per workgroup = two
// tiles of 10), and the two dot products an epilogue combines sit in one lane's accumulators.
#pragma once
#include "kernels_bf16.h"
#include "prefill_plan.h"

namespace ks {

constexpr int PF_NT = 512;             // threads per workgroup of the prefill GEMM (8 wavefronts)
constexpr int PF_RT = 1024;            // ... and of the row kernels between the products (at most, where columns are on their own)
constexpr int PF_NP = 3;               // bf16 planes of an activation

struct PfArgs {
    GemmOp op;              // type, W, N, K, q_out, kv_block, cos_t, sin_t, H, Hkv, hd, max_seq
    const bf16_t *frag_in;  // [planes][K/32][TT][512] fragment order
    const float *rstd;      // [n_tok] RMSNorm factor of the input rows; nullptr: none
    float *out;             // PF_PARTS: [K part][out_rows][n_mt * rows of a tile], tile order along the columns
    bf16_t *frag_out;       // PF_SWIGLU: the next product's operands, fragment order over the N features
    const u32x2 *rows;      // (PfRow) [n_mt * rows of a tile] where each row of the tiles lies
    int TT;                 // token tiles the fragment buffers are laid out for
    int n_tok, out_rows;    // live rows; row stride of a K part in out
    int n_mt, n_mr;         // row tiles of the matrix; OP_QKV: those that hold rotary pairs (the others hold value rows)
    int n_tt;               // token tiles (workgroup tiles) of the launch
    int S, steps, longer;   // K parts, 32-column steps of a part, and how many parts take one more
    float inv_tiles;        // 1 / (n_mt * n_tt)
};

__device__ __forceinline__ size_t frag_off(int KS, int TT, int pl, int ks, int tt) {
    return (((size_t)pl * KS + ks) * TT + tt) * 512;
}

// The bf16 planes of N neighbouring values (truncation: hi + mid + lo = v), two values per word. (contract off: where v is a
// product, the remainder has to be that of the rounded one.)
template <int N>
__device__ __forceinline__ void split_planes(const float *v, unsigned int (*w)[N / 2]) {
#pragma clang fp contract(off)
#pragma unroll
    for (int e = 0; e < N / 2; ++e) {
        // the upper halves of two neighbouring values make one register of a plane
        const float a = v[2 * e], b = v[2 * e + 1];
        const unsigned int a0 = __float_as_uint(a), b0 = __float_as_uint(b);
        const float ra = a - __uint_as_float(a0 & 0xffff0000u), rb = b - __uint_as_float(b0 & 0xffff0000u);
        const unsigned int a1 = __float_as_uint(ra), b1 = __float_as_uint(rb);
        const unsigned int a2 = __float_as_uint(ra - __uint_as_float(a1 & 0xffff0000u)), b2 = __float_as_uint(rb - __uint_as_float(b1 & 0xffff0000u));
        w[0][e] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
        w[1][e] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
        w[2][e] = __builtin_amdgcn_perm(b2, a2, 0x07060302u);
    }
}
// The planes of the eight values at features n..n+7 (n a multiple of 8) of row (tt, m), fragment order: one 16-byte store
// per plane; of the four at n..n+3 (n a multiple of 4): 8 bytes per plane.
__device__ __forceinline__ bf16_t *frag_at(bf16_t *frag, int KS, int TT, int pl, int tt, int m, int n) {
    return frag + frag_off(KS, TT, pl, n >> 5, tt) + (((n & 31) >> 3) * 16 + m) * 8 + (n & 7);
}
__device__ __forceinline__ void store_frag8(bf16_t *frag, int KS, int TT, int tt, int m, int n, const float *v) {
    unsigned int w[PF_NP][4];
    split_planes<8>(v, w);
#pragma unroll
    for (int pl = 0; pl < PF_NP; ++pl) *reinterpret_cast<u32x4 *>(frag_at(frag, KS, TT, pl, tt, m, n)) = u32x4{w[pl][0], w[pl][1], w[pl][2], w[pl][3]};
}
__device__ __forceinline__ void store_frag4(bf16_t *frag, int KS, int TT, int tt, int m, int n, f32x4 v4) {
    const float v[4] = {v4[0], v4[1], v4[2], v4[3]};
    unsigned int w[PF_NP][2];
    split_planes<4>(v, w);
#pragma unroll
    for (int pl = 0; pl < PF_NP; ++pl) *reinterpret_cast<u32x2 *>(frag_at(frag, KS, TT, pl, tt, m, n)) = u32x2{w[pl][0], w[pl][1]};
}

// four values rounded to bf16 (nearest even), 8-byte store
__device__ __forceinline__ void pf_store_bf16x4(bf16_t *p, f32x4 v) {
    *reinterpret_cast<u32x2 *>(p) = u32x2{(unsigned int)float_to_bf16_rne(v[0]) | ((unsigned int)float_to_bf16_rne(v[1]) << 16),
                                          (unsigned int)float_to_bf16_rne(v[2]) | ((unsigned int)float_to_bf16_rne(v[3]) << 16)};
}

// Loads that go straight to LDS: lane l's 16 bytes land at LDS byte lds_off + 16*l, whatever its source address is.
// (s_nop: a scalar address that a vector instruction has just written, e.g. one kept in a vector lane, may be read by a
// vector memory instruction five wait states later at the earliest, and inside asm nobody else sees to that.)
// The compiler does not count them; every use of the data sits behind a hand-placed vmcnt wait and a workgroup meeting.
__device__ __forceinline__ void dma_lane(const void *p, unsigned int lds_off) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(p), "s"(lds_off) : "memory");
}
__device__ __forceinline__ void dma_lane_nt(const void *p, unsigned int lds_off) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" : : "v"(p), "s"(lds_off) : "memory");
}
__device__ __forceinline__ void dma_linear(const void *base, unsigned int voff, unsigned int lds_off) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(base), "s"(lds_off) : "memory");
}
template <int KEEP> __device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(KEEP) : "memory"); }
// a workgroup meeting that leaves loads in flight (LDS reads of this wavefront have returned)
__device__ __forceinline__ void pf_meet() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// Where one row of a tile lies in the packed matrix. Tabulated when the context is created (prefill_row_table_kernel), one
// entry per row of each tile: x = the row's first 16-byte piece (8 columns) of step 0, in pieces from the matrix's start;
// y = rows of the decode layout's tile it belongs to (pieces between column groups, a quarter of a unit) | gshift << 16.
typedef u32x2 PfRow;

// workgroup of the decode layout that owns item n of N (inverse of wg_share)
__device__ __forceinline__ int pf_owner(int n, int N) { return (int)((((unsigned int)n + 1u) * (unsigned int)KS_NWG - 1u) / (unsigned int)N); }

// Row sr of row tile mt (TM rows). Which matrix row that is, is free to choose, since every row is fetched from wherever
// it lies: pairs whose two dot products meet in an epilogue (rotary halves, gate / up rows) sit in neighbouring 16-row
// tiles at the same place, so that one lane holds both. Rows past the end repeat the last one (never used).
// op: type, N, K, head counts and split table of the matrix; n_mr: its row tiles of rotary pairs (OP_QKV).
__global__ void prefill_row_table_kernel(GemmOp op, int TM, int n_mr, int n_entries, PfRow *table) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_entries) return;
    const int mt = i / TM, sr = i - mt * TM;
    const bool pairs = op.type == OP_SWIGLU || (op.type == OP_QKV && mt < n_mr);
    int wg, lr;
    if (pairs) {
        const int P = op.type == OP_SWIGLU ? op.N : (op.H + op.Hkv) * (op.hd >> 1);
        const int p = min(mt * (TM / 2) + (sr >> 5) * 16 + (sr & 15), P - 1);
        wg = pf_owner(p, P);
        lr = p - wg_share(P, wg) + ((sr >> 4) & 1) * op.split[wg].n_first;
    } else if (op.type == OP_QKV) {
        const int VR = op.Hkv * op.hd, v = min((mt - n_mr) * TM + sr, VR - 1);
        wg = pf_owner(v, VR);
        lr = v - wg_share(VR, wg) + 2 * op.split[wg].n_first;
    } else {
        const int n = min(mt * TM + sr, op.N - 1);
        wg = pf_owner(n, op.N);
        lr = n - wg_share(op.N, wg);
    }
    const WgSplit &s = op.split[wg];
    const int t = lr / s.rpt, rit = lr - t * s.rpt, rows_t = min(s.rpt, s.R - t * s.rpt);
    table[i] = u32x2{(unsigned int)((s.wg_base + (size_t)(t * s.rpt) * op.K) / 8 + rit), (unsigned int)(rows_t | (s.gshift << 16))};
}

// position of 32-column step st among the units of a tile (the order pack_matrix_kernel wrote them in)
__device__ __forceinline__ int pf_unit_index(int st, int KS, int gshift) {
    const int nfull = KS >> 4, rem = KS & 15, g = 1 << gshift, w16 = st & 15, kpart = w16 >> gshift;
    return nfull * g * kpart + min(rem, kpart * g) + (st >> 4) * g + (w16 & (g - 1));
}

// Epilogue arithmetic on four neighbours (a head's half and every row count are multiples of 4)
__device__ __forceinline__ f32x4 pf_swiglu(f32x4 g, f32x4 u) {
    f32x4 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = (g[q] / (1.0f + expf(-g[q]))) * u[q];
    return r;
}
// rotary pairs p..p+3 (first and second members x0, x1) of row tok (the prompt starts at position 0)
__device__ __forceinline__ void pf_rope_store(const GemmOp &op, int tok, int p, f32x4 x0, f32x4 x1) {
    const int half = op.hd >> 1, head = p >> (op.hd == 128 ? 6 : 5), d = p & (half - 1);      // head_dim is 64 or 128
    const f32x4 c = *reinterpret_cast<const f32x4 *>(op.cos_t + (size_t)tok * half + d);
    const f32x4 sn = *reinterpret_cast<const f32x4 *>(op.sin_t + (size_t)tok * half + d);
    f32x4 ra, rb;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        ra[q] = x0[q] * c[q] - x1[q] * sn[q];
        rb[q] = x1[q] * c[q] + x0[q] * sn[q];
    }
    if (head < op.H) {
        float *qp = op.q_out + ((size_t)tok * op.H + head) * op.hd + d;
        *reinterpret_cast<f32x4 *>(qp) = ra;
        *reinterpret_cast<f32x4 *>(qp + half) = rb;
    } else {
        bf16_t *kp = op.kv_block + ((size_t)(head - op.H) * op.max_seq + tok) * op.hd + d;
        pf_store_bf16x4(kp, ra);
        pf_store_bf16x4(kp + half, rb);
    }
}
__device__ __forceinline__ void pf_value_store(const GemmOp &op, int tok, int v, f32x4 val) {
    const int head = v >> (op.hd == 128 ? 7 : 6), d = v & (op.hd - 1);
    pf_store_bf16x4(op.kv_block + (((size_t)op.Hkv + head) * op.max_seq + tok) * op.hd + d, val);
}

// TA x TB tiles of 16 rows x 16 tokens per workgroup, 8 wavefronts in a WA x 8/WA grid, NS staged steps in LDS (PfShape).
// What bounds it. 256 x 256 and 256 x 128: the matrix cores, at 1.53-1.6 PFLOP/s issued (three instructions per product), where a
// large library product in bf16 reaches 1.59 on this card; one meeting per step for all wavefronts together kept the matrix
// pipe 55 % busy, two groups one phase apart 80 %. 13B-shaped, 4096 rows: QKV 1.52-1.55 ms (with its own sums, below),
// gate+up 2.26-2.33, O 0.44, down 1.12. 256 x 192 (three staged steps, a step's matrix instructions in one cluster): 1.36 us a step, 0.113 a token tile
// where 256 x 256 takes 1.93 and 0.121, 256 x 128 1.04 and 0.13; with its own sums 1.65. 128 x 64 (few rows): operand reads out of LDS about as much as the weight stream: a 4 x 2 grid
// of wavefronts reads 8 KB a wavefront and step, 8 x 1 reads 13 (7B, 45 rows, gate+up unsplit 79 -> 75 us); 5-6 us of a
// launch are its fixed cost. Half of the wavefronts request the weights and half the activations, so that the weights run five steps
// ahead and the activations three, and the operands of the next step are read under the matrix instructions of this one: whole prompts
// of 45 rows 7B 777 -> 761, 13B 1056 -> 1001, Qwen 1160 -> 1099 us. (Three steps of both 1031 and four 1005 us at 13B; six and
// two 1348; the steps in the order in which the units lie in memory: no faster.) Which tile a matrix and a length take: pf_plan.
// PP: the wavefronts form two groups (one wavefront of each on every SIMD) that run one phase apart: while one group
// issues its matrix instructions the other reads its operands from LDS.
constexpr int PF_ACT_STAGES = 3;       // steps of activations in LDS where half of the wavefronts fetch the weights, NS steps of them
template <int TA, int TB, int WA, int NS, bool PP>
struct PfShape {
    static constexpr int NSA = NS, NSB = PP ? NS : PF_ACT_STAGES;   // buffers for weights, for activations
    static constexpr int WB = 8 / WA, TAW = TA / WA, TBW = TB / WB;
    static constexpr int TM = TA * 16;
    static constexpr int A_BYTES = TA * 1024, B_BYTES = PF_NP * TB * 1024;      // a step's weights and activations in LDS
    // PP: a step's two side by side; otherwise each kind on its own, as their buffers differ in number
    static constexpr int A_NEXT = PP ? A_BYTES + B_BYTES : A_BYTES, B0 = PP ? A_BYTES : NSA * A_BYTES, B_NEXT = PP ? A_BYTES + B_BYTES : B_BYTES;
    // pieces per thread (fragments per wavefront) and step. PP: every wavefront takes weights and activations; otherwise the first
    // four take the weights, the others the activations: a wavefront's loads return in order, so this is what lets the
    // weights be requested further ahead than the activations.
    static constexpr int NA = PP ? TA / 8 : TA / 4, NB = PP ? (PF_NP * TB + 7) / 8 : PF_NP * TB / 4;
    static constexpr size_t LDS = (size_t)NSA * A_BYTES + NSB * B_BYTES;
};

template <int TA, int TB, int WA, int NS, bool PP, int EPI, bool OWN>
__global__ __launch_bounds__(PF_NT, TA == 16 ? 2 : 4) void prefill_gemm_kernel(PfArgs a) {
    typedef PfShape<TA, TB, WA, NS, PP> Sh;
    constexpr int NSA = Sh::NSA, NSB = Sh::NSB;
    constexpr int TAW = Sh::TAW, TBW = Sh::TBW, TM = Sh::TM;
    extern __shared__ __align__(16) char lds[];
    const GemmOp &op = a.op;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wa = PP ? wave >> 2 : wave / Sh::WB, wb = PP ? wave & 3 : wave % Sh::WB, kg = lane >> 4, r16 = lane & 15;
    const int KS = op.K >> 5;

    // workgroup -> (K part, token tile, row tile). Workgroups are dealt to the 8 dies by index: each die takes a run of the
    // order below, in which neighbours share weights (four token tiles) or activations. At most seven workgroups of a launch
    // are left over: ones that return at once still take their turn on the units, and 48 of them among 240 cost the
    // others a second round.
    const int tiles = a.n_mt * a.n_tt, total = tiles * a.S, run = blockIdx.x & 7;
    int lin = (total * run >> 3) + (int)(blockIdx.x >> 3), sp = 0;
    if (lin >= total * (run + 1) >> 3) return;
    if (a.S > 1) { sp = div_small(lin, tiles, a.inv_tiles); lin -= sp * tiles; }
    int mt = lin, tk = 0;
    if (a.n_tt > 1) {
        const int tb4 = lin / (a.n_mt * 4), in_blk = lin - tb4 * (a.n_mt * 4), tw = min(4, a.n_tt - tb4 * 4);
        mt = in_blk / tw;
        tk = tb4 * 4 + (in_blk - mt * tw);
    }
    const int tt0 = tk * TB;
    const int st0 = sp * a.steps + min(sp, a.longer), cnt = a.steps + (sp < a.longer);

    // what this thread stages per step
    const bf16_t *ap[Sh::NA];
    unsigned int ar[Sh::NA];
#pragma unroll
    for (int q = 0; q < Sh::NA; ++q) {
        const PfRow r = a.rows[mt * TM + (PP ? wave + q * 8 : (wave & 3) * Sh::NA + q) * 16 + r16];
        ar[q] = r.y;
        ap[q] = op.W + ((size_t)r.x + kg * (r.y & 0xffffu)) * 8;
    }
    const unsigned int l0 = (unsigned int)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const char *bsrc[Sh::NB];
    unsigned int bdst[Sh::NB];
#pragma unroll
    for (int q = 0; q < Sh::NB; ++q) {
        const int f = PP ? min(wave + q * 8, PF_NP * TB - 1) : (wave & 3) * Sh::NB + q, pl = f / TB, t = f - pl * TB;    // a repeat writes the same bytes again
        bsrc[q] = reinterpret_cast<const char *>(a.frag_in + frag_off(KS, a.TT, pl, st0, min(tt0 + t, a.TT - 1)));
        bdst[q] = Sh::B0 + f * 1024;
    }
    const size_t bstep = (size_t)a.TT * 1024;
    const unsigned int voff = lane * 16;
    const bool once = a.n_tt == 1;                 // every weight byte is used by one workgroup only: nothing to keep in a cache
    auto weight_piece = [&](int t, int q) {        // (the three possible deals of the columns in scalar arithmetic, then a choice)
        const int u0 = pf_unit_index(st0 + t, KS, 0), u1 = pf_unit_index(st0 + t, KS, 1), u2 = pf_unit_index(st0 + t, KS, 2);
        const unsigned int u = ar[q] >= 0x20000u ? u2 : (ar[q] >= 0x10000u ? u1 : u0);
        return ap[q] + (unsigned long long)u * ((ar[q] & 0xffffu) * 32u);
    };
    auto issue_b = [&](int t, int buf) {           // activations of step st0 + t into LDS buffer buf
#pragma unroll
        for (int q = 0; q < Sh::NB; ++q) dma_linear(bsrc[q] + t * bstep, voff, l0 + buf * Sh::B_NEXT + bdst[q]);
    };
    auto issue_a = [&](int t, int buf) {           // ... and its weights as they are
#pragma unroll
        for (int q = 0; q < Sh::NA; ++q) {
            const unsigned int d = l0 + buf * Sh::A_NEXT + (PP ? wave + q * 8 : (wave & 3) * Sh::NA + q) * 1024;
            if (once) dma_lane_nt(weight_piece(t, q), d);
            else dma_lane(weight_piece(t, q), d);
        }
    };
    f32x4 acc[TAW][TBW];
#pragma unroll
    for (int i = 0; i < TAW; ++i)
#pragma unroll
        for (int j = 0; j < TBW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const char *la = lds + wa * TAW * 1024 + voff, *lb = lds + Sh::B0 + wb * TBW * 1024 + voff;
    constexpr int JC = TBW <= 3 ? TBW : 2, CL = TBW / JC;      // token tiles per cluster of matrix instructions, clusters per step
    constexpr int SETS = PP ? 1 : 2;                           // operands of two steps in registers: the next one's are read under this one's matrix instructions
    u32x4 avs[SETS][TAW], bvs[SETS][JC][PF_NP];
    auto read_a = [&](int buf, int set = 0) {
#pragma unroll
        for (int i = 0; i < TAW; ++i) avs[set][i] = *reinterpret_cast<const u32x4 *>(la + buf * Sh::A_NEXT + i * 1024);
    };
    auto read_b = [&](int buf, int c, int set = 0) {
#pragma unroll
        for (int jj = 0; jj < JC; ++jj)
#pragma unroll
            for (int p = 0; p < PF_NP; ++p) bvs[set][jj][p] = *reinterpret_cast<const u32x4 *>(lb + buf * Sh::B_NEXT + (p * TB + c * JC + jj) * 1024);
    };
    // OWN: a step's three planes are summed on their own, from the lowest up, and then added to the running sums: one rounding at
    // the size of the whole sum per 32 columns instead of three. For the QKV rows, whose keys and values the cache rounds to
    // bf16: entries that land on another value than in 64 bits 5.8e-4 -> 2.3e-4 (13B-shaped block, 1024 rows), for 335 -> 378
    // us (a vector addition takes 0.6 of its time from the matrix pipe, among the matrix instructions or in the reading phase).
    // In the other products, whose rows stay fp32, it changed neither that share nor the hidden state's error (gate+up 640 ->
    // 726 us). The 128 x 64 build has it always: the matrix pipe waits there anyway. In groups of GR tiles: a group's additions stand among the next
    // group's matrix instructions, the last group's in the next reading phase (settle).
    constexpr int NT_CL = TAW * JC, GR = NT_CL < 4 ? NT_CL : 4, NG = NT_CL / GR;
    f32x4 own[2][GR];
    auto add = [&](int c, int g) {
#pragma unroll
        for (int k = 0; k < GR; ++k) {
            f32x4 &d = acc[(g * GR + k) % TAW][c * JC + (g * GR + k) / TAW];
            d += own[g & 1][k];
            asm volatile("" : "+v"(d));        // here, not at the step's end, where every group's sums would have to be kept
        }
    };
    auto settle = [&](int c) { add(c, NG - 1); };
    auto mfma_cluster = [&](int c, int set = 0) {
        const auto &av = avs[set];
        const auto &bv = bvs[set];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
#pragma unroll
            for (int p = PF_NP - 1; p >= 0; --p)
#pragma unroll
                for (int k = 0; k < GR; ++k) {
                    const int i = (g * GR + k) % TAW, jj = (g * GR + k) / TAW;
                    const bf16x8 w = __builtin_bit_cast(bf16x8, av[i]), x = __builtin_bit_cast(bf16x8, bv[jj][p]);
                    if constexpr (OWN) {
                        const f32x4 from = p == PF_NP - 1 ? f32x4{0.f, 0.f, 0.f, 0.f} : own[g & 1][k];
                        own[g & 1][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, from, 0, 0, 0);
                    } else {
                        f32x4 &d = acc[i][c * JC + jj];
                        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, d, 0, 0, 0);
                    }
                }
            if constexpr (OWN) {
                if (g > 0) add(c, g - 1);
                __builtin_amdgcn_sched_barrier(0);     // (at most two groups of sums: registers)
            }
        }
    };
    if constexpr (OWN)
#pragma unroll
        for (int k = 0; k < GR; ++k) own[(NG - 1) & 1][k] = f32x4{0.f, 0.f, 0.f, 0.f};     // nothing to settle before the first step

    // the first steps (a step past the end repeats the last one, here and below: the loads stay countable)
    const bool takes_a = wave < 4;
    if constexpr (PP) {
#pragma unroll
        for (int t = 0; t < NS - 1; ++t) {
            issue_a(min(t, cnt - 1), t);
            issue_b(min(t, cnt - 1), t);
        }
        dma_wait<0>();
    } else if (takes_a) {
#pragma unroll
        for (int t = 0; t < NSA; ++t) issue_a(min(t, cnt - 1), t);
        dma_wait<(NSA - 1) * Sh::NA>();
    } else {
#pragma unroll
        for (int t = 0; t < NSB; ++t) issue_b(min(t, cnt - 1), t);
        dma_wait<(NSB - 1) * Sh::NB>();
    }
    pf_meet();
    if constexpr (PP) {
        // Phases of a group: read operands | meet | matrix instructions | meet. The second group enters one phase later.
        // With three buffers (one cluster per step) step t+2 is staged while step t is read, when the last reads of step
        // t-1 are one phase old; with two (two clusters per step) step t+1 is requested while cluster 0 of step t is read.
        constexpr int YOUNG = Sh::NB + Sh::NA;     // loads issued in one reading phase
        if (wa == 1) pf_meet();
        int buf = 0;
        for (int t = 0; t < cnt; ++t) {
            const int nb = NS == 2 ? buf ^ 1 : (buf == 0 ? 2 : buf - 1), tn = min(t + NS - 1, cnt - 1);
            read_a(buf);
            read_b(buf, 0);
            issue_a(tn, nb);
            issue_b(tn, nb);
            if constexpr (OWN) settle(CL - 1);     // of the step before
            if constexpr (CL == 1) dma_wait<YOUNG>();       // step t+1 has arrived (what was issued just now stays in flight)
            pf_meet();
            __builtin_amdgcn_s_setprio(1);
            mfma_cluster(0);
            __builtin_amdgcn_s_setprio(0);
            pf_meet();
            if constexpr (CL == 2) {
                read_b(buf, 1);
                if constexpr (OWN) settle(0);
                if (wa == 1) dma_wait<0>();        // the first group reads step t+1 one phase from here
                pf_meet();
                __builtin_amdgcn_s_setprio(1);
                mfma_cluster(1);
                __builtin_amdgcn_s_setprio(0);
                if (wa == 0) dma_wait<0>();
                pf_meet();
            }
            buf = NS == 2 ? buf ^ 1 : (buf == 2 ? 0 : buf + 1);
        }
        if (wa == 0) pf_meet();
    } else {
        static_assert(CL == 1, "a step's operands are read together");
        int ba = 0, bb = 0;                                // buffers of the step whose operands are read
        read_a(0, 0);
        read_b(0, 0, 0);
        auto step = [&](int t, auto set) {                 // matrix instructions of step t, operands of step t + 1
            constexpr int S = decltype(set)::value;
            if (takes_a) dma_wait<(NSA - 2) * Sh::NA>();   // step t + 1 has arrived
            else dma_wait<(NSB - 2) * Sh::NB>();
            pf_meet();                                     // ... and every wavefront has its operands of step t
            if (takes_a) issue_a(min(t + NSA, cnt - 1), ba);
            else issue_b(min(t + NSB, cnt - 1), bb);
            ba = ba == NSA - 1 ? 0 : ba + 1;
            bb = bb == NSB - 1 ? 0 : bb + 1;
            if constexpr (OWN) settle(0);
            read_a(ba, S ^ 1);
            read_b(bb, 0, S ^ 1);
            mfma_cluster(0, S);
        };
        for (int t = 0; t < cnt; t += 2) {
            step(t, std::integral_constant<int, 0>{});
            if (t + 1 < cnt) step(t + 1, std::integral_constant<int, 1>{});
        }
    }
    if constexpr (OWN) settle(CL - 1);
    dma_wait<0>();                                 // nothing is in flight towards LDS when the workgroup ends

    // lane (kg, r16) holds rows 4*kg..4*kg+3 of its TAW row tiles for token r16 of its TBW token tiles
#pragma unroll
    for (int j = 0; j < TBW; ++j) {
        const int tok = (tt0 + wb * TBW + j) * 16 + r16;
        if (tok >= a.n_tok) continue;
        const float scale = a.rstd ? a.rstd[tok] : 1.0f;
        if constexpr (EPI == PF_PARTS) {
            float *o = a.out + ((size_t)sp * a.out_rows + tok) * ((size_t)a.n_mt * TM) + mt * TM + wa * TAW * 16 + 4 * kg;
#pragma unroll
            for (int i = 0; i < TAW; ++i) *reinterpret_cast<f32x4 *>(o + i * 16) = acc[i][j] * scale;
        } else if (EPI == PF_SWIGLU || mt < a.n_mr) {
#pragma unroll
            for (int i = 0; i < TAW; i += 2) {
                const int p = mt * (TM / 2) + (wa * TAW + i) * 8 + 4 * kg;
                if constexpr (EPI == PF_SWIGLU) {
                    if (p < op.N) store_frag4(a.frag_out, op.N >> 5, a.TT, tt0 + wb * TBW + j, r16, p, pf_swiglu(acc[i][j] * scale, acc[i + 1][j] * scale));
                } else if (p < (op.H + op.Hkv) * (op.hd >> 1)) {
                    pf_rope_store(op, tok, p, acc[i][j] * scale, acc[i + 1][j] * scale);
                }
            }
        } else {    // value rows
#pragma unroll
            for (int i = 0; i < TAW; ++i) {
                const int v = (mt - a.n_mr) * TM + (wa * TAW + i) * 16 + 4 * kg;
                if (v < op.Hkv * op.hd) pf_value_store(op, tok, v, acc[i][j] * scale);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// Prompts of up to PF_THIN token tiles over large matrices: the weight stream is what counts, as in a decode pass.
// A workgroup owns 256 weight rows x all of the prompt's rows. Eight wavefronts take two row tiles each and load their weights from
// memory straight into registers (a weight is an operand of one wavefront only, so LDS would be a detour); TB more do
// nothing but fetch a token tile of the activations each, which all eight read, into LDS, so that the workgroup meets once per
// pair of steps and neither kind of load waits behind the other. K is not cut into equal parts: the tiles' pairs of steps stand in one
// row and each of the G workgroups takes an equal run of them (pf_share), so that no workgroup is left over
// whatever the number of row tiles, and the stream runs on where a run crosses from one tile into the next.
// Measured against the 128 x 64 tiles of prefill_gemm_kernel (7B widths, 17 / 45 rows, us a launch): QKV 29 / 32 -> 21 / 26, gate+up 58 / 62 ->
// 40 / 48, down 26 / 28 -> 19 / 24; whole prompts of 17 rows, two blocks, 7B 372 -> 321 and 13B 511 -> 426, of 40 to 45 rows 410 -> 372 and
// 538 -> 479, Qwen 33 rows 675 -> 617. What is left above the stream (17 / 30 / 15 us): 3 us to start, 4-7 us for the parts' way
// out (22 MB), and the activations, each of which crosses from the L2 once per row tile: 0.3 us per token tile and step more than
// the weights take. Four token tiles: as fast as prefill_gemm_kernel (7B, 64 rows 423 against 426). Four wavefronts with four row tiles each
// (half the LDS reads): no change. Six steps ahead instead of four, three of activations per meeting: no change. A run's sums are folded into a second
// set every PF_THIN_FOLD pairs, so that a run longer than prefill_gemm_kernel's parts (7B's gate+up rows: 44 steps instead of 32) has no more
// roundings in a row: no change in time (45 rows, 7B 348 -> 339, 13B 460 -> 455, Qwen 421 -> 417 us); cache entries of the next block on another bf16 value
// than in 64 bits, against the 128 x 64 tiles (geometric means over 192 prompts each of 17, 33 and 45 rows): 7B 0.92, 0.97, 0.98 without, 0.84, 0.89, 0.90 with;
// 13B 0.84 and 0.78, Qwen 0.66 to 0.77 and 0.64 to 0.78.
// ------------------------------------------------------------------------------------------
constexpr int PF_THIN_WAVES = 8, PF_THIN_BUFS = 5;     // pairs of steps whose activations are in LDS
constexpr int pf_thin_nt(int tb) { return (PF_THIN_WAVES + tb) * 64; }
constexpr size_t pf_thin_lds_bytes(int tb) { return (size_t)PF_THIN_BUFS * 2 * PF_NP * tb * 1024 + PF_THIN_TILES * 256 * sizeof(PfRow); }

template <int TB>
__global__ __launch_bounds__(pf_thin_nt(TB)) void prefill_thin_kernel(PfArgs a) {
    constexpr int NB = PF_THIN_BUFS, TM = 256, RT = 16 / PF_THIN_WAVES;
    constexpr int STEP = PF_NP * TB * 1024, PAIR = 2 * STEP, PER = 2 * PF_NP;
    extern __shared__ __align__(16) char lds[];
    const GemmOp &op = a.op;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = lane >> 4, r16 = lane & 15;
    const int KS = op.K >> 5, KP = (KS + 1) >> 1, units = a.n_mt * KP, G = gridDim.x;
    const int q0 = __builtin_amdgcn_readfirstlane(pf_share(units, G, blockIdx.x));        // (quotients come out of the vector unit)
    const int n = __builtin_amdgcn_readfirstlane(pf_share(units, G, blockIdx.x + 1)) - q0;
    int mt = __builtin_amdgcn_readfirstlane(q0 / KP), kp = q0 - mt * KP;
    if (wave >= PF_THIN_WAVES) {
        const int fw = wave - PF_THIN_WAVES;       // its token tile
        const unsigned int l0 = (unsigned int)(uintptr_t)(__attribute__((address_space(3))) char *)lds + fw * 1024, voff = lane * 16;
        const char *src = reinterpret_cast<const char *>(a.frag_in + frag_off(KS, a.TT, 0, 0, fw));
        const size_t plane = (size_t)KS * a.TT * 1024, step = (size_t)a.TT * 1024;
        int buf = 0;
        auto fetch = [&]() {                       // the next pair (a step past the end of K repeats the last one)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int pl = 0; pl < PF_NP; ++pl)
                    dma_linear(src + min(2 * kp + s, KS - 1) * step + pl * plane, voff, l0 + buf * PAIR + s * STEP + pl * TB * 1024);
            kp = kp == KP - 1 ? 0 : kp + 1;
            buf = buf == NB - 1 ? 0 : buf + 1;
        };
        for (int c = 0; c < min(n, NB - 1); ++c) fetch();
        for (int c = 0; c < n; ++c) {
            const int younger = min(n - 1 - c, NB - 2);
            static_assert(NB == 5, "the waits below");
            if (younger == 3) dma_wait<3 * PER>();
            else if (younger == 2) dma_wait<2 * PER>();
            else if (younger == 1) dma_wait<PER>();
            else dma_wait<0>();
            pf_meet();                             // pair c is here, and everybody is done with pair c - 1
            if (c + NB - 1 < n) fetch();
        }
        return;
    }
    float scale[TB];
#pragma unroll
    for (int j = 0; j < TB; ++j) scale[j] = a.rstd ? a.rstd[min(j * 16 + r16, a.n_tok - 1)] : 1.0f;
    // where the wavefront's rows of the run's tiles lie, kept in LDS: fetched again where the run crosses into the next tile, a load would wait
    // behind the weights
    PfRow *const rows = reinterpret_cast<PfRow *>(lds + NB * PAIR) + wave * PF_THIN_TILES * RT * 16 + r16;
    static_assert(PF_THIN_TILES == 4, "a group of 16 lanes per tile");
#pragma unroll
    for (int i = 0; i < RT; ++i) rows[(kg * RT + i) * 16] = a.rows[min(mt + kg, a.n_mt - 1) * TM + wave * RT * 16 + i * 16 + r16];
    PfRow row[RT];
    const unsigned int nfull = KS >> 4, rem = KS & 15;
    u32x4 av[2][2][RT];                            // weights of two pairs
    int lt = 0, lk = kp, lc = 0;                   // the next pair to be requested: tile of the run, place in it, number in the run
    auto load_a = [&](int u, int s) {              // its step s; past the end one piece that all lanes share
        unsigned int live = lc < n && 2 * lk + s < KS ? 0xffffffffu : 0u;
        asm volatile("" : "+v"(live));             // (no branch around the loads: they stay countable)
        const unsigned int st = 2 * lk + s, w16 = st & 15, blk = st >> 4;
#pragma unroll
        for (int i = 0; i < RT; ++i) {             // pf_unit_index, a lane's own deal of the columns
            const unsigned int gs = row[i].y >> 16, rt = row[i].y & 0xffffu, first = (w16 >> gs) << gs;
            const unsigned int unit = __umul24(nfull, first) + min(rem, first) + (blk << gs) + (w16 - first);
            const unsigned int piece = (row[i].x + kg * rt + unit * rt * 4) & live;
            av[u][s][i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(op.W) + piece);
        }
    };
    auto rows_of = [&]() {
#pragma unroll
        for (int i = 0; i < RT; ++i) row[i] = rows[(min(lt, PF_THIN_TILES - 1) * RT + i) * 16];
    };
    auto advance = [&]() {
        ++lc;
        lt += lk == KP - 1;
        lk = lk == KP - 1 ? 0 : lk + 1;
        rows_of();
    };
    rows_of();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        load_a(u, 0);
        load_a(u, 1);
        advance();
    }
    f32x4 acc[RT][TB], sum[RT][TB];                // of the last pairs, of those before
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const char *lb = lds + lane * 16;
    int buf = 0, young = 0;                        // pairs in acc
    auto pair = [&](int c, int u) {                // (one past the end requests its weights like the others, so that the loads in flight stay countable)
        const bool on = c < n;
        if (on) pf_meet();
        const char *b = lb + buf * PAIR;
        bf16x8 x[2][PF_NP];
        f32x4 own[2][RT];                          // a step's three planes are summed on their own, see prefill_gemm_kernel; added under the next tile's matrix instructions
        auto read = [&](int s, int j) {
#pragma unroll
            for (int p = 0; p < PF_NP; ++p) x[j & 1][p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(b + s * STEP + (p * TB + j) * 1024));
        };
        auto step = [&](int s) {
            read(s, 0);
#pragma unroll
            for (int j = 0; j <= TB; ++j) {
                if (j + 1 < TB) read(s, j + 1);
                if (j < TB) {
#pragma unroll
                    for (int p = PF_NP - 1; p >= 0; --p)
#pragma unroll
                        for (int i = 0; i < RT; ++i)
                            own[j & 1][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[u][s][i]), x[j & 1][p],
                                                                                    p == PF_NP - 1 ? f32x4{0.f, 0.f, 0.f, 0.f} : own[j & 1][i], 0, 0, 0);
                }
                if (j > 0)
#pragma unroll
                    for (int i = 0; i < RT; ++i) {
                        acc[i][j - 1] += own[(j - 1) & 1][i];
                        asm volatile("" : "+v"(acc[i][j - 1]));    // here, not behind all steps, where every step's sums would have to be kept
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (on) step(0);
        __builtin_amdgcn_sched_barrier(0);
        load_a(u, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (on && 2 * kp + 1 < KS) step(1);
        __builtin_amdgcn_sched_barrier(0);
        load_a(u, 1);
        advance();
        __builtin_amdgcn_sched_barrier(0);
        const bool last = kp == KP - 1;            // of its tile
        if (on && (++young == PF_THIN_FOLD || last || c == n - 1)) {
            young = 0;
#pragma unroll
            for (int j = 0; j < TB; ++j)
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    sum[i][j] += acc[i][j];
                    acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
        if (on && (last || c == n - 1)) {
            const int part = (int)blockIdx.x - pf_share_owner(units, G, mt * KP);
#pragma unroll
            for (int j = 0; j < TB; ++j) {
                const int tok = j * 16 + r16;
                float *o = a.out + ((size_t)part * a.out_rows + tok) * ((size_t)a.n_mt * TM) + mt * TM + wave * RT * 16 + 4 * kg;
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    if (tok < a.n_tok) *reinterpret_cast<f32x4 *>(o + i * 16) = sum[i][j] * scale[j];
                    sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
            ++mt;
        }
        kp = last ? 0 : kp + 1;
        buf = buf == NB - 1 ? 0 : buf + 1;
    };
    for (int c = 0; c < n; c += 2) {
        pair(c, 0);
        pair(c + 1, 1);
    }
}

// ------------------------------------------------------------------------------------------
// Row kernels, between the products: they add up the K parts, finish a row and write the next product's operands. Bound by
// memory. Four neighbouring features per thread, so that the loads of neighbouring lanes adjoin (with eight, 1024 rows of
// 5120 in three parts take 32 us instead of 30, SwiGLU of 45 x 11008 in four parts 17.6 instead of 11.2). A row's share of a
// fragment is 16 bytes of each 256: the workgroups of the 16 rows that share the fragments are neighbours on one die, so that
// its L2 puts whole lines together.
// ------------------------------------------------------------------------------------------
struct PfRowArgs {
    GemmOp op;                  // as in PfArgs
    const int32_t *toks;        // embedding: token ids
    const float *in;            // [S][out_rows][ld] K parts
    int n_tok, S, out_rows, ld, TM;     // TM: rows per tile of the product's column order
    int KP, units, G;           // G > 0: the tiles' KP pairs of steps were dealt to G workgroups in one row of `units` (pf_share), a tile's number of parts follows
    int d;                      // features of the row
    float inv_dim, eps;
    float *x;                   // [n_tok][d] residual stream
    const float *gain;
    bf16_t *frag;
    float *rstd;
    int TT;
};

// The workgroup's token: tiles of 16 tokens are dealt to the dies, a die's consecutive workgroups take a tile's rows. The rows of up
// to PF_SPREAD tiles are dealt to the dies singly, since most dies would be idle otherwise (7B, 20 / 45 / 64 rows 718 / 767 / 829
// -> 682 / 743 / 784 us; 100 rows 942 -> 950, 13B 200 rows 1913 -> 1966: there the lines put together count).
constexpr int PF_SPREAD = 4;
inline unsigned int pf_row_grid(int n_tok, int tiles) { return tiles <= PF_SPREAD ? n_tok : (tiles + 7) / 8 * 128; }
__device__ __forceinline__ int pf_row_token(int n_tok) {
    if (n_tok <= PF_SPREAD * 16) return blockIdx.x;
    const int die = blockIdx.x & 7, i = blockIdx.x >> 3;
    return ((i >> 4) * 8 + die) * 16 + (i & 15);
}

// parts that the tile of column c was summed in. (CUT, a build of its own: a number that differs between lanes keeps the sum's loops in the
// vector unit; 1300 rows of 256 in 6.5 us without, 8.8 with.)
template <bool CUT> __device__ __forceinline__ int pf_n_parts(const PfRowArgs &a, int c) {
    if (!CUT) return a.S;
    const int u = c / a.TM * a.KP;
    return pf_share_owner(a.units, a.G, u + a.KP - 1) - pf_share_owner(a.units, a.G, u) + 1;
}
// columns c..c+3 of the S parts, added up in order
__device__ __forceinline__ f32x4 pf_sum_parts(const PfRowArgs &a, int tok, int c, int S) {
    const float *p = a.in + (size_t)tok * a.ld + c;
    const size_t st = (size_t)a.out_rows * a.ld;
    f32x4 v = *reinterpret_cast<const f32x4 *>(p);
    int s = 1;
    auto take = [&](auto n) {              // that many loads in flight
        f32x4 t[decltype(n)::value];
#pragma unroll
        for (int i = 0; i < decltype(n)::value; ++i) t[i] = *reinterpret_cast<const f32x4 *>(p + (s + i) * st);
#pragma unroll
        for (int i = 0; i < decltype(n)::value; ++i) v += t[i];
        s += decltype(n)::value;
    };
    while (s + 8 <= S) take(std::integral_constant<int, 8>{});
    if (s + 4 <= S) take(std::integral_constant<int, 4>{});
    if (s + 2 <= S) take(std::integral_constant<int, 2>{});
    if (s < S) take(std::integral_constant<int, 1>{});
    return v;
}
// column of the first member of pair p (the second sits 16 columns on): the row order of the product's tiles
__device__ __forceinline__ int pf_pair_col(int p, int TM) {
    const int mt = p / (TM / 2), r = p - mt * (TM / 2);
    return mt * TM + (r >> 4) * 32 + (r & 15);
}

// x = E[tok] or x += the product's row; the next norm's operands gain (.) x and the row's factor. One workgroup per token.
template <bool EMBED, bool CUT>
__global__ __launch_bounds__(PF_RT) void prefill_x_row_kernel(PfRowArgs a) {
    __shared__ float shares[PF_RT / 64];
    const int tok = pf_row_token(a.n_tok);
    if (tok >= a.n_tok) return;
    float sq = 0.f;
    for (int n = threadIdx.x * 4; n < a.d; n += PF_RT * 4) {
        f32x4 *xp = reinterpret_cast<f32x4 *>(a.x + (size_t)tok * a.d + n);
        f32x4 v, g;
        if constexpr (EMBED) {
            const u32x2 w = *reinterpret_cast<const u32x2 *>(a.op.embed + (size_t)a.toks[tok] * a.d + n);
            v = f32x4{bf_lo(w.x), bf_hi(w.x), bf_lo(w.y), bf_hi(w.y)};
        } else {
            const f32x4 x0 = *xp;
            v = x0 + pf_sum_parts(a, tok, n, CUT ? __builtin_amdgcn_readfirstlane(pf_n_parts<CUT>(a, n)) : a.S);     // (a wavefront's columns lie in one tile)
        }
        *xp = v;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            g[q] = a.gain[n + q] * v[q];          // (gains may lie at any multiple of 4 bytes)
            sq = fmaf(v[q], v[q], sq);
        }
        store_frag4(a.frag, a.d >> 5, a.TT, tok >> 4, tok & 15, n, g);
    }
    sq = wave_sum(sq);
    if ((threadIdx.x & 63) == 0) shares[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < PF_RT / 64; ++w) s += shares[w];
        a.rstd[tok] = 1.0f / sqrtf(s * a.inv_dim + a.eps);
    }
}

// SwiGLU of a gate+up product's K parts; gridDim.y workgroups per row
template <bool CUT>
__global__ __launch_bounds__(PF_RT) void prefill_u_row_kernel(PfRowArgs a) {
    const int tok = pf_row_token(a.n_tok);
    if (tok >= a.n_tok) return;
    for (int n = (blockIdx.y * blockDim.x + threadIdx.x) * 4; n < a.d; n += gridDim.y * blockDim.x * 4) {
        const int c = pf_pair_col(n, a.TM), S = pf_n_parts<CUT>(a, c);
        store_frag4(a.frag, a.d >> 5, a.TT, tok >> 4, tok & 15, n, pf_swiglu(pf_sum_parts(a, tok, c, S), pf_sum_parts(a, tok, c + 16, S)));
    }
}

// rotary embedding, queries and cache entries from the K parts of a split QKV product (n_mr: its row tiles of rotary pairs)
template <bool CUT>
__global__ __launch_bounds__(PF_RT) void prefill_qkv_row_kernel(PfRowArgs a, int n_mr) {
    const int tok = pf_row_token(a.n_tok);
    if (tok >= a.n_tok) return;
    const int P = (a.op.H + a.op.Hkv) * (a.op.hd >> 1), VR = a.op.Hkv * a.op.hd;
    for (int i = (blockIdx.y * blockDim.x + threadIdx.x) * 4; i < P + VR; i += gridDim.y * blockDim.x * 4) {     // gridDim.y workgroups per row
        if (i < P) {
            const int c = pf_pair_col(i, a.TM), S = pf_n_parts<CUT>(a, c);
            const f32x4 x0 = pf_sum_parts(a, tok, c, S), x1 = pf_sum_parts(a, tok, c + 16, S);
            pf_rope_store(a.op, tok, i, x0, x1);
        } else {
            const int c = n_mr * a.TM + i - P;
            pf_value_store(a.op, tok, i - P, pf_sum_parts(a, tok, c, pf_n_parts<CUT>(a, c)));
        }
    }
}

// The prompt's last row after the last block: the final norm's operands and shares as a one-row pass of the decode
// kernels reads them (the LM head follows), and the final-norm hidden state.
// (It also sets the control block of that pass: one row at position pos.)
__global__ __launch_bounds__(NT) void prefill_last_row_kernel(PassCtl *ctl, int pos, const float *x_row, const float *gain, int d, float eps,
                                                              float *act, float *ss, float *out0, float *out1) {
    __shared__ float scratch[NWV];
    if (threadIdx.x == 0) { ctl->active = 1; ctl->n_rows = 1; ctl->start = pos; ctl->head_from = 0; }
    float s = 0.f;
    for (int n = threadIdx.x; n < d; n += NT) s = fmaf(x_row[n], x_row[n], s);
    const float sum = block_sum(s, scratch), rs = 1.0f / sqrtf(sum / (float)d + eps);
    if (threadIdx.x < KS_NWG) ss[threadIdx.x] = threadIdx.x == 0 ? sum : 0.f;
    for (int n = threadIdx.x; n < d; n += NT) {
        const float v = gain[n] * x_row[n];
        act[n] = v;
        out0[n] = v * rs;
        if (out1) out1[n] = v * rs;
    }
}

// ------------------------------------------------------------------------------------------
// Causal attention of the prompt rows over the bf16 cache, on the matrix cores. A workgroup = one query head x four
// consecutive 16-row tiles (one wavefront each); keys and values go to LDS in chunks of 64 positions shared by the four
// wavefronts, one chunk ahead. Q and P stay exact as three bf16 planes.
// Everything is computed transposed, S^T = K Q^T and O^T = V^T P^T, so that a lane keeps one query from end to end: the
// accumulators of two 16-position tiles of S^T (4 positions each) are the eight positions that lane needs as the operand of
// the second product, with V's rows taken in the same order; no exchange through LDS, two shuffles per row maximum. V is
// read as it lies: a lane takes HD/16 neighbouring dimensions of its eight positions and regroups them with byte permutes,
// so that matrix instruction t produces the dimensions {HD/16 * n + t}, which end up next to each other in one lane.
// LDS rows are not padded (the loads to LDS are linear); the 16-byte pieces of a row are stored rotated by an exclusive or
// with the row number instead, which spreads the 16 rows of an operand read over the banks.
// Bound by the vector ALUs and the matrix cores about equally. 13B-shaped, 40 heads, before (values transposed on their way
// into LDS by 2-byte stores, P through LDS, expf) and after: 1024 rows 97 -> 45 us, 4096 rows 1.20 -> 0.49 ms.
// ------------------------------------------------------------------------------------------
struct PfAttn {
    const float *q;          // [n_tok][H*hd] rotated queries
    const bf16_t *kv_block;  // [2][Hkv][max_seq][hd]
    bf16_t *frag_out;        // attention output over H*hd features, fragment order
    int H, Hkv, max_seq, n_tok, TT;
};

// eight fp32 values -> the three bf16 planes of an MFMA operand fragment
__device__ __forceinline__ void split_planes8(const float *v, bf16x8 *out3) {
    unsigned int w[PF_NP][4];
    split_planes<8>(v, w);
#pragma unroll
    for (int p = 0; p < PF_NP; ++p) out3[p] = __builtin_bit_cast(bf16x8, u32x4{w[p][0], w[p][1], w[p][2], w[p][3]});
}

// a * b rounded, also where the compiler could fold the product into a following sum
__device__ __forceinline__ float pf_rounded_product(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}

template <int HD> constexpr size_t pf_attn_lds_bytes() { return (size_t)2 * 2 * 64 * HD * 2; }

template <int HD>
__global__ __launch_bounds__(256, 2) void prefill_attn_kernel(PfAttn a) {
    constexpr int CH = 64, QS = HD / 32, DT = HD / 16, SL = HD / 8, RB = HD * 2;
    constexpr int KV = CH * RB;                               // bytes of a chunk's keys (or values)
    constexpr int ROWS = 1024 / RB, NI = KV / 1024 / 4;       // rows one wavefront load covers, loads per wavefront for the keys
    extern __shared__ __align__(16) char lds[];               // [2][keys | values]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, r16 = lane & 15;
    const int n_rt = (a.n_tok + 15) >> 4, n_b = (n_rt + 3) >> 2;
    const int b = n_b - 1 - (int)(blockIdx.x / a.H);          // long blocks first
    const int h = blockIdx.x % a.H, kvh = h / (a.H / a.Hkv);
    const int rt = min(b * 4 + wave, n_rt - 1);               // a wavefront past the last tile repeats it and stores nothing
    const bool live = b * 4 + wave < n_rt;
    const int n_chunks = b + 1;                               // positions 0 .. 64b+63 cover every row of the block
    const int last_pos = a.n_tok - 1, qd = a.H * HD;
    constexpr float c2 = (float)(1.4426950408889634 * (HD == 128 ? 0.08838834764831845 : 0.125));   // softmax in powers of two: log2(e) / sqrt(hd)
    const bf16_t *kg_ = a.kv_block + (size_t)kvh * a.max_seq * HD;
    const bf16_t *vg_ = a.kv_block + ((size_t)a.Hkv + kvh) * a.max_seq * HD;
    const unsigned int l0 = (unsigned int)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    auto swz = [](int row) { return HD == 128 ? row & 15 : (row >> 1) & 7; };

    auto issue = [&](int c, int buf) {                        // chunk c of keys and values into buffer buf
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int row = (i * 4 + wave) * ROWS + lane / SL, piece = (lane % SL) ^ swz(row);
            const size_t off = (size_t)min(c * CH + row, last_pos) * HD + piece * 8;
            const unsigned int d = l0 + buf * 2 * KV + (i * 4 + wave) * 1024;
            dma_lane(kg_ + off, d);
            dma_lane(vg_ + off, d + KV);
        }
    };
    issue(0, 0);
    // the wavefront's 16 query rows as operand fragments: lane (kg, n) holds query n, dims 32*ks + 8*kg .. +7
    bf16x8 qa[QS][3];
    {
        const float *qp = a.q + (size_t)min(rt * 16 + r16, last_pos) * qd + h * HD + kg * 8;     // rows past the prompt repeat its last one
#pragma unroll
        for (int ks = 0; ks < QS; ++ks) {
            float v[8];
            const f32x4 v0 = *reinterpret_cast<const f32x4 *>(qp + ks * 32), v1 = *reinterpret_cast<const f32x4 *>(qp + ks * 32 + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = v0[e]; v[4 + e] = v1[e]; }
            split_planes8(v, qa[ks]);
        }
    }

    const int qpos = rt * 16 + r16;                           // the lane's query
    float mrun = -INFINITY, off = -INFINITY, lsum = 0.f;      // largest score so far, and its exponent
    f32x4 o[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int c = 0; c < n_chunks; ++c) {
        const int buf = c & 1;
        dma_wait<0>();
        pf_meet();                                            // chunk c is here and every wavefront is done with chunk c-1
        if (c + 1 < n_chunks) issue(c + 1, buf ^ 1);
        const char *kl = lds + buf * 2 * KV, *vl = kl + KV;
        // S^T = K Q^T: lane (kg, n) holds positions 16*pt + 4*kg .. +3 of query n
        const int n_pt = c * CH + CH - 1 <= rt * 16 ? 4 : min(4, (rt * 16 + 15 - c * CH) / 16 + 1);     // tiles that hold a visible position
        f32x4 s[4];
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) {
            if (pt < n_pt) {
                f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
                bf16x8 kf[QS];
                const int row = pt * 16 + r16;
#pragma unroll
                for (int ks = 0; ks < QS; ++ks) kf[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kl + row * RB + ((ks * 4 + kg) ^ swz(row)) * 16));
                // the lowest plane first: QS roundings at the size of the whole score instead of 3 QS
#pragma unroll
                for (int p = 2; p >= 0; --p)
#pragma unroll
                    for (int ks = 0; ks < QS; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qa[ks][p], acc, 0, 0, 0);
                s[pt] = acc;
            } else {
                s[pt] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            }
        }
        if (c * CH + CH - 1 > rt * 16) {                      // the diagonal runs through this chunk
#pragma unroll
            for (int pt = 0; pt < 4; ++pt)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (c * CH + pt * 16 + 4 * kg + q > qpos) s[pt][q] = -INFINITY;
        }
        // running softmax of the lane's query (its positions are spread over the four kg lanes)
        float cm = s[0][0];
#pragma unroll
        for (int pt = 0; pt < 4; ++pt)
#pragma unroll
            for (int q = 0; q < 4; ++q) cm = fmaxf(cm, s[pt][q]);
        cm = fmaxf(cm, lane_xor(cm, 16));
        cm = fmaxf(cm, lane_xor(cm, 32));
        const float mnew = fmaxf(mrun, cm);                   // finite: position 0 is visible to every row
        // Weights are 2^(score * c2 - off) with off rounded once per maximum; what earlier chunks hold moves on by the difference
        // of the rounded values, so that all chunks are weighed against one reference. (Weights under 2^-126 of the row's
        // largest are zero.)
        const float off_new = pf_rounded_product(mnew, c2), f = __builtin_amdgcn_exp2f(off - off_new);
        mrun = mnew;
        off = off_new;
        float ps = 0.f;
#pragma unroll
        for (int pt = 0; pt < 4; ++pt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s[pt][q] = __builtin_amdgcn_exp2f(fmaf(s[pt][q], c2, -off));
                ps += s[pt][q];
            }
        lsum = lsum * f + ps;
        if (__any(f != 1.0f)) {
#pragma unroll
            for (int t = 0; t < DT; ++t) o[t] *= f;
        }
        // O^T += V^T P^T, 32 positions at a time: the lane's positions 4*kg..+3 of two tiles, V's rows in the same order
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            if (hf * 2 >= n_pt) continue;
            const float pv[8] = {s[2 * hf][0], s[2 * hf][1], s[2 * hf][2], s[2 * hf][3], s[2 * hf + 1][0], s[2 * hf + 1][1], s[2 * hf + 1][2], s[2 * hf + 1][3]};
            bf16x8 pb[3];
            split_planes8(pv, pb);
            unsigned int vr[8][DT / 2];                       // [position][pairs of dims DT*n + 2w, +1]
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = hf * 32 + (i >> 2) * 16 + 4 * kg + (i & 3);
                if constexpr (HD == 128) {
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(vl + row * RB + (r16 ^ swz(row)) * 16);
#pragma unroll
                    for (int w = 0; w < 4; ++w) vr[i][w] = v[w];
                } else {
                    const u32x2 v = *reinterpret_cast<const u32x2 *>(vl + row * RB + ((r16 >> 1) ^ swz(row)) * 16 + (r16 & 1) * 8);
                    vr[i][0] = v.x; vr[i][1] = v.y;
                }
            }
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                u32x4 vf;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    vf[j] = __builtin_amdgcn_perm(vr[2 * j + 1][t >> 1], vr[2 * j][t >> 1], (t & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
                for (int p = 2; p >= 0; --p)
                    o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), pb[p], o[t], 0, 0, 0);
            }
        }
    }
    lsum += lane_xor(lsum, 16);
    lsum += lane_xor(lsum, 32);
    if (live && qpos <= last_pos) {
        const float inv = 1.0f / lsum;
        // accumulator row 4*kg + q of instruction t is dimension DT * (4*kg + q) + t: eight neighbours at a time
#pragma unroll
        for (int q = 0; q < 4; q += 8 / DT) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = o[e % DT][q + e / DT] * inv;
            store_frag8(a.frag_out, qd >> 5, a.TT, rt, r16, h * HD + DT * (4 * kg + q), v);
        }
    }
}

}  // namespace ks
