// Prompt prefill for the tuned bf16 path (gfx950): the full model over hundreds to thousands of rows.
//
// Unlike a decode pass this is bound by the matrix cores, so it has kernels of its own. They read the
// SAME stream-order weights as the decode kernels (a unit = <= 16 rows x 32 columns is one MFMA A
// operand) and keep the same arithmetic: activations stay fp32-exact as three bf16 planes, so an
// output takes three MFMAs per 32 columns and the products are exact in the fp32 accumulator.
//
// Activations of all rows live in "fragment order": [plane][32-column step][16-row tile][lane][8],
// lane = 16*kg + r holding row r of the tile and columns 8*kg..8*kg+7 of the step, i.e. the MFMA B
// operand of v_mfma_f32_16x16x32_bf16 as stored, so staging a tile is a linear copy.
//
// prefill_gemm_kernel: a workgroup owns TA tiles of 16 weight rows x TB tiles of 16 tokens and walks K (or one of S parts
// of it) in steps of 32 columns. Weights and activations go from memory straight to LDS (16-byte loads whose LDS side is
// linear and whose memory side is free), so a tile is filled with whatever rows suit it, wherever they lie in the decode
// layout: no dead rows from the decode layout's short tiles (20 rows per workgroup = two tiles of 10), and the two dot
// products an epilogue combines sit in one lane's accumulators, so epilogues run in registers on four rows at a time.
#pragma once
#include "kernels_bf16.h"

namespace ks {

constexpr int PF_NT = 512;             // threads per workgroup of the prefill GEMM (8 wavefronts)

struct PfArgs {
    GemmOp op;              // type, W, N, K, split, x, gain_next, q_out, kv_block, cos_t, sin_t, H, Hkv, hd, max_seq, inv_dim, eps
    const bf16_t *frag_in;  // [3][K/32][TT][512] fragment order
    bf16_t *frag_out;       // same layout over the output features (OP_RESID / OP_SWIGLU)
    const float *ss_in;     // [n_ss][TT*16] shares of sum(x^2) per input row; nullptr: input is not normalised
    int n_ss;
    float *ss_out;          // OP_RESID: [row tiles][TT*16] this workgroup's share of sum(x^2) per row
    float *part;            // split K: [tile][S][wavefront][accumulator tile][lane][4] partial sums
    int *arrivals;          // split K: [tile] arrival counters, zero between launches
    int TT;                 // token tiles the fragment buffers are laid out for
    int n_tok;              // live rows
    int n_mt, n_mr;         // row tiles of the matrix; OP_QKV: those that hold rotary pairs (the others hold value rows)
    int n_tt, S;            // token tiles (workgroup tiles) of the launch, parts K is split into
};

__device__ __forceinline__ size_t frag_off(int KS, int TT, int pl, int ks, int tt) {
    return (((size_t)pl * KS + ks) * TT + tt) * 512;
}

// the three bf16 planes of v at feature n of row (tt, m), fragment order
__device__ __forceinline__ void store_frag(bf16_t *frag, int KS, int TT, int tt, int m, int n, float v) {
    const unsigned int u = __float_as_uint(v);
    const float hi = __uint_as_float(u & 0xffff0000u);
    const float r1 = v - hi;
    const float mid = __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
    const float lo = r1 - mid;
    const size_t in_tile = (size_t)((((n & 31) >> 3) * 16 + m) * 8 + (n & 7));
    frag[frag_off(KS, TT, 0, n >> 5, tt) + in_tile] = (bf16_t)(u >> 16);
    frag[frag_off(KS, TT, 1, n >> 5, tt) + in_tile] = (bf16_t)(__float_as_uint(mid) >> 16);
    frag[frag_off(KS, TT, 2, n >> 5, tt) + in_tile] = (bf16_t)(__float_as_uint(lo) >> 16);
}

// ... of the four values at features n..n+3 (n a multiple of 4): one 8-byte store per plane
__device__ __forceinline__ void store_frag4(bf16_t *frag, int KS, int TT, int tt, int m, int n, f32x4 v) {
    unsigned int h[4], md[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        h[e] = __float_as_uint(v[e]);
        const float r1 = v[e] - __uint_as_float(h[e] & 0xffff0000u);
        md[e] = __float_as_uint(r1);
        l[e] = __float_as_uint(r1 - __uint_as_float(md[e] & 0xffff0000u));
    }
    const size_t in_tile = (size_t)((((n & 31) >> 3) * 16 + m) * 8 + (n & 7));
    auto put = [&](int pl, const unsigned int *u) {
        *reinterpret_cast<u32x2 *>(frag + frag_off(KS, TT, pl, n >> 5, tt) + in_tile) =
            u32x2{__builtin_amdgcn_perm(u[1], u[0], 0x07060302u), __builtin_amdgcn_perm(u[3], u[2], 0x07060302u)};
    };
    put(0, h); put(1, md); put(2, l);
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

// Partial sums that another workgroup of the launch reads: written through to memory and read from there, whichever die's
// L2 the two sit behind.
__device__ __forceinline__ void store_part(char *base, unsigned int off, f32x4 v) {
    asm volatile("s_nop 4\n\tglobal_store_dwordx4 %0, %1, %2 sc1" : : "v"(off), "v"(v), "s"(base) : "memory");
}
// N pieces, 1 KB apart (the wait is part of the block: no register is ever seen with a load in flight)
template <int N> __device__ __forceinline__ void load_part(const char *base, unsigned int off, f32x4 *v);
template <> __device__ __forceinline__ void load_part<4>(const char *base, unsigned int off, f32x4 *v) {
    asm volatile(
        "s_nop 4\n\tglobal_load_dwordx4 %0, %4, %5 offset:-4096 sc1\n\t"
        "global_load_dwordx4 %1, %4, %5 offset:-3072 sc1\n\t"
        "global_load_dwordx4 %2, %4, %5 offset:-2048 sc1\n\t"
        "global_load_dwordx4 %3, %4, %5 offset:-1024 sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
        : "v"(off), "s"(base + 4096) : "memory");
}
template <> __device__ __forceinline__ void load_part<16>(const char *base, unsigned int off, f32x4 *v) {
    asm volatile(
        "s_nop 4\n\tglobal_load_dwordx4 %0, %16, %17 offset:-4096 sc1\n\t"
        "global_load_dwordx4 %1, %16, %17 offset:-3072 sc1\n\t"
        "global_load_dwordx4 %2, %16, %17 offset:-2048 sc1\n\t"
        "global_load_dwordx4 %3, %16, %17 offset:-1024 sc1\n\t"
        "global_load_dwordx4 %4, %16, %17 offset:0 sc1\n\t"
        "global_load_dwordx4 %5, %16, %17 offset:1024 sc1\n\t"
        "global_load_dwordx4 %6, %16, %17 offset:2048 sc1\n\t"
        "global_load_dwordx4 %7, %16, %17 offset:3072 sc1\n\t"
        "global_load_dwordx4 %8, %16, %18 offset:-4096 sc1\n\t"
        "global_load_dwordx4 %9, %16, %18 offset:-3072 sc1\n\t"
        "global_load_dwordx4 %10, %16, %18 offset:-2048 sc1\n\t"
        "global_load_dwordx4 %11, %16, %18 offset:-1024 sc1\n\t"
        "global_load_dwordx4 %12, %16, %18 offset:0 sc1\n\t"
        "global_load_dwordx4 %13, %16, %18 offset:1024 sc1\n\t"
        "global_load_dwordx4 %14, %16, %18 offset:2048 sc1\n\t"
        "global_load_dwordx4 %15, %16, %18 offset:3072 sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7]), "=&v"(v[8]), "=&v"(v[9]), "=&v"(v[10]), "=&v"(v[11]), "=&v"(v[12]), "=&v"(v[13]), "=&v"(v[14]), "=&v"(v[15])
        : "v"(off), "s"(base + 4096), "s"(base + 12288) : "memory");
}

// Where one row of a workgroup's tile lies in the packed matrix: the 16-byte piece (8 columns 8*kg..) of step 0's unit
struct PfRow { const bf16_t *p; int unit, gshift; };

// workgroup of the decode layout that owns item n of N (inverse of wg_share)
__device__ __forceinline__ int pf_owner(int n, int N) { return (int)((((unsigned int)n + 1u) * (unsigned int)KS_NWG - 1u) / (unsigned int)N); }

// Row sr of row tile mt (TM rows). Which matrix row that is, is free to choose, since every row is fetched from wherever
// it lies: pairs whose two dot products meet in an epilogue (rotary halves, gate / up rows) sit in neighbouring 16-row
// tiles at the same place, so that one lane holds both. Rows past the end repeat the last one (never stored).
template <int TM>
__device__ __forceinline__ PfRow pf_row(const PfArgs &a, int mt, int sr, int kg) {
    const GemmOp &op = a.op;
    const bool pairs = op.type == OP_SWIGLU || (op.type == OP_QKV && mt < a.n_mr);
    int wg, lr;
    if (pairs) {
        const int P = op.type == OP_SWIGLU ? op.N : (op.H + op.Hkv) * (op.hd >> 1);
        const int p = min(mt * (TM / 2) + (sr >> 5) * 16 + (sr & 15), P - 1);
        wg = pf_owner(p, P);
        lr = p - wg_share(P, wg) + ((sr >> 4) & 1) * a.op.split[wg].n_first;
    } else if (op.type == OP_QKV) {
        const int VR = op.Hkv * op.hd, v = min((mt - a.n_mr) * TM + sr, VR - 1);
        wg = pf_owner(v, VR);
        lr = v - wg_share(VR, wg) + 2 * a.op.split[wg].n_first;
    } else {
        const int n = min(mt * TM + sr, op.N - 1);
        wg = pf_owner(n, op.N);
        lr = n - wg_share(op.N, wg);
    }
    const WgSplit &s = a.op.split[wg];
    const int t = lr / s.rpt, rit = lr - t * s.rpt, rows_t = min(s.rpt, s.R - t * s.rpt);
    PfRow r;
    r.p = op.W + s.wg_base + (size_t)(t * s.rpt) * op.K + (size_t)(kg * rows_t + rit) * 8;
    r.unit = rows_t * 32;
    r.gshift = s.gshift;
    return r;
}

// position of 32-column step st among the units of a tile (the order pack_matrix_kernel wrote them in)
__device__ __forceinline__ int pf_unit_index(int st, int KS, int gshift) {
    const int nfull = KS >> 4, rem = KS & 15, g = 1 << gshift, w16 = st & 15, kpart = w16 >> gshift;
    return nfull * g * kpart + min(rem, kpart * g) + (st >> 4) * g + (w16 & (g - 1));
}

// TA x TB tiles of 16 rows x 16 tokens per workgroup, 8 wavefronts in a WA x 8/WA grid, NS staged steps in LDS.
// PP: the wavefronts form two groups (one wavefront of each on every SIMD) that run one phase apart: while one group
// issues its matrix instructions the other reads its operands from LDS.
// What bounds it: at 256 x 256 the matrix cores (96 matrix instructions of 16 cycles per wavefront and step against 20 KB
// of LDS reads); 13B-shaped, 4096 rows: 1.50-1.55 PFLOP/s issued (three planes) on QKV and gate+up, where a large library
// product in bf16 reaches 1.59 on this card; one meeting per step for all wavefronts together ran at 1.18. Up to 64 rows
// it is the weight stream: 128-row tiles, two workgroups per unit, K split until every unit has work.
// Whole prompts, 4 blocks, before (a tile per decode-layout tile, the last rows in a 16-row pass of their own) and after:
// 7B 45 rows 4.47 -> 0.82 ms, Qwen-14B 777 rows 8.24 -> 5.28, 13B 1024 rows 9.41 -> 6.17, 13B 4096 rows 37.3 -> 27.2.
template <int TA, int TB, int WA, int NS, bool PP>
struct PfShape {
    static constexpr int WB = 8 / WA, TAW = TA / WA, TBW = TB / WB;
    static constexpr int TM = TA * 16;
    static constexpr int A_BYTES = TA * 1024, STAGE = A_BYTES + 3 * TB * 1024;
    static constexpr int NA = TA * 64 / PF_NT;                   // weight pieces per thread and step
    static constexpr int NB = (3 * TB + 7) / 8;                  // token fragments per wavefront and step
    static constexpr size_t LDS = (size_t)NS * STAGE + (size_t)TB * 16 * 4 * (1 + WA);
};

template <int TA, int TB, int WA, int NS, bool PP>
__global__ __launch_bounds__(PF_NT, TA == 16 ? 2 : 4) void prefill_gemm_kernel(PfArgs a) {
    typedef PfShape<TA, TB, WA, NS, PP> Sh;
    constexpr int TAW = Sh::TAW, TBW = Sh::TBW, TM = Sh::TM;
    extern __shared__ __align__(16) char lds[];
    float *rs = reinterpret_cast<float *>(lds + NS * Sh::STAGE);     // [TB*16] norm scale of the tile's tokens
    float *sq = rs + TB * 16;                                        // [WA][TB*16]
    __shared__ int ticket;
    const GemmOp &op = a.op;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wa = PP ? wave >> 2 : wave / Sh::WB, wb = PP ? wave & 3 : wave % Sh::WB, kg = lane >> 4, r16 = lane & 15;
    const int KS = op.K >> 5;

    // workgroup -> (K part, token tile, row tile). Workgroups are dealt to the 8 dies by index: each die takes a run of
    // the order below, in which neighbours share weights (four token tiles) or activations (consecutive row tiles)
    const int total = a.n_mt * a.n_tt * a.S;
    const int per = (total + 7) >> 3, lin = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || lin >= total) return;
    const int part_tiles = a.n_mt * a.n_tt;
    const int sp = lin / part_tiles, in_part = lin - sp * part_tiles;
    const int tb4 = in_part / (a.n_mt * 4), in_blk = in_part - tb4 * (a.n_mt * 4), tw = min(4, a.n_tt - tb4 * 4);
    const int mt = in_blk / tw, tk = tb4 * 4 + (in_blk - mt * tw);
    const int tt0 = tk * TB;
    const int st0 = (int)((long long)KS * sp / a.S), cnt = (int)((long long)KS * (sp + 1) / a.S) - st0;

    // what this thread stages per step
    PfRow ar[Sh::NA];
#pragma unroll
    for (int q = 0; q < Sh::NA; ++q) ar[q] = pf_row<TM>(a, mt, (wave + q * 8) * 16 + r16, kg);
    const unsigned int l0 = (unsigned int)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const char *bsrc[Sh::NB];
    unsigned int bdst[Sh::NB];
#pragma unroll
    for (int q = 0; q < Sh::NB; ++q) {
        const int f = min(wave + q * 8, 3 * TB - 1), pl = f / TB, t = f - pl * TB;    // a repeat writes the same bytes again
        bsrc[q] = reinterpret_cast<const char *>(a.frag_in + frag_off(KS, a.TT, pl, st0, min(tt0 + t, a.TT - 1)));
        bdst[q] = Sh::A_BYTES + f * 1024;
    }
    const size_t bstep = (size_t)a.TT * 1024;
    const unsigned int voff = lane * 16;
    const bool once = a.n_tt == 1;                 // every weight byte is used by one workgroup only: nothing to keep in a cache
    auto issue = [&](int t, int buf) {             // step st0 + t into LDS buffer buf
        const unsigned int d = l0 + buf * Sh::STAGE;
#pragma unroll
        for (int q = 0; q < Sh::NA; ++q) {
            const bf16_t *p = ar[q].p + (size_t)pf_unit_index(st0 + t, KS, ar[q].gshift) * ar[q].unit;
            if (once) dma_lane_nt(p, d + (wave + q * 8) * 1024);
            else dma_lane(p, d + (wave + q * 8) * 1024);
        }
#pragma unroll
        for (int q = 0; q < Sh::NB; ++q) dma_linear(bsrc[q] + t * bstep, voff, d + bdst[q]);
    };

    f32x4 acc[TAW][TBW];
#pragma unroll
    for (int i = 0; i < TAW; ++i)
#pragma unroll
        for (int j = 0; j < TBW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const char *la = lds + wa * TAW * 1024 + lane * 16, *lb = lds + Sh::A_BYTES + wb * TBW * 1024 + lane * 16;
    auto read_a = [&](int buf, bf16x8 *v) {
#pragma unroll
        for (int i = 0; i < TAW; ++i) v[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(la + buf * Sh::STAGE + i * 1024));
    };
    auto read_b = [&](int buf, int j, bf16x8 *v) {
#pragma unroll
        for (int p = 0; p < 3; ++p) v[p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(lb + buf * Sh::STAGE + (p * TB + j) * 1024));
    };

    constexpr int NDMA = Sh::NA + Sh::NB;          // loads per wavefront and step
    constexpr int JC = TBW < 2 ? TBW : 2, CL = TBW / JC;      // token tiles per cluster of matrix instructions, clusters per step
    bf16x8 av[TAW], bv[JC][3];
    auto mfma_cluster = [&](int c) {
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int jj = 0; jj < JC; ++jj)
#pragma unroll
                for (int i = 0; i < TAW; ++i)
                    acc[i][c * JC + jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv[jj][p], acc[i][c * JC + jj], 0, 0, 0);
    };
#pragma unroll
    for (int t = 0; t < NS - 1; ++t) issue(min(t, cnt - 1), t);     // (a step past the end re-reads the last one: loads stay countable)
    // norm scale of the tile's tokens, from the producers' shares in their order (read while the first steps arrive)
    if (a.ss_in && tid < TB * 16) {
        float s = 0.f;
        const float *p = a.ss_in + tt0 * 16 + tid;
        const int stride = a.TT * 16;
        for (int i0 = 0; i0 < a.n_ss; i0 += 16) {      // sixteen loads at a time: one memory round trip, not sixteen
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = p[(size_t)min(i0 + i, a.n_ss - 1) * stride];
#pragma unroll
            for (int i = 0; i < 16; ++i) s += i0 + i < a.n_ss ? v[i] : 0.f;
        }
        rs[tid] = 1.0f / sqrtf(s * op.inv_dim + op.eps);
    }
    dma_wait<0>();
    pf_meet();
    if constexpr (PP) {
        // Phases of a group: read operands | meet | matrix instructions | meet. The second group enters one phase later.
        // With two buffers (two clusters per step) step t+1 is requested while cluster 0 of step t is read, when the
        // last reads of step t-1 are one phase old; with three (one cluster per step) step t+2 is.
        if (wa == 1) pf_meet();
        int buf = 0;
        for (int t = 0; t < cnt; ++t) {
            read_a(buf, av);
#pragma unroll
            for (int jj = 0; jj < JC; ++jj) read_b(buf, jj, bv[jj]);
            const int nb = NS == 2 ? buf ^ 1 : (buf == 0 ? 2 : buf - 1);
            issue(min(t + NS - 1, cnt - 1), nb);
            if (CL == 1) dma_wait<NDMA>();         // step t+1 has arrived (t+2 stays in flight)
            pf_meet();
            __builtin_amdgcn_s_setprio(1);
            mfma_cluster(0);
            __builtin_amdgcn_s_setprio(0);
            pf_meet();
            if constexpr (CL == 2) {
#pragma unroll
                for (int jj = 0; jj < JC; ++jj) read_b(buf, JC + jj, bv[jj]);
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
        int buf = 0;
        for (int t = 0; t < cnt; ++t) {
            if (t > 0) { dma_wait<(NS - 2) * NDMA>(); pf_meet(); }      // step t has arrived; every wavefront is done with step t-1
            const int nb = buf == 0 ? NS - 1 : buf - 1;
            issue(min(t + NS - 1, cnt - 1), nb);
            read_a(buf, av);
#pragma unroll
            for (int c = 0; c < CL; ++c) {
#pragma unroll
                for (int jj = 0; jj < JC; ++jj) read_b(buf, c * JC + jj, bv[jj]);
                mfma_cluster(c);
            }
            buf = buf == NS - 1 ? 0 : buf + 1;
        }
    }
    dma_wait<0>();                                 // nothing is in flight towards LDS from here on

    if (a.S > 1) {
        // partial sums of this K part, written through; the workgroup that arrives last adds the parts up in order
        const int tile = mt * a.n_tt + tk;
        constexpr int NACC = TAW * TBW, NBT = NACC < 16 ? NACC : 16;        // tiles fetched per round trip
        char *pw = reinterpret_cast<char *>(a.part) + (size_t)tile * a.S * (NACC * PF_NT * 16) + wave * (NACC * 1024);
        char *mine = pw + (size_t)sp * (NACC * PF_NT * 16);
#pragma unroll
        for (int i = 0; i < TAW; ++i)
#pragma unroll
            for (int j = 0; j < TBW; ++j) store_part(mine + (i * TBW + j) * 1024, voff, acc[i][j]);
        if (!last_arrival(a.arrivals + tile, a.S, &ticket)) return;
#pragma unroll
        for (int i = 0; i < TAW; ++i)
#pragma unroll
            for (int j = 0; j < TBW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < a.S; ++k) {
#pragma unroll
            for (int t0 = 0; t0 < NACC; t0 += NBT) {
                f32x4 v[NBT];
                load_part<NBT>(pw + (size_t)k * (NACC * PF_NT * 16) + t0 * 1024, voff, v);
#pragma unroll
                for (int t = 0; t < NBT; ++t) acc[(t0 + t) / TBW][(t0 + t) % TBW] += v[t];
            }
        }
    }

    // epilogue: lane (kg, r16) holds rows 4*kg..4*kg+3 of its TAW row tiles for token r16 of its TBW token tiles
    const bool pairs = op.type == OP_SWIGLU || (op.type == OP_QKV && mt < a.n_mr);
#pragma unroll
    for (int j = 0; j < TBW; ++j) {
        const int ttl = wb * TBW + j, tt = tt0 + ttl, tok = tt * 16 + r16;
        const bool live = tok < a.n_tok;
        const float scale = a.ss_in ? rs[ttl * 16 + r16] : 1.0f;
        float s = 0.f;
        if (op.type == OP_RESID) {
#pragma unroll
            for (int i = 0; i < TAW; ++i) {
                const int n = mt * TM + (wa * TAW + i) * 16 + 4 * kg;
                if (live && n < op.N) {
                    f32x4 *xp = reinterpret_cast<f32x4 *>(op.x + (size_t)tok * op.N + n);
                    const f32x4 xn = *xp + acc[i][j];
                    *xp = xn;
                    store_frag4(a.frag_out, op.N >> 5, a.TT, tt, r16, n, *reinterpret_cast<const f32x4 *>(op.gain_next + n) * xn);
#pragma unroll
                    for (int q = 0; q < 4; ++q) s = fmaf(xn[q], xn[q], s);
                }
            }
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (kg == 0) sq[wa * TB * 16 + ttl * 16 + r16] = s;
        } else if (pairs) {
#pragma unroll
            for (int i = 0; i < TAW; i += 2) {
                const int p = mt * (TM / 2) + (wa * TAW + i) * 8 + 4 * kg;
                if (op.type == OP_SWIGLU) {
                    if (live && p < op.N) {
                        f32x4 u;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float g = acc[i][j][q] * scale;
                            u[q] = (g / (1.0f + expf(-g))) * (acc[i + 1][j][q] * scale);
                        }
                        store_frag4(a.frag_out, op.N >> 5, a.TT, tt, r16, p, u);
                    }
                } else {
                    const int half = op.hd >> 1, qd = op.H * op.hd;
                    if (live && p < (op.H + op.Hkv) * half) {
                        const int head = p / half, d = p - head * half;            // four neighbours of one head: half is a multiple of 4
                        const f32x4 c = *reinterpret_cast<const f32x4 *>(op.cos_t + (size_t)tok * half + d);
                        const f32x4 sn = *reinterpret_cast<const f32x4 *>(op.sin_t + (size_t)tok * half + d);
                        f32x4 ra, rb;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float x0 = acc[i][j][q] * scale, x1 = acc[i + 1][j][q] * scale;
                            ra[q] = x0 * c[q] - x1 * sn[q];
                            rb[q] = x1 * c[q] + x0 * sn[q];
                        }
                        if (head < op.H) {
                            float *qp = op.q_out + (size_t)tok * qd + head * op.hd + d;
                            *reinterpret_cast<f32x4 *>(qp) = ra;
                            *reinterpret_cast<f32x4 *>(qp + half) = rb;
                        } else {
                            bf16_t *kp = op.kv_block + ((size_t)(head - op.H) * op.max_seq + tok) * op.hd + d;   // the prompt starts at position 0
                            pf_store_bf16x4(kp, ra);
                            pf_store_bf16x4(kp + half, rb);
                        }
                    }
                }
            }
        } else {    // value rows of OP_QKV
#pragma unroll
            for (int i = 0; i < TAW; ++i) {
                const int v = (mt - a.n_mr) * TM + (wa * TAW + i) * 16 + 4 * kg;
                if (live && v < op.Hkv * op.hd) {
                    const int head = v / op.hd, d = v - head * op.hd;
                    pf_store_bf16x4(op.kv_block + (((size_t)op.Hkv + head) * op.max_seq + tok) * op.hd + d, acc[i][j] * scale);
                }
            }
        }
    }
    if (op.type == OP_RESID) {
        __syncthreads();
        if (tid < TB * 16) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < WA; ++w) s += sq[w * TB * 16 + tid];
            a.ss_out[(size_t)mt * a.TT * 16 + tt0 * 16 + tid] = s;
        }
    }
}

// ------------------------------------------------------------------------------------------
// Embedding of the prompt rows: x = E[tok], the first norm's operands gain (.) x in fragment order
// and the row's sum(x^2) as its only share. One workgroup per row; d is a multiple of 32.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prefill_embed_kernel(const int32_t *toks, const bf16_t *embed, const float *gain, int d,
                                                            int TT, float *x, bf16_t *frag, float *ss) {
    __shared__ float part[4];
    const int tok = blockIdx.x, tt = tok >> 4, m = tok & 15;
    const bf16_t *row = embed + (size_t)toks[tok] * d;
    float sq = 0.f;
    for (int n = threadIdx.x * 4; n < d; n += 256 * 4) {
        const u32x2 w = *reinterpret_cast<const u32x2 *>(row + n);
        const f32x4 v = f32x4{bf_lo(w.x), bf_hi(w.x), bf_lo(w.y), bf_hi(w.y)};
        *reinterpret_cast<f32x4 *>(x + (size_t)tok * d + n) = v;
        store_frag4(frag, d >> 5, TT, tt, m, n, *reinterpret_cast<const f32x4 *>(gain + n) * v);
#pragma unroll
        for (int q = 0; q < 4; ++q) sq = fmaf(v[q], v[q], sq);
    }
    sq = wave_sum(sq);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) ss[tok] = (part[0] + part[1]) + (part[2] + part[3]);
}

// The prompt's last row after the last block: the final norm's operands and shares as a one-row pass of the decode
// kernels reads them (the LM head follows), and the final-norm hidden state.
__global__ __launch_bounds__(NT) void prefill_last_row_kernel(const float *x_row, const float *gain, int d, float eps, float *act,
                                                              float *ss, float *out0, float *out1) {
    __shared__ float scratch[NWV];
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
// Causal attention of the prompt rows over the bf16 cache, on the matrix cores. A workgroup = one query
// head x four consecutive 16-row tiles (one wavefront each); keys and values go through LDS in chunks
// of 64 positions shared by the four wavefronts (values transposed on the way in, so that both are
// MFMA B operands as stored). Per chunk a wavefront computes S = Q K^T (Q exact as three bf16 planes),
// the running softmax in fp32 on the vector ALUs, and O += P V with P exact as three bf16 planes;
// P changes from accumulator layout to operand layout through a wavefront-private LDS tile.
// ------------------------------------------------------------------------------------------
struct PfAttn {
    const float *q;          // [n_tok][H*hd] rotated queries
    const bf16_t *kv_block;  // [2][Hkv][max_seq][hd]
    bf16_t *frag_out;        // attention output in fragment order over H*hd features
    int H, Hkv, max_seq, TT, n_tok;
};

// eight fp32 values -> the three bf16 planes of an MFMA operand fragment (exact: hi + mid + lo = value)
__device__ __forceinline__ void split_planes8(const float *v, bf16x8 *out3) {
    unsigned int w[3][4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const unsigned int u = __float_as_uint(v[e]);
        const float hi = __uint_as_float(u & 0xffff0000u);
        const float r1 = v[e] - hi;
        const unsigned int um = __float_as_uint(r1);
        const float mid = __uint_as_float(um & 0xffff0000u);
        const unsigned int ul = __float_as_uint(r1 - mid);
        const unsigned int h16 = u >> 16, m16 = um >> 16, l16 = ul >> 16;
        if (e & 1) { w[0][e >> 1] |= h16 << 16; w[1][e >> 1] |= m16 << 16; w[2][e >> 1] |= l16 << 16; }
        else { w[0][e >> 1] = h16; w[1][e >> 1] = m16; w[2][e >> 1] = l16; }
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) out3[p] = __builtin_bit_cast(bf16x8, u32x4{w[p][0], w[p][1], w[p][2], w[p][3]});
}

template <int HD>
__global__ __launch_bounds__(256) void prefill_attn_kernel(PfAttn a) {
    constexpr int CH = 64, LPP = HD / 8, QS = HD / 32, DT = HD / 16;
    constexpr int KSTR = HD * 2 + 16;      // bytes per staged key row (+16: the 16 rows of an operand read spread over the banks)
    constexpr int VSTR = CH * 2 + 16;      // bytes per staged (transposed) value row
    constexpr int PSTR = CH + 4;           // floats per row of the P tile
    constexpr int PIECES = CH * LPP, PQ = PIECES / 256;
    __shared__ __align__(16) char kl[CH * KSTR];
    __shared__ __align__(16) char vl[HD * VSTR];
    __shared__ __align__(16) float pb[4][16 * PSTR];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, r16 = lane & 15;
    const int n_rt = (a.n_tok + 15) >> 4, n_b = (n_rt + 3) >> 2;
    const int b = n_b - 1 - (int)(blockIdx.x / a.H);          // long blocks first
    const int h = blockIdx.x % a.H, kvh = h / (a.H / a.Hkv);
    const int rt = min(b * 4 + wave, n_rt - 1);               // a wavefront past the last tile repeats it and stores nothing
    const bool live = b * 4 + wave < n_rt;
    const int n_chunks = b + 1;                               // positions 0 .. 64b+63 cover every row of the block
    const int last_pos = a.n_tok - 1, qd = a.H * HD;
    const float scale = 1.0f / sqrtf((float)HD);
    const bf16_t *kg_ = a.kv_block + (size_t)kvh * a.max_seq * HD;
    const bf16_t *vg_ = a.kv_block + ((size_t)a.Hkv + kvh) * a.max_seq * HD;

    // the wavefront's 16 query rows as operand fragments: lane (kg, i) holds row i, dims 32*ks + 8*kg .. +7
    bf16x8 qa[QS][3];
    {
        const float *qp = a.q + (size_t)min(rt * 16 + r16, last_pos) * qd + h * HD + kg * 8;     // rows past the prompt repeat its last one
#pragma unroll
        for (int ks = 0; ks < QS; ++ks) {
            float v[8];
            const float4 v0 = *reinterpret_cast<const float4 *>(qp + ks * 32), v1 = *reinterpret_cast<const float4 *>(qp + ks * 32 + 4);
            v[0] = v0.x; v[1] = v0.y; v[2] = v0.z; v[3] = v0.w; v[4] = v1.x; v[5] = v1.y; v[6] = v1.z; v[7] = v1.w;
            split_planes8(v, qa[ks]);
        }
    }

    u32x4 kr[PQ], vr[PQ];
    auto chunk_load = [&](int c) {
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const int i = tid + q * 256;
            const int pos = min(c * CH + i / LPP, last_pos);
            kr[q] = *reinterpret_cast<const u32x4 *>(kg_ + (size_t)pos * HD + (i % LPP) * 8);
            vr[q] = *reinterpret_cast<const u32x4 *>(vg_ + (size_t)pos * HD + (i % LPP) * 8);
        }
    };
    auto chunk_store = [&]() {
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const int i = tid + q * 256, pos = i / LPP, d0 = (i % LPP) * 8;
            *reinterpret_cast<u32x4 *>(kl + pos * KSTR + d0 * 2) = kr[q];
            const unsigned int w[4] = {vr[q].x, vr[q].y, vr[q].z, vr[q].w};
#pragma unroll
            for (int e = 0; e < 8; ++e)        // transpose: value of dim d0+e at position pos
                *reinterpret_cast<bf16_t *>(vl + (d0 + e) * VSTR + pos * 2) = (bf16_t)((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xffffu));
        }
    };

    float mrun[4], lsum[4];
    f32x4 o[DT];
#pragma unroll
    for (int q = 0; q < 4; ++q) { mrun[q] = -INFINITY; lsum[q] = 0.f; }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float *pw = pb[wave];
    const int row_tok = rt * 16 + 4 * kg;                     // position of accumulator row q of this lane: row_tok + q

    chunk_load(0);
    for (int c = 0; c < n_chunks; ++c) {
        __syncthreads();                                      // the previous chunk has been consumed by every wavefront
        chunk_store();
        __syncthreads();
        chunk_load(min(c + 1, n_chunks - 1));
        // S = Q K^T for the chunk's four position tiles: lane (kg, j) holds rows 4*kg..4*kg+3 at position 16*pt + j
        float sc[4][4];
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) {
            f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < QS; ++ks) {
                const bf16x8 kb = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kl + (pt * 16 + r16) * KSTR + (ks * 32 + kg * 8) * 2));
#pragma unroll
                for (int p = 0; p < 3; ++p) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[ks][p], kb, acc, 0, 0, 0);
            }
            const int pos = c * CH + pt * 16 + r16;
#pragma unroll
            for (int q = 0; q < 4; ++q) sc[pt][q] = (pos <= row_tok + q) ? acc[q] * scale : -INFINITY;
        }
        // running softmax per row (rows are replicated over the 16 lanes of a kg group)
        float f[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float cm = fmaxf(fmaxf(sc[0][q], sc[1][q]), fmaxf(sc[2][q], sc[3][q]));
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) cm = fmaxf(cm, __shfl_xor(cm, off, 64));
            const float mnew = fmaxf(mrun[q], cm);            // finite: position 0 is visible to every row
            f[q] = (mrun[q] > -INFINITY) ? expf(mrun[q] - mnew) : 0.f;
            mrun[q] = mnew;
            float ps = 0.f;
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) {
                const float e = (sc[pt][q] > -INFINITY) ? expf(sc[pt][q] - mnew) : 0.f;
                pw[(4 * kg + q) * PSTR + pt * 16 + r16] = e;
                ps += e;
            }
            lsum[q] = lsum[q] * f[q] + ps;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int q = 0; q < 4; ++q) o[dt][q] *= f[q];
        // O += P V: P back from LDS in operand layout (lane (kg, i): row i, positions 32*ks2 + 8*kg .. +7)
#pragma unroll
        for (int ks2 = 0; ks2 < 2; ++ks2) {
            float pv[8];
            const float4 p0 = *reinterpret_cast<const float4 *>(pw + r16 * PSTR + ks2 * 32 + kg * 8);
            const float4 p1 = *reinterpret_cast<const float4 *>(pw + r16 * PSTR + ks2 * 32 + kg * 8 + 4);
            pv[0] = p0.x; pv[1] = p0.y; pv[2] = p0.z; pv[3] = p0.w; pv[4] = p1.x; pv[5] = p1.y; pv[6] = p1.z; pv[7] = p1.w;
            bf16x8 pa[3];
            split_planes8(pv, pa);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const bf16x8 vb = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(vl + (dt * 16 + r16) * VSTR + (ks2 * 32 + kg * 8) * 2));
#pragma unroll
                for (int p = 0; p < 3; ++p) o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa[p], vb, o[dt], 0, 0, 0);
            }
        }
    }
    // row sums over the 16 lanes of a kg group, then the rows' outputs in fragment order
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) lsum[q] += __shfl_xor(lsum[q], off, 64);
    }
    if (live) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float inv = 1.0f / lsum[q];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
                store_frag(a.frag_out, qd >> 5, a.TT, rt, 4 * kg + q, h * HD + dt * 16 + r16, o[dt][q] * inv);
        }
    }
}

}  // namespace ks
