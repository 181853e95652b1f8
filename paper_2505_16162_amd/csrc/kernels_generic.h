// Generic (any shape, fp32 or bf16 storage) kernels of the decode path, written for gfx950:
// 64-wide wavefronts, 16-byte coalesced weight loads, wavefront reductions.
// These are the kernels of the fp32 path and the building blocks the tuned bf16 kernels
// fall back to when a shape does not fit their tiling.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_types.h"
#include "prompt_plan.h"

namespace ks {

typedef uint16_t bf16_t;  // raw bit pattern

__device__ __forceinline__ float bf16_to_float(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// fp32 -> bf16, round to nearest even (inf/nan pass through with the payload truncated)
__device__ __forceinline__ bf16_t float_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (bf16_t)(u >> 16);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

__device__ __forceinline__ float load_as_float(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_as_float(const bf16_t *p, size_t i) { return bf16_to_float(p[i]); }
__device__ __forceinline__ void store_rounded(float *p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void store_rounded(bf16_t *p, size_t i, float v) { p[i] = float_to_bf16_rne(v); }

// One 16-byte chunk of a weight row as floats.
template <typename WT> struct WChunk;
template <> struct WChunk<float> {
    static constexpr int N = 4;
    float v[4];
    __device__ __forceinline__ void load(const float *p) {
        float4 t = *reinterpret_cast<const float4 *>(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
};
template <> struct WChunk<bf16_t> {
    static constexpr int N = 8;
    float v[8];
    __device__ __forceinline__ void load(const bf16_t *p) {
        uint4 t = *reinterpret_cast<const uint4 *>(p);
        v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
        v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
        v[4] = __uint_as_float(t.z << 16); v[5] = __uint_as_float(t.z & 0xffff0000u);
        v[6] = __uint_as_float(t.w << 16); v[7] = __uint_as_float(t.w & 0xffff0000u);
    }
};

// The value of lane ^ off (off: 1, 2, 4, .. 32, a constant once the loop around it is unrolled) by the cross-lane moves of the
// vector ALU. __shfl_xor goes through the LDS unit instead: 64 and more cycles for each of the dependent exchanges of a
// reduction, where these take 4 to 8. The reductions add the same pairs in the same order either way. K-best search (200 000 x 5120,
// three queries): 466 -> 455 us, the two selection stages 25.5 + 21.0 -> 23.5 + 19.8 us; routing over a small table 22.8 -> 21.7 us.
template <int CTRL, int BANKS = 0xf>
__device__ __forceinline__ int lane_dpp(int old, int v) { return __builtin_amdgcn_update_dpp(old, v, CTRL, 0xf, BANKS, false); }
__device__ __forceinline__ int lane_xor(int v, int off) {
    switch (off) {
        case 1: return lane_dpp<0xb1>(v, v);                                // quad_perm 1 0 3 2
        case 2: return lane_dpp<0x4e>(v, v);                                // quad_perm 2 3 0 1
        case 4: return lane_dpp<0x114, 0xa>(lane_dpp<0x104, 0x5>(v, v), v); // even quads from the quad above, odd ones from the one below
        case 8: return lane_dpp<0x128>(v, v);                               // the row of 16 rotated by half
        case 16: {
            const auto r = __builtin_amdgcn_permlane16_swap((unsigned int)v, (unsigned int)v, false, false);
            return (int)((threadIdx.x & 16) ? r[0] : r[1]);
        }
        default: {
            const auto r = __builtin_amdgcn_permlane32_swap((unsigned int)v, (unsigned int)v, false, false);
            return (int)((threadIdx.x & 32) ? r[0] : r[1]);
        }
    }
}
__device__ __forceinline__ float lane_xor(float v, int off) { return __int_as_float(lane_xor(__float_as_int(v), off)); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += lane_xor(v, off);
    return v;
}
// the same sum with __shfl_xor, for the kernels whose loads are placed by hand: the lane exchanges above take register copies, which
// the build's check of those kernels does not tell from copies of a load in flight
__device__ __forceinline__ float wave_sum_shfl(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, lane_xor(v, off));
    return v;
}

// ------------------------------------------------------------------------------------------
// pass control
// ------------------------------------------------------------------------------------------
__global__ void set_pass_kernel(PassCtl *ctl, PassCtl value) {
    static_assert(sizeof(PassCtl) % 4 == 0 && sizeof(PassCtl) <= 256, "a word per thread");
    if (threadIdx.x < sizeof(PassCtl) / 4) reinterpret_cast<int *>(ctl)[threadIdx.x] = reinterpret_cast<const int *>(&value)[threadIdx.x];
}

// ------------------------------------------------------------------------------------------
// RoPE table: cos/sin of pos * base^(-2i/head_dim), evaluated in double, stored fp32
// ------------------------------------------------------------------------------------------
__global__ void rope_table_kernel(float *cos_t, float *sin_t, int max_seq, int half, int head_dim, double base) {
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= max_seq * half) return;
    int pos = idx / half, i = idx % half;
    double ang = (double)pos * pow(base, -2.0 * (double)i / (double)head_dim);
    cos_t[idx] = (float)cos(ang);
    sin_t[idx] = (float)sin(ang);
}

// ------------------------------------------------------------------------------------------
// embedding gather: x[r][:] = E[tok[r]][:]
// ------------------------------------------------------------------------------------------
// A prompt's rows as chunks of PR_CHUNK side by side (PromptRows): chunk c's control block is ctl[c], its rows lie behind those of the chunks
// before it. The row kernels take a chunk where a pass takes its rows, with the same device code, so a row has the bits that
// it has in a pass. A pass of 16 rows leaves most of the chip idle and pays five launches a block (or a one-launch pass's chain of
// hand-overs) for them: 250 rows, two blocks, fp32 / bf16: 200 columns 1049 / 1014 us in passes, 151 / 161 here, 520 columns 2362 / 1939 and 348 / 366, 1000
// columns 3604 / 2734 and 732 / 743, 1912 columns 6610 / 4489 and 2418 / 2393 (bound by the rows' way through the L1); where passes are the
// better way: prompt_rows. Chunks of eight rows: the products' builds of up to nine rows are the ones whose loads the compiler places well.
struct PromptRows {
    int32_t start, n;           // position of the first row, rows
    int32_t tok[PR_ROWS];
};
__global__ void set_prompt_kernel(PassCtl *ctl, PromptRows p) {
    const int c = blockIdx.x, first = c * PR_CHUNK, n = min(PR_CHUNK, p.n - first);
    if (threadIdx.x < KS_MAX_ROWS) ctl[c].tok[threadIdx.x] = (int)threadIdx.x < n ? p.tok[first + threadIdx.x] : 0;
    if (threadIdx.x == 0) { ctl[c].active = 1; ctl[c].n_rows = n; ctl[c].start = p.start + first; ctl[c].head_from = n; }
}

// (gridDim.y chunks)
template <typename WT>
__global__ void embed_kernel(const PassCtl *ctl, const WT *E, float *x, int d) {
    ctl += blockIdx.y;
    x += (size_t)blockIdx.y * PR_CHUNK * d;
    if (!ctl->active) return;
    int r = blockIdx.x;
    if (r >= ctl->n_rows) return;
    const WT *row = E + (size_t)ctl->tok[r] * d;
    for (int i = threadIdx.x; i < d; i += blockDim.x) x[(size_t)r * d + i] = load_as_float(row, i);
}

// ------------------------------------------------------------------------------------------
// RMSNorm: out[r][:] = x[r][:] * rsqrt(mean(x^2) + eps) * gain       (one workgroup per row)
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rmsnorm_kernel(const PassCtl *ctl, const float *x, const float *gain,
                                                      float *out, int d, float eps) {
    if (!ctl->active) return;
    int r = blockIdx.x;
    if (r >= ctl->n_rows) return;
    __shared__ float part[4];
    const float *xr = x + (size_t)r * d;
    float ss = 0.f;
    for (int i = threadIdx.x; i < d; i += 256) { float v = xr[i]; ss = fmaf(v, v, ss); }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = (part[0] + part[1]) + (part[2] + part[3]);
    float rs = 1.0f / sqrtf(tot / (float)d + eps);
    for (int i = threadIdx.x; i < d; i += 256) out[(size_t)r * d + i] = xr[i] * rs * gain[i];
}

// ------------------------------------------------------------------------------------------
// Y = X W^T for up to MR rows of X, one output feature (or pair of them) per wavefront (lanes stride over K in
// 16-byte chunks of the weight row), with what surrounds a product in the decoder folded in: the RMSNorm in front of it
// (gain into the weights, every wavefront sums x^2 beside its dot products) and the epilogues.
// Small models are bound by the length of this chain of dependent launches (a launch is at least 1.5-2 us, most of them a
// few round trips to the L2), so there are five per block, not eight, every operand load of a step goes out before the
// first is used (rows past the last live one repeat it: no load sits under a condition), and the MR sums are reduced over
// the wavefront together: with every exchange a lane hands over half of its rows, 17 exchanges for 16 rows instead of 96,
// the same tree for every row whatever MR is. fp32 configuration (4 blocks of d = 256), prompt 32 + 32 tokens in rounds of
// four drafts, before (norms and RoPE in launches of their own, 16-row builds for every verification, one position at a time
// per wavefront in the attention) and after: 15.3-16.1 -> 8.9-10.2 ms; attention 9.7 -> 4.2 us, 5-row products 8.9 -> 3.9 us.
// MR is the pass's row count (launch_rows), so no pass carries dead rows.
// ------------------------------------------------------------------------------------------
enum { EPI_STORE = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_QKV = 3 };

// sums of v[0..MR-1] over the wavefront: lane l returns that of row l & (MR' - 1), MR' = MR rounded up to a power of two. SHFL: the
// exchanges through the LDS unit (the same sums).
template <int MR, bool SHFL = false>
__device__ __forceinline__ float wave_sum_rows(float *v) {
    auto other = [](float x, int off) { return SHFL ? __shfl_xor(x, off, 64) : lane_xor(x, off); };
    constexpr int P = MR > 8 ? 16 : (MR > 4 ? 8 : (MR > 2 ? 4 : MR));
    float t[P];
#pragma unroll
    for (int i = 0; i < P; ++i) t[i] = i < MR ? v[i] : 0.f;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < P; off <<= 1) {
        // lanes that differ in this bit swap: the one without it keeps the even rows, the other the odd ones
        const bool hi = (lane & off) != 0;
#pragma unroll
        for (int i = 0; i < P / (2 * off); ++i) {
            const float keep = hi ? t[2 * i + 1] : t[2 * i], give = hi ? t[2 * i] : t[2 * i + 1];
            t[i] = keep + other(give, off);
        }
    }
#pragma unroll
    for (int off = P; off < 64; off <<= 1) t[0] += other(t[0], off);
    return t[0];
}

// The lane's operands of an item's products: N 16-byte pieces of weight row w0 (and w1 for a pair), 64 pieces apart, and the
// gain of the RMSNorm in front (nullptr: none). Past the row's end the last piece again.
template <typename WT, bool DUAL, int N>
struct RowsPieces {
    WChunk<WT> w[N > 0 ? N : 1], w2[N > 0 ? N : 1];
    float g[N > 0 ? N : 1][WChunk<WT>::N];
    __device__ __forceinline__ void load(const WT *w0, const WT *w1, const float *gain, int K) {
        constexpr int VEC = WChunk<WT>::N;
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int k = min((i * 64 + lane) * VEC, K - VEC);
            w[i].load(w0 + k);
            if (DUAL) w2[i].load(w1 + k);
#pragma unroll
            for (int j = 0; j < VEC; ++j) g[i][j] = gain ? gain[k + j] : 1.0f;
        }
    }
};

// Dot products of one item with MR rows of X (n_rows live ones, past them the last again): lane r returns row r's in a (and
// b). p: the lane's first N pieces, fetched by the caller (N = 0: none).
template <typename WT, int MR, bool DUAL, bool NORM, int N, bool SHFL = false>
__device__ __forceinline__ void rows_product(const RowsPieces<WT, DUAL, N> &p, const WT *w0, const WT *w1, const float *X, int ldx, int n_rows, int K,
                                             const float *gain, float eps, float &a, float &b) {
    constexpr int VEC = WChunk<WT>::N;
    const int lane = threadIdx.x & 63;
    float acc[MR], acc2[MR], ss[MR];
#pragma unroll
    for (int r = 0; r < MR; ++r) { acc[r] = 0.f; acc2[r] = 0.f; ss[r] = 0.f; }
    auto add = [&](WChunk<WT> w, WChunk<WT> w2, const float *g, int k) {
        if (gain) {
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                w.v[j] *= g[j];
                if (DUAL) w2.v[j] *= g[j];
            }
        }
#pragma unroll
        for (int r = 0; r < MR; ++r) {
            const float *xp = X + (size_t)min(r, n_rows - 1) * ldx + k;
#pragma unroll
            for (int j = 0; j < VEC; j += 4) {
                const float4 xv = *reinterpret_cast<const float4 *>(xp + j);
                const float x[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[r] = fmaf(w.v[j + e], x[e], acc[r]);
                    if (DUAL) acc2[r] = fmaf(w2.v[j + e], x[e], acc2[r]);
                    if (NORM) ss[r] = fmaf(x[e], x[e], ss[r]);
                }
            }
        }
    };
#pragma unroll
    for (int i = 0; i < N; ++i)
        if ((i * 64 + lane) * VEC < K) add(p.w[i], p.w2[i], p.g[i], (i * 64 + lane) * VEC);
    for (int k = (N * 64 + lane) * VEC; k < K; k += 64 * VEC) {
        WChunk<WT> w, w2;
        w.load(w0 + k);
        if (DUAL) w2.load(w1 + k);
        add(w, w2, gain + k, k);
    }
    a = wave_sum_rows<MR, SHFL>(acc);
    b = DUAL ? wave_sum_rows<MR, SHFL>(acc2) : 0.f;
    if (NORM) {
        const float sum = wave_sum_rows<MR, SHFL>(ss);
        if (gain) {
            const float rs = 1.0f / sqrtf(sum / (float)K + eps);
            a *= rs;
            b *= rs;
        }
    }
}

// a rotary pair, with the one rounding order that every kernel of these shapes has
__device__ __forceinline__ void rotate_pair(float a, float b, float c, float s, float &ra, float &rb) {
    ra = fmaf(a, c, -(b * s));
    rb = fmaf(b, c, a * s);
}

struct RowsOp {
    const float *X;             // [rows][ldx]
    int ldx;
    float *Y;                   // [rows][ldy]
    int ldy, N, K;              // N: output features (EPI_SWIGLU: per half; EPI_QKV: (H + 2 Hkv) * hd)
    const float *gain;          // RMSNorm in front of the product; nullptr: none
    float eps;
    int from_head;              // only rows from ctl->head_from on (LM head)
    // EPI_QKV: rotated queries to Y, keys and values (rounded to the cache type) to the cache [2][Hkv][max_seq][hd]
    void *kv_block;
    const float *cos_t, *sin_t;
    int H, Hkv, hd, max_seq;
    int chunks;                 // of a prompt's rows
};

// CHUNKS: a prompt's rows, op.chunks chunks of MR; the workgroups that share weights (one group of items, all chunks) are consecutive ones
// of a die, so that its L2 fetches a weight once.
template <typename WT, typename KT, int MR, int EPI, bool CHUNKS = false>
__global__ __launch_bounds__(256) void gemm_rows_kernel(const PassCtl *ctl, const WT *__restrict__ W, RowsOp op) {
    int group = blockIdx.x, n_groups = gridDim.x;
    if constexpr (CHUNKS) {
        const int i = blockIdx.x >> 3, g = i / op.chunks, c = i - g * op.chunks;
        group = g * 8 + (blockIdx.x & 7);
        n_groups = gridDim.x / op.chunks;
        ctl += c;
        op.X += (size_t)c * MR * op.ldx;
        op.Y += (size_t)c * MR * op.ldy;
    }
    if (!ctl->active) return;
    const int row_lo = op.from_head ? ctl->head_from : 0;
    const int n_rows = min(ctl->n_rows - row_lo, MR);
    if (n_rows <= 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = (group * blockDim.x + threadIdx.x) >> 6;
    const int n_waves = (n_groups * blockDim.x) >> 6;
    constexpr bool DUAL = EPI == EPI_SWIGLU || EPI == EPI_QKV;      // two weight rows per item
    const int K = op.K, half = op.hd >> 1;
    const int P = EPI == EPI_QKV ? (op.H + op.Hkv) * half : 0;      // rotary pairs; behind them pairs of value rows
    const int items = EPI == EPI_QKV ? P + op.Hkv * half : op.N;
    const float *X = op.X + (size_t)row_lo * op.ldx;

    for (int o = wave; o < items; o += n_waves) {
        int r0 = o, r1 = o + op.N;
        if (EPI == EPI_QKV) {
            if (o < P) { const int head = o / half; r0 = head * op.hd + (o - head * half); r1 = r0 + half; }
            else { r0 = (op.H + op.Hkv) * op.hd + (o - P) * 2; r1 = r0 + 1; }
        }
        float a, b;
        const WT *w0 = W + (size_t)r0 * K, *w1 = W + (size_t)r1 * K;
        // No piece is requested ahead here, as the one-launch pass does: that takes more registers and other waits (1000 to 1500 columns, fp32: O and
        // down with six and seven rows 8-9 us -> 20-30, QKV with eleven to sixteen 9-12 -> 15-29; bf16: SwiGLU 17.3 -> 22.2 with sixteen).
        // Exchanges: the compiler places the loads better around those without the LDS unit in most builds (fp32, O and down with eight
        // and nine rows 27-39 -> 9 us; bf16, QKV with fourteen and fifteen 14-19 -> 8-11) and worse in these (fp32 QKV 12.0 -> 14.6, a head
        // of 20 000 rows 54 -> 62).
        constexpr bool SHFL = EPI == EPI_STORE ? MR == 10 || MR == 14 : EPI == EPI_QKV && sizeof(WT) == 4 && (MR == 12 || MR == 14 || MR == 15);
        rows_product<WT, MR, DUAL, EPI == EPI_QKV || EPI == EPI_SWIGLU, 0, SHFL>(RowsPieces<WT, DUAL, 0>(), w0, w1, X, op.ldx, n_rows, K, op.gain, op.eps, a, b);
        if (lane < n_rows) {           // lane r holds row r
            const int row = row_lo + lane;
            float *yp = op.Y + (size_t)row * op.ldy;
            if (EPI == EPI_STORE) yp[o] = a;
            if (EPI == EPI_RESID) yp[o] += a;
            if (EPI == EPI_SWIGLU) yp[o] = (a / (1.0f + expf(-a))) * b;
            if constexpr (EPI == EPI_QKV) {
                const int pos = ctl->start + row;
                KT *kc = reinterpret_cast<KT *>(op.kv_block), *vc = kc + (size_t)op.Hkv * op.max_seq * op.hd;
                if (o < P) {
                    const int head = o / half, i = o - head * half;
                    const float c = op.cos_t[(size_t)pos * half + i], s = op.sin_t[(size_t)pos * half + i];
                    float ra, rb;
                    rotate_pair(a, b, c, s, ra, rb);
                    if (head < op.H) {
                        yp[r0] = ra; yp[r1] = rb;
                    } else {
                        const size_t base = ((size_t)(head - op.H) * op.max_seq + pos) * op.hd;
                        store_rounded(kc, base + i, ra);
                        store_rounded(kc, base + i + half, rb);
                    }
                } else {
                    const int v = (o - P) * 2, head = v / op.hd, i = v - head * op.hd;
                    const size_t base = ((size_t)head * op.max_seq + pos) * op.hd + i;
                    store_rounded(vc, base, a);
                    store_rounded(vc, base + 1, b);
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// Attention of one (row, head): softmax(q K^T / sqrt(hd)) V over positions 0..start+r.
// 256 threads per (head, row); scores are kept in LDS (max_seq floats). A group of HD/4 lanes takes a
// position (four dimensions per lane), 16 or 8 positions side by side, four rounds of them in flight.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float4 load4_as_float(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ float4 load4_as_float(const bf16_t *p) {
    const uint2 t = *reinterpret_cast<const uint2 *>(p);
    return float4{__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xffff0000u), __uint_as_float(t.y << 16), __uint_as_float(t.y & 0xffff0000u)};
}

struct AttnItemLds {
    float red[8];
    __align__(16) float outp[4][128];
};

constexpr int ATI_U = 4;                                     // rounds of positions in flight
// the position of thread tid in round u (clamped)
template <int HD> __device__ __forceinline__ int attention_position(int tid, int u, int len) { return min(tid / (HD / 4) + u * (256 / (HD / 4)), len - 1); }

// One item by 256 threads (tid), q: the lane's four query dimensions; key(t), value(t): its four dimensions of position t;
// k0, v0: those of the first ATI_U rounds, fetched by the caller. Every thread of the workgroup gets here (three meetings).
// out(dim, value) is called by HD of the threads.
template <int HD, typename FK, typename FV, typename FO>
__device__ __forceinline__ void attention_item(float4 q, int len, int tid, float *scores, AttnItemLds &l, const float4 (&k0)[ATI_U], const float4 (&v0)[ATI_U], FK key, FV value, FO out) {
    constexpr int LPP = HD / 4, NP = 256 / LPP, U = ATI_U;   // lanes per position, positions side by side
    const int lane = tid & 63, wave = tid >> 6, grp = tid / LPP, d0 = (tid % LPP) * 4;
    const float scale = 1.0f / sqrtf((float)HD);

    float lmax = -INFINITY;
    auto score = [&](int t0, const float4 (&k)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float p = q.x * k[u].x;
            p = fmaf(q.y, k[u].y, p); p = fmaf(q.z, k[u].z, p); p = fmaf(q.w, k[u].w, p);
#pragma unroll
            for (int off = 1; off < LPP; off <<= 1) p += lane_xor(p, off);
            p *= scale;
            if (t0 + u * NP < len) {
                if (d0 == 0) scores[t0 + u * NP] = p;
                lmax = fmaxf(lmax, p);
            }
        }
    };
    score(grp, k0);
    for (int t0 = grp + NP * U; t0 < len; t0 += NP * U) {
        float4 k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = key(min(t0 + u * NP, len - 1));
        score(t0, k);
    }
    lmax = wave_max(lmax);
    if (lane == 0) l.red[wave] = lmax;
    __syncthreads();
    const float mx = fmaxf(fmaxf(l.red[0], l.red[1]), fmaxf(l.red[2], l.red[3]));
    float lsum = 0.f;
    for (int t = tid; t < len; t += 256) {
        const float e = expf(scores[t] - mx);
        scores[t] = e;
        lsum += e;
    }
    lsum = wave_sum(lsum);
    if (lane == 0) l.red[4 + wave] = lsum;
    __syncthreads();
    const float den = (l.red[4] + l.red[5]) + (l.red[6] + l.red[7]);
    float4 o = float4{0.f, 0.f, 0.f, 0.f};
    auto weigh = [&](int t0, const float4 (&v)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float e = t0 + u * NP < len ? scores[t0 + u * NP] : 0.f;
            if (t0 + u * NP < len) { o.x = fmaf(e, v[u].x, o.x); o.y = fmaf(e, v[u].y, o.y); o.z = fmaf(e, v[u].z, o.z); o.w = fmaf(e, v[u].w, o.w); }
        }
    };
    weigh(grp, v0);
    for (int t0 = grp + NP * U; t0 < len; t0 += NP * U) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = value(min(t0 + u * NP, len - 1));
        weigh(t0, v);
    }
#pragma unroll
    for (int off = LPP; off < 64; off <<= 1) {               // the wavefront's positions side by side
        o.x += lane_xor(o.x, off); o.y += lane_xor(o.y, off);
        o.z += lane_xor(o.z, off); o.w += lane_xor(o.w, off);
    }
    if (lane < LPP) *reinterpret_cast<float4 *>(&l.outp[wave][d0]) = o;
    __syncthreads();
    if (tid < HD) {
        const float s = (l.outp[0][tid] + l.outp[1][tid]) + (l.outp[2][tid] + l.outp[3][tid]);
        out(tid, s / den);
    }
}

template <typename KT, int HD>
__global__ __launch_bounds__(256) void attention_kernel(const PassCtl *ctl, const float *qkv, const KT *kv_block,
                                                        float *att, int H, int Hkv, int max_seq) {
    const int h = blockIdx.x, r = blockIdx.y, c = blockIdx.z;      // (gridDim.z chunks of a prompt's rows)
    ctl += c;
    qkv += (size_t)c * PR_CHUNK * (H + 2 * Hkv) * HD;
    att += (size_t)c * PR_CHUNK * H * HD;
    if (!ctl->active) return;
    if (r >= ctl->n_rows) return;
    extern __shared__ float scores[];                        // [len]
    __shared__ AttnItemLds lds;
    const int kvh = h / (H / Hkv);
    const int ld = (H + 2 * Hkv) * HD;
    const int d0 = (threadIdx.x % (HD / 4)) * 4;
    const float4 q = *reinterpret_cast<const float4 *>(qkv + (size_t)r * ld + h * HD + d0);
    const KT *kc = kv_block + (size_t)kvh * max_seq * HD + d0;
    const KT *vc = kv_block + ((size_t)Hkv + kvh) * max_seq * HD + d0;
    const int len = ctl->start + r + 1;
    auto key = [&](int t) { return load4_as_float(kc + (size_t)t * HD); };
    auto value = [&](int t) { return load4_as_float(vc + (size_t)t * HD); };
    float4 k0[ATI_U], v0[ATI_U];
#pragma unroll
    for (int u = 0; u < ATI_U; ++u) k0[u] = key(attention_position<HD>(threadIdx.x, u, len));
#pragma unroll
    for (int u = 0; u < ATI_U; ++u) v0[u] = value(attention_position<HD>(threadIdx.x, u, len));
    attention_item<HD>(q, len, threadIdx.x, scores, lds, k0, v0, key, value,
                       [&](int dim, float v) { att[(size_t)r * (H * HD) + h * HD + dim] = v; });
}

// ------------------------------------------------------------------------------------------
// arg-max (lowest index on ties) and top-1 softmax probability of each logits row
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }

__global__ __launch_bounds__(1024) void argmax_kernel(const PassCtl *ctl, const float *logits, int V, HeadResult *res) {
    if (!ctl->active) return;
    const int r = blockIdx.x;
    if (r >= ctl->n_rows || r < ctl->head_from) return;
    __shared__ float sv[16];
    __shared__ int si[16];
    __shared__ float ssum[16];
    const float *row = logits + (size_t)r * V;
    float bv = -INFINITY; int bi = 0x7fffffff;
    for (int i = threadIdx.x; i < V; i += 1024) { float v = row[i]; if (better(v, i, bv, bi)) { bv = v; bi = i; } }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        float ov = lane_xor(bv, off); int oi = lane_xor(bi, off);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { sv[wave] = bv; si[wave] = bi; }
    __syncthreads();
    bv = sv[0]; bi = si[0];
    for (int w = 1; w < 16; ++w) if (better(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; }
    float s = 0.f;
    for (int i = threadIdx.x; i < V; i += 1024) s += expf(row[i] - bv);
    s = wave_sum(s);
    if (lane == 0) ssum[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float tot = 0.f;
        for (int w = 0; w < 16; ++w) tot += ssum[w];
        res->tok[r] = bi;
        res->prob[r] = 1.0f / tot;
    }
}

// The same for models whose passes may run in one launch (kernels_small.h): there HEAD_CLASSES wavefronts work out the logits, each
// those of its own class (token modulo HEAD_CLASSES), and a row's sum of exponentials is formed class by class. Here a thread takes a
// class, so that the probability has the same bits whichever way the pass ran, and a confidence rule never decides by it.
constexpr int HEAD_GROUPS = 64, HEAD_WAVES = 8, HEAD_CLASSES = HEAD_GROUPS * HEAD_WAVES;     // class: wavefront * HEAD_GROUPS + workgroup
// a class's largest logit so far (the lowest token on ties) and sum of exponentials: one more logit
__device__ __forceinline__ void head_fold(float v, int o, float &m, float &s, int &mi) {
    if (v > m) { s = fmaf(s, expf(m - v), 1.0f); m = v; mi = o; }
    else {
        if (better(v, o, m, mi)) mi = o;
        s += v == -INFINITY ? 0.f : expf(v - m);
    }
}
// a workgroup's classes, `stride` apart in hm, hs, hi
__device__ __forceinline__ void head_join(const float *hm, const float *hs, const int *hi, int stride, float &bm, int &bi, float &sum) {
    bm = hm[0]; bi = hi[0]; sum = 0.f;
    for (int w = 1; w < HEAD_WAVES; ++w) if (better(hm[w * stride], hi[w * stride], bm, bi)) { bm = hm[w * stride]; bi = hi[w * stride]; }
    for (int w = 0; w < HEAD_WAVES; ++w) if (hi[w * stride] != 0x7fffffff) sum = fmaf(hs[w * stride], expf(hm[w * stride] - bm), sum);
}
// all workgroups' shares, a lane each
__device__ __forceinline__ void head_merge(float m, int mi, float s, int &token, float &prob) {
    float bm = m;
    token = mi;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float ov = lane_xor(bm, off);
        const int oi = lane_xor(token, off);
        if (better(ov, oi, bm, token)) { bm = ov; token = oi; }
    }
    prob = 1.0f / wave_sum(mi != 0x7fffffff ? s * expf(m - bm) : 0.f);
}

__global__ __launch_bounds__(HEAD_CLASSES) void argmax_classes_kernel(const PassCtl *ctl, const float *logits, int V, HeadResult *res) {
    if (!ctl->active) return;
    const int r = blockIdx.x;
    if (r >= ctl->n_rows || r < ctl->head_from) return;
    __shared__ float hm[HEAD_CLASSES], hs[HEAD_CLASSES];
    __shared__ int hi[HEAD_CLASSES];
    const float *row = logits + (size_t)r * V;
    float m = -INFINITY, s = 0.f;
    int mi = 0x7fffffff;
    for (int o = threadIdx.x; o < V; o += HEAD_CLASSES) head_fold(row[o], o, m, s, mi);
    hm[threadIdx.x] = m; hs[threadIdx.x] = s; hi[threadIdx.x] = mi;
    __syncthreads();
    if (threadIdx.x >= HEAD_GROUPS) return;
    float prob;
    int token;
    head_join(hm + threadIdx.x, hs + threadIdx.x, hi + threadIdx.x, HEAD_GROUPS, m, mi, s);
    head_merge(m, mi, s, token, prob);
    if (threadIdx.x == 0) { res->tok[r] = token; res->prob[r] = prob; }
}

// ------------------------------------------------------------------------------------------
// KNN routing, Eq. 4: score_n = (v . a_n) / |a_n|  (|v| is a common positive factor), then arg-max
// ------------------------------------------------------------------------------------------
template <int Q, typename AT>
__global__ __launch_bounds__(256) void knn_scores_multi_kernel(const float *__restrict__ queries, const AT *__restrict__ anchors,
                                                               int N, int D, float *scores);

__global__ __launch_bounds__(1024) void knn_argmax_kernel(const float *scores, const float *query, const int32_t *labels,
                                                          int N, int D, KnnResult *res) {
    __shared__ float sv[16];
    __shared__ int si[16];
    __shared__ int bad;
    __shared__ float qn[16];
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    float bv = -INFINITY; int bi = 0x7fffffff; int mybad = 0;
    for (int i = threadIdx.x; i < N; i += 1024) {
        float v = scores[i];
        if (!isfinite(v)) mybad = 1;
        else if (better(v, i, bv, bi)) { bv = v; bi = i; }
    }
    float q2 = 0.f;
    for (int i = threadIdx.x; i < D; i += 1024) { float v = query[i]; q2 = fmaf(v, v, q2); }
    q2 = wave_sum(q2);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        float ov = lane_xor(bv, off); int oi = lane_xor(bi, off);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (mybad) atomicOr(&bad, 1);
    if (lane == 0) { sv[wave] = bv; si[wave] = bi; qn[wave] = q2; }
    __syncthreads();
    if (threadIdx.x == 0) {
        bv = sv[0]; bi = si[0];
        float qtot = qn[0];
        for (int w = 1; w < 16; ++w) { if (better(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; } qtot += qn[w]; }
        int degenerate = bad || !(qtot > 0.f) || !isfinite(qtot) || bi == 0x7fffffff;
        res->degenerate = degenerate;
        res->idx = degenerate ? -1 : bi;
        res->label = degenerate ? -1 : labels[bi];
        res->score = bv;
    }
}

// ------------------------------------------------------------------------------------------
// K nearest anchors for a few queries at once (Eq. 4 generalised from the arg-max to the K best), then the
// majority domain among them. One pass over the anchor table serves up to KNN_QMAX queries: a wavefront
// streams one anchor (16-byte nontemporal loads, all of a block in flight before the first is used) and
// forms its dot product with every query (the queries are small and stay in cache) and its own norm.
// ------------------------------------------------------------------------------------------
#define KNN_QMAX 4
#define KNN_KMAX 16

__global__ void fill_zero_kernel(int *p, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

struct KnnTopk {
    int32_t idx[KNN_KMAX];
    float cosine[KNN_KMAX];
    int32_t domain;       // majority label among the K; ties go to the tied label whose best anchor ranks first
    int32_t degenerate;   // 1: zero-norm / non-finite query or anchor met
};

// AT = float or bf16_t: the type the anchor table is stored in (queries, products and sums are fp32 either way). A lane's
// 16-byte load covers EPL = 4 or 8 consecutive elements of an anchor. A wavefront takes A consecutive anchors at a
// time and L loads per lane of each, so 8 loads per lane are in flight whatever the storage type and query count, a
// query value fetched from the cache serves A anchors (with four queries the query reads would otherwise be four
// times the table's bytes), and 5120 elements are whole blocks in every variant. An anchor's sums are formed in the
// same order whatever A is: a lane adds its elements in column order, then the 64 lanes are summed.
template <int Q, typename AT>
struct KnnTile {
    static constexpr int EPL = 16 / (int)sizeof(AT);
    static constexpr int A = (Q >= 3 || EPL == 8) ? 4 : 2;
    static constexpr int L = 8 / A;
};

// The scores of A consecutive anchors from the lanes' sums (dot: [Q][A]): all of them are added up over the wavefront together
// (wave_sum_rows: 17 exchanges for up to 16 sums instead of 96), lane q * A + t ends up with query q's score of anchor n0 + t.
template <int Q, int A>
__device__ __forceinline__ void knn_store_scores(float *dot, float *nn, int n0, int N, float *scores) {
    const int lane = threadIdx.x & 63, t = lane & (A - 1), q = lane / A;
    const float d = wave_sum_rows<Q * A>(dot), n2 = wave_sum_rows<A>(nn);
    const bool ok = n2 > 0.f && isfinite(n2);
    if (q < Q && n0 + t < N) scores[(size_t)q * N + n0 + t] = ok ? d * (1.0f / sqrtf(n2)) : NAN;
}

template <int Q, typename AT>
__global__ __launch_bounds__(256) void knn_scores_multi_kernel(const float *__restrict__ queries, const AT *__restrict__ anchors,
                                                               int N, int D, float *scores /*[Q][N]*/) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    constexpr int EPL = KnnTile<Q, AT>::EPL;          // elements per lane and load
    constexpr int A = KnnTile<Q, AT>::A, L = KnnTile<Q, AT>::L;
    constexpr int BLK = L * 64 * EPL;                 // elements of an anchor per block of L loads per lane
    const int lane = threadIdx.x & 63;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int n_waves = (gridDim.x * blockDim.x) >> 6;
    for (int n0 = wave * A; n0 < N; n0 += n_waves * A) {
        const AT *a[A];
#pragma unroll
        for (int t = 0; t < A; ++t) a[t] = anchors + (size_t)min(n0 + t, N - 1) * D;      // past the table: the last anchor again, not stored
        float dot[Q][A], nn[A];
#pragma unroll
        for (int t = 0; t < A; ++t) {
            nn[t] = 0.f;
#pragma unroll
            for (int q = 0; q < Q; ++q) dot[q][t] = 0.f;
        }
        for (int k0 = 0; k0 < D; k0 += BLK) {            // blocks of A x L 16-byte loads per lane, issued together
            f4 av[A][L];
#pragma unroll
            for (int j = 0; j < L; ++j) {
                const int k = min(k0 + (j * 64 + lane) * EPL, D - EPL);           // clamped, masked below
#pragma unroll
                for (int t = 0; t < A; ++t) av[t][j] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(a[t] + k));
            }
#pragma unroll
            for (int j = 0; j < L; ++j) {
                const int k = k0 + (j * 64 + lane) * EPL;
                if (k < D) {
                    float4 qv[Q][EPL / 4];
#pragma unroll
                    for (int q = 0; q < Q; ++q)
#pragma unroll
                        for (int i4 = 0; i4 < EPL / 4; ++i4)
                            qv[q][i4] = *reinterpret_cast<const float4 *>(queries + (size_t)q * D + k + 4 * i4);
#pragma unroll
                    for (int t = 0; t < A; ++t) {
                        float e[EPL];
                        if constexpr (EPL == 4) {
                            e[0] = av[t][j].x; e[1] = av[t][j].y; e[2] = av[t][j].z; e[3] = av[t][j].w;
                        } else {
#pragma unroll
                            for (int w = 0; w < 4; ++w) {
                                const unsigned int u = __float_as_uint(av[t][j][w]);
                                e[2 * w] = __uint_as_float(u << 16); e[2 * w + 1] = __uint_as_float(u & 0xffff0000u);
                            }
                        }
#pragma unroll
                        for (int i = 0; i < EPL; ++i) nn[t] = fmaf(e[i], e[i], nn[t]);
#pragma unroll
                        for (int q = 0; q < Q; ++q) {
#pragma unroll
                            for (int i4 = 0; i4 < EPL / 4; ++i4) {
                                dot[q][t] = fmaf(e[4 * i4], qv[q][i4].x, dot[q][t]); dot[q][t] = fmaf(e[4 * i4 + 1], qv[q][i4].y, dot[q][t]);
                                dot[q][t] = fmaf(e[4 * i4 + 2], qv[q][i4].z, dot[q][t]); dot[q][t] = fmaf(e[4 * i4 + 3], qv[q][i4].w, dot[q][t]);
                            }
                        }
                    }
                }
            }
        }
        knn_store_scores<Q, A>(&dot[0][0], nn, n0, N, scores);
    }
}

// The same scan for several queries and large tables (knn_streams). The one above takes its queries from the L1, behind the
// anchors in the queue of loads, so a wavefront drains its loads in every block: 5.0 TB/s with three queries where one query
// reaches 6.7. Here the queries lie in LDS (zeros behind D; the two halves of eight elements apart, so that neighbouring
// lanes read neighbouring 16 bytes), the only loads in the queue are the table's, and a wavefront has KNN_STAGES blocks of A of
// them under way, each requested again for a later block as soon as it has been used, also across anchors.
// One workgroup per unit stays for all its anchors. Sums are formed in the same order as above.
constexpr int KNN_STAGES = 3, KNN_STREAM_NT = 1024;
template <typename AT> constexpr int knn_block() { return 64 * 16 / (int)sizeof(AT); }      // elements of an anchor a wavefront's load covers
template <typename AT> inline size_t knn_stream_lds(int Q, int D) { return (size_t)Q * ((D + knn_block<AT>() - 1) / knn_block<AT>() * knn_block<AT>()) * 4; }

template <int Q, typename AT>
__global__ __launch_bounds__(KNN_STREAM_NT) void knn_scores_stream_kernel(const float *__restrict__ queries, const AT *__restrict__ anchors,
                                                                          int N, int D, float *scores /*[Q][N]*/) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    constexpr int EPL = 16 / (int)sizeof(AT), A = 4, BLK = knn_block<AT>(), H = EPL / 4;
    extern __shared__ __align__(16) char lds_bytes[];
    float *qs = reinterpret_cast<float *>(lds_bytes);         // [Q][blocks][H][64 lanes][4]
    const int nb = (D + BLK - 1) / BLK, lane = threadIdx.x & 63, wave = (blockIdx.x * KNN_STREAM_NT + threadIdx.x) >> 6;
    const int n_waves = (gridDim.x * KNN_STREAM_NT) >> 6, n_groups = (N + A - 1) / A;

    int fg = min(wave, n_groups - 1), fb = 0;                 // group of A anchors and block that are requested next
    auto fetch = [&](f4 *to) {
        const int k = min(fb * BLK + lane * EPL, D - EPL);    // clamped, masked below
#pragma unroll
        for (int t = 0; t < A; ++t) to[t] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(anchors + (size_t)min(fg * A + t, N - 1) * D + k));
        if (++fb == nb) { fb = 0; fg = min(fg + n_waves, n_groups - 1); }      // (behind the last group it again; not used)
    };
    f4 av[KNN_STAGES][A];
#pragma unroll
    for (int s = 0; s < KNN_STAGES; ++s) fetch(av[s]);
    for (int i = threadIdx.x * 4; i < Q * nb * BLK; i += KNN_STREAM_NT * 4) {
        const int q = i / (nb * BLK), k = i - q * (nb * BLK), b = k / BLK, in = k - b * BLK, l = in / EPL, h = (in - l * EPL) / 4;
        const f4 v = k < D ? *reinterpret_cast<const f4 *>(queries + (size_t)q * D + k) : f4{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f4 *>(qs + (((size_t)(q * nb + b) * H + h) * 64 + l) * 4) = v;
    }
    __syncthreads();
    if (wave >= n_groups) return;
    float dot[Q * A], nn[A];
    int g = wave, b = 0;
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < Q * A; ++i) dot[i] = 0.f;
#pragma unroll
        for (int t = 0; t < A; ++t) nn[t] = 0.f;
    };
    clear();
    for (;;) {
#pragma unroll
        for (int s = 0; s < KNN_STAGES; ++s) {
            if (b * BLK + lane * EPL < D) {
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    float e[A][4];
#pragma unroll
                    for (int t = 0; t < A; ++t) {
                        if constexpr (EPL == 4) {
                            e[t][0] = av[s][t].x; e[t][1] = av[s][t].y; e[t][2] = av[s][t].z; e[t][3] = av[s][t].w;
                        } else {
#pragma unroll
                            for (int w = 0; w < 2; ++w) {
                                const unsigned int u = __float_as_uint(av[s][t][2 * h + w]);
                                e[t][2 * w] = __uint_as_float(u << 16); e[t][2 * w + 1] = __uint_as_float(u & 0xffff0000u);
                            }
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) nn[t] = fmaf(e[t][i], e[t][i], nn[t]);
                    }
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        const f4 qv = *reinterpret_cast<const f4 *>(qs + (((size_t)(q * nb + b) * H + h) * 64 + lane) * 4);
#pragma unroll
                        for (int t = 0; t < A; ++t)
#pragma unroll
                            for (int i = 0; i < 4; ++i) dot[q * A + t] = fmaf(e[t][i], qv[i], dot[q * A + t]);
                    }
                }
            }
            fetch(av[s]);
            if (++b == nb) {
                knn_store_scores<Q, A>(dot, nn, g * A, N, scores);
                clear();
                b = 0;
                g += n_waves;
                if (g >= n_groups) return;
            }
        }
    }
}

#define KNN_ROUNDS_MAX_N (16 * 64 * 64)      // scores a workgroup ranks at most: a lane keeps one mask bit per entry it looks at
#define KNN_SLICES_MAX 256       // slices per query: 256 x KNN_ROUNDS_MAX_N anchors at most

// An entry as one number: its value in an order-preserving form, above the complement of its index, so that the larger key is
// the better entry (finite values; 0: a dead entry).
typedef unsigned long long KnnKey;
__device__ __forceinline__ KnnKey knn_key(float v, int idx) {
    const unsigned int u = __float_as_uint(v + 0.0f);          // (-0 counts as 0)
    return ((KnnKey)(u ^ (u & 0x80000000u ? 0xffffffffu : 0x80000000u)) << 32) | (0xffffffffu - (unsigned int)idx);
}
__device__ __forceinline__ float knn_key_value(KnnKey k) {
    const unsigned int u = (unsigned int)(k >> 32);
    return __uint_as_float(u ^ (u & 0x80000000u ? 0x80000000u : 0xffffffffu));
}
__device__ __forceinline__ int knn_key_index(KnnKey k) { return (int)(0xffffffffu - (unsigned int)k); }
// the wavefront's largest number, in every lane: rotations within the rows of 16, then the rows
__device__ __forceinline__ unsigned int wave_max_u32(unsigned int x) {
    x = max(x, (unsigned int)lane_dpp<0x121>((int)x, (int)x));
    x = max(x, (unsigned int)lane_dpp<0x122>((int)x, (int)x));
    x = max(x, (unsigned int)lane_dpp<0x124>((int)x, (int)x));
    x = max(x, (unsigned int)lane_dpp<0x128>((int)x, (int)x));
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = max((unsigned int)r[0], (unsigned int)r[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return max((unsigned int)h[0], (unsigned int)h[1]);
}
// the wavefront's largest key, in every lane: its value first, then the index among those that have it
__device__ __forceinline__ KnnKey knn_wave_best(KnnKey k) {
    const unsigned int hi = wave_max_u32((unsigned int)(k >> 32));
    return ((KnnKey)hi << 32) | wave_max_u32((unsigned int)(k >> 32) == hi ? (unsigned int)k : 0u);
}
// four keys of a lane, the largest first
__device__ __forceinline__ void knn_sort4(KnnKey *k) {
    auto order = [&](int i, int j) {
        const KnnKey a = k[i], b = k[j];
        k[i] = a > b ? a : b;
        k[j] = a > b ? b : a;
    };
    order(0, 1); order(2, 3); order(0, 2); order(1, 3); order(1, 2);
}
// the largest of four is given away if `won`
__device__ __forceinline__ void knn_take(KnnKey *k, bool won) {
#pragma unroll
    for (int i = 0; i < 3; ++i) k[i] = won ? k[i + 1] : k[i];
    k[3] = won ? 0 : k[3];
}

struct KnnRankLds {
    KnnKey key[16][KNN_KMAX];
    KnnKey best[KNN_KMAX];       // the K best in rank order (0 once the entries run out)
    float qn[16];
    int last;
};

// The K best (largest value, lowest anchor index on ties) of n entries, in rank order, by one workgroup of 1024
// threads; entry(i) is an entry's key. Two levels of K rounds of arg-max, both inside single wavefronts (registers and cross-lane
// moves, no meeting per round): every wavefront ranks the K best of its sixteenth of the entries (a lane looks at entries 64
// apart and marks the ones it has given away in a 64-bit mask, hence n <= KNN_ROUNDS_MAX_N), the workgroup meets once,
// and the first wavefront ranks the K best of the 16 x K survivors into l.best, which it alone may read without a meeting.
template <typename F> __device__ __forceinline__ void knn_rounds(int n, int K, KnnRankLds &l, F entry) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    {
        const int w0 = (int)((long long)n * wave / 16), w1 = (int)((long long)n * (wave + 1) / 16);
        const int M = (w1 - w0 + 63) >> 6;                 // <= 64
        unsigned long long given = 0;                       // bit m: this lane's entry w0 + 64 m + lane is among the winners (m >= 4)
        // the lane's first four entries stay in registers over the rounds, in order (slices of a few thousand scores and the
        // candidate lists have no more); entries beyond are read again in every round
        KnnKey rk[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int i = w0 + (m << 6) + lane;
            rk[m] = i < w1 ? entry(i) : 0;
        }
        knn_sort4(rk);
        for (int r = 0; r < K; ++r) {
            KnnKey mine = rk[0];
            int far = -1;                                   // where mine comes from, past the registers
            for (int m = 4; m < M; ++m) {
                const int i = w0 + (m << 6) + lane;
                if (i >= w1 || ((given >> m) & 1ull)) continue;
                const KnnKey k = entry(i);
                if (k > mine) { mine = k; far = m; }
            }
            const KnnKey best = knn_wave_best(mine);
            const bool won = best == mine && best != 0;     // indices are all different: one lane
            if (won && far >= 0) given |= 1ull << far;
            knn_take(rk, won && far < 0);
            if (lane == 0) l.key[wave][r] = best;
        }
    }
    __syncthreads();
    if (wave == 0) {
        // 16 x KNN_KMAX slots, four per lane; slots of rounds that were not played are dead
        KnnKey ck[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int c = (m << 6) + lane;
            ck[m] = c % KNN_KMAX < K ? l.key[c / KNN_KMAX][c % KNN_KMAX] : 0;
        }
        knn_sort4(ck);
        for (int r = 0; r < K; ++r) {
            const KnnKey best = knn_wave_best(ck[0]);
            knn_take(ck, best == ck[0]);
            if (lane == 0) l.best[r] = best;
        }
    }
}

// The ranking behind a scan, in one launch: workgroup (query q, slice b) ranks the K best of its slice of the scores; with several
// slices it leaves them as candidates, and the one that arrives last ranks all slices' candidates and takes the vote. Nobody waits for anybody:
// candidates are written through (agent scope), acknowledged, and counted in; `arrivals` is zero between launches.
// Bound by dependent latencies: the rounds, and the hand-over between slices. As two launches (each with its own rounds of 64-bit
// exchanges, the second with one thread for the vote) 31-33 us behind the scan of three queries over 200 000 anchors, 22 over 3000;
// now 24 and 10. Whole calls with results in host memory: three queries over up to 3000 anchors 47-48 -> 32-34 us.
// `res` may lie in host memory: a thread writes an entry.
__global__ __launch_bounds__(1024) void knn_rank_kernel(const float *scores /*[Q][N]*/, int N, int K, int n_slices, KnnKey *cand /*[Q][n_slices][K]*/,
                                                        int *bad_flag /*[Q][n_slices]*/, int *arrivals /*[Q]*/, const float *queries,
                                                        const int32_t *labels, int D, KnnTopk *res) {
    __shared__ KnnRankLds l;
    const int q = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = (int)((long long)N * b / n_slices), n = (int)((long long)N * (b + 1) / n_slices) - i0;
    const float *val = scores + (size_t)q * N + i0;
    int bad = 0;
    knn_rounds(n, min(K, n), l, [&](int i) -> KnnKey {
        const float v = val[i];
        if (!isfinite(v)) { bad = 1; return 0; }
        return knn_key(v, i0 + i);
    });
    bad = __syncthreads_or(bad);
    if (n_slices > 1) {
        KnnKey *const mine = cand + ((size_t)q * n_slices + b) * K;
        if (tid < K) __hip_atomic_store(mine + tid, tid < n ? l.best[tid] : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (tid == 0) __hip_atomic_store(bad_flag + q * n_slices + b, bad ? 1 : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        static_assert(KNN_KMAX <= 64, "the first wavefront's stores");
        if (wave == 0) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // they are where everybody looks for them
            if (lane == 0) {
                l.last = __hip_atomic_fetch_add(arrivals + q, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_slices - 1;
                if (l.last) __hip_atomic_store(arrivals + q, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
        if (!l.last) return;
    }
    const float *qv = queries + (size_t)q * D;
    float q2 = 0.f;
    for (int i = tid; i < D; i += 1024) { const float v = qv[i]; q2 = fmaf(v, v, q2); }
    if (n_slices > 1) {
        for (int i = tid; i < n_slices; i += 1024) bad |= __hip_atomic_load(bad_flag + q * n_slices + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const KnnKey *const all = cand + (size_t)q * n_slices * K;
        knn_rounds(n_slices * K, K, l, [&](int i) -> KnnKey { return __hip_atomic_load(all + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); });
    }
    q2 = wave_sum(q2);
    if (lane == 0) l.qn[wave] = q2;
    bad = __syncthreads_or(bad);
    if (wave != 0) return;
    float qtot = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) qtot += l.qn[w];
    const KnnKey first = l.best[0];
    const bool degenerate = bad || !(qtot > 0.f) || !isfinite(qtot) || first == 0;
    const float invq = degenerate ? 0.f : 1.0f / sqrtf(qtot);
    // lane r: the anchor of rank r and its label
    const KnnKey key = lane < K && !degenerate ? l.best[lane] : 0;
    const int idx = key ? knn_key_index(key) : -1;
    const int lab = key ? labels[idx] : -1;
    // The vote: every label is counted, the best-ranked one among those with the highest count wins. A label below zero ends the list.
    const unsigned long long over = __ballot(lab < 0);
    const int live = min(__ffsll((long long)over) - 1, K);         // (lanes from K on have none)
    int count = 0;
    for (int r = 0; r < K; ++r) count += __shfl(lab, r) == lab;
    int best_rank = 0, best_count = 0;
    for (int r = 0; r < live; ++r) {
        const int c = __shfl(count, r);
        if (c > best_count) { best_count = c; best_rank = r; }
    }
    const int domain = __shfl(lab, best_rank);
    if (lane < KNN_KMAX) {
        res[q].idx[lane] = idx;
        res[q].cosine[lane] = key ? knn_key_value(key) * invq : 0.f;
    }
    if (lane == 0) {
        res[q].domain = live > 0 ? domain : -1;
        res[q].degenerate = degenerate ? 1 : 0;
    }
}

// ------------------------------------------------------------------------------------------
// draft / verify round control (Sec. 4.2), advanced on the device
// ------------------------------------------------------------------------------------------
// A round begins: the draft's first control block
__device__ inline void round_begin(GenState *st, PassCtl *draft) {
    int remaining = st->max_new - st->emitted;
    int kmax = st->done ? 0 : min(st->max_draft, remaining - 1);
    if (kmax < 0) kmax = 0;
    st->kmax = kmax; st->k = 0;
    draft->active = kmax > 0; draft->n_rows = 1; draft->start = st->cache_len; draft->head_from = 0;
    draft->tok[0] = st->x_last;
    st->t_begin = wall_clock64();
}

__global__ void gen_init_kernel(GenState *st, PassCtl *draft, int cache_len, int x_last, int max_new, int max_draft, float thr,
                                int32_t *out_tokens) {
    st->cache_len = cache_len; st->x_last = x_last; st->emitted = 1; st->max_new = max_new;
    st->max_draft = max_draft; st->conf_thr = thr; st->done = (max_new <= 1);
    st->n_accepted = 0; st->rounds = 0; st->drafted = 0; st->accepted = 0; st->draft_passes = 0;
    st->ticks_draft = 0; st->ticks_verify = 0;
    out_tokens[0] = x_last;
    round_begin(st, draft);
}

// What a pass of a generation tells the host: one 8-byte word in host memory, its number and what came of it, so that the host sees both
// or neither. [0]: the last draft step, [1]: the last verification (a step that did not run says how things stand).
__device__ __forceinline__ void tell_host(unsigned long long *word, unsigned int number, unsigned int value) {
    __hip_atomic_store(word, ((unsigned long long)number << 32) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
constexpr unsigned int DRAFT_GOES_ON = 256;       // beside the drafts made so far in the round

__device__ inline void draft_end(GenState *st, PassCtl *draft, const HeadResult *res, unsigned long long *host, unsigned int number) {
    if (!draft->active) { tell_host(host, number, st->k); return; }
    int k = st->k;
    int d = res->tok[0]; float p = res->prob[0];
    st->drafts[k] = d; st->draft_p[k] = p;
    k += 1; st->k = k; st->draft_passes += 1;
    bool stop = (k >= st->kmax) || (st->conf_thr > 0.f && p < st->conf_thr);
    draft->active = stop ? 0 : 1;
    tell_host(host, number, k + (stop ? 0 : DRAFT_GOES_ON));
    draft->tok[0] = d;
    draft->start = st->cache_len + k;
    st->t_draft_end = wall_clock64();
}
__global__ void draft_end_kernel(GenState *st, PassCtl *draft, const HeadResult *res, unsigned long long *host, unsigned int number) { draft_end(st, draft, res, host, number); }

// expect_k >= 0: the pass was enqueued ahead of the host's knowledge, for a round of exactly expect_k drafts (its
// launch arguments and activation layout are those of expect_k + 1 rows); it runs only if the draft did stop there
__device__ inline void verify_begin(const GenState *st, const PassCtl *draft, PassCtl *ver, int expect_k) {
    const bool as_expected = expect_k < 0 || (draft->active == 0 && st->k == expect_k);
    ver->active = (st->done || !as_expected) ? 0 : 1;
    ver->n_rows = st->k + 1; ver->start = st->cache_len; ver->head_from = 0;
    ver->tok[0] = st->x_last;
    for (int i = 0; i < st->k; ++i) ver->tok[i + 1] = st->drafts[i];
}
__global__ void verify_begin_kernel(const GenState *st, const PassCtl *draft, PassCtl *ver, int expect_k) { verify_begin(st, draft, ver, expect_k); }

// Greedy acceptance and rollback: keep the leading drafts that equal the full model's own
// token, emit the model's next token after them, move the cache length behind the last kept row. The next round begins at once.
// The host learns the new count of emitted tokens.
// ver: the pass whose result this is; a pass that did not run (enqueued ahead for a draft count that did not come
// true) leaves the state alone
__device__ inline void accept(GenState *st, PassCtl *draft, const PassCtl *ver, const HeadResult *res, int32_t *out_tokens, unsigned long long *host, unsigned int number) {
    if (st->done || !ver->active) { tell_host(host + 1, number, st->emitted); return; }
    int k = st->k, j = 0;
    while (j < k && st->drafts[j] == res->tok[j]) ++j;
    int e = st->emitted;
    for (int i = 0; i < j; ++i) out_tokens[e + i] = st->drafts[i];
    out_tokens[e + j] = res->tok[j];
    st->emitted = e + j + 1;
    tell_host(host + 1, number, e + j + 1);
    st->cache_len += j + 1;
    st->x_last = res->tok[j];
    st->n_accepted = j;
    st->rounds += 1; st->drafted += k; st->accepted += j;
    if (st->emitted >= st->max_new) st->done = 1;
    // between a round's beginning and its end nothing is left out: what lies in front of a pass counts with it
    if (k > 0) st->ticks_draft += st->t_draft_end - st->t_begin;
    st->ticks_verify += wall_clock64() - (k > 0 ? st->t_draft_end : st->t_begin);
    round_begin(st, draft);
}
__global__ void accept_kernel(GenState *st, PassCtl *draft, const PassCtl *ver, const HeadResult *res, int32_t *out_tokens, unsigned long long *host, unsigned int number) {
    accept(st, draft, ver, res, out_tokens, host, number);
}

// Acceptance for a stand-alone verification call: rows tok[0..n-1] = [x_last, d_1..d_k].
__device__ inline void verify_accept(const PassCtl *ver, const HeadResult *res, int32_t *out3) {
    int k = ver->n_rows - 1, j = 0;
    while (j < k && ver->tok[j + 1] == res->tok[j]) ++j;
    out3[0] = j; out3[1] = res->tok[j]; out3[2] = ver->start + j + 1;
}
__global__ void verify_accept_kernel(const PassCtl *ver, const HeadResult *res, int32_t *out3) { verify_accept(ver, res, out3); }

// What surrounds a pass. Its control block is there already, or comes from the host (set), or a verification of a generation works it
// out (verify_begin); at its end a draft step makes draft_end, a verification accept, a verification by itself verify_accept.
enum { ENDS_NONE = 0, ENDS_DRAFT, ENDS_VERIFY, ENDS_CHECK };
struct PassEnds {
    int kind = ENDS_NONE;
    GenState *st = nullptr;
    PassCtl *draft = nullptr;
    int expect_k = -1;               // verify_begin
    int32_t *out_tokens = nullptr;   // accept
    unsigned long long *host = nullptr;      // tell_host
    unsigned int number = 0;         // of the pass
    int32_t *out3 = nullptr;         // verify_accept
    int set = 0;                     // the control block is `ctl`
    PassCtl ctl = {};
};
// The pass's control block for every workgroup of its first kernel (own: LDS); the first one leaves it for the other kernels.
__device__ __forceinline__ const PassCtl *pass_begin(const PassEnds &e, PassCtl *ctl, PassCtl *own) {
    if (e.kind != ENDS_VERIFY && !e.set) return ctl;
    if (threadIdx.x == 0) {
        if (e.set) *own = e.ctl;
        else verify_begin(e.st, e.draft, own, e.expect_k);
        if (blockIdx.x == 0) *ctl = *own;
    }
    __syncthreads();
    return own;
}
// The pass's last step, by one thread (res is not looked at if the pass did not run). seen: what pass_begin returned, where this
// is the same kernel (in memory the first workgroup may have left it a moment ago).
__device__ __forceinline__ void pass_end(const PassEnds &e, PassCtl *ctl, const PassCtl *seen, const HeadResult *res) {
    if (e.kind == ENDS_DRAFT) draft_end(e.st, ctl, res, e.host, e.number);
    else if (e.kind == ENDS_VERIFY) accept(e.st, e.draft, seen, res, e.out_tokens, e.host, e.number);
    else if (e.kind == ENDS_CHECK) verify_accept(seen, res, e.out3);
}

}  // namespace ks
