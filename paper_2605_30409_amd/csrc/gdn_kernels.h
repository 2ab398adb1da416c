// The gfx950 kernels of the GDN chunk forward.
//
// Notation (per batch b, head h; state H = S^T of shape [Dk][Dv]).  Inside a
// chunk of C = 64 tokens r = 0..63 with entry state H_0:
//   g_r   = sum_{s <= r} log alpha_s                    (log-space decay)
//   A     = strict_lower( beta_r e^{g_r - g_s} k_r . k_s )
//   T     = (I + A)^{-1}                                 (unit lower triangular)
//   W     = T diag(beta e^g) K,   Ut = T diag(beta) V    (WY factors)
//   U     = Ut - W H_0                                   (pseudo-values)
//   O     = diag(e^g) Q H_0 + (Q K^T o M) U,   M_rs = e^{g_r - g_s} (s <= r)
//   H_C   = e^{g_C} H_0 + (diag(e^{g_C - g}) K)^T U
// This is the recurrence S_t = alpha_t S_{t-1}(I - beta_t k_t k_t^T) +
// beta_t v_t k_t^T, o_t = S_t q_t, unrolled over the chunk: the token-wise
// analog of the paper's split into per-frame summaries and a short scan
// (Section "Efficient System Co-design", S_f = alpha_f P_f S_{f-1} + A_f; the
// three stages mirror its Phase A / B / C pipeline, appendix "GDN Kernel
// Details").  Decay ratios are formed as exp of log-space differences, with
// s > r masked before the exp.
//
// Workspace per (b*H + h, chunk) -- see gdn_api.hip for the byte layout:
//   gf [68]       fp32   e^{g_C - g_r} (the update's per-token key scale),
//                        then g_C, the log decay over the chunk, as one fp64,
//                        and gamma = e^{g_C}
//   W  64*Dk      E      -W (the WY factor, negated), fragment-major for the scan
//   Ut Dv*64      E      Ut, fragment-major
//   Qf 64*Dk      E      diag(e^g) Q, row fragments for the output (RAW: Q itself)
//   Pf 64*64      E      (Q K^T o M), row fragments for the output
//   er 64         fp32   RAW only: e^{g_r}
// "Fragment-major" means the exact per-lane order in which the scan's MFMAs
// consume the operand, so every scan load is one contiguous wave access:
//   W  [Dk/64 wave][4 token tile][2 k block][64 lane][8]
//        = -W[32 m + p32_row(a, li)][64 wave + 32 kb + 8 lg + e]    (tile 2 m + a)
//   Ut [Dv/16 column tile][4 token tile][64 lane][4]
//        = Ut[32 m + 8 lg + 4 a + e][16 jt + li]                      (tile 2 m + a)
// RAW (fp32, and bf16 with several scan groups): the output's products take the
// queries as they are given and e^{g_r} multiplies their fp32 sum, and the decays
// in P are the exponential of an fp64 difference, so that neither is rounded to
// the storage type, or to fp32 logarithms, before its product.  A single bf16
// scan has one rounding more in each (Q~ to bf16, wy_decay's logarithms to fp32)
// and its output waves one multiplication less per value.
// The scan reads the keys from the input itself and applies their decay
// factors in registers: the update takes K^T (diag(e^{g_C - g}) U), so no
// scaled copy of K is written.
#pragma once

#include <type_traits>

#include "gdn_device.h"

namespace gdn {

constexpr int kGateRec = kChunk + 4;  // floats per chunk gate record (see gf above)

template <class E> struct Params {
    const E *q, *k, *v;
    const float *alpha, *beta, *state_in;
    E *out;
    float *state_out;
    int B, H, T, NC;
    int c0;           // first chunk of this launch; chunk indices below count from it, up to NC
    int G, NG;        // chunks per scan group, number of groups
    float *gf;        // per (b*H + h, chunk): e^{g_C - g_r} [64], g_C (fp64), e^{g_C}, 1 unused
    E *W, *Ut, *Qf, *Pf;
    float *er;        // RAW: per (b*H + h, chunk): e^{g_r} [64]
    E *Nf;            // per (b*H + h, group): N_g = Phi_g - Gamma_g I, fragment-major
    float *PsiT;      // per (b*H + h, group): Psi_g^T [Dv][Dk]
    double *lgam;     // per (b*H + h, group): log Gamma_g
    float *HgT;       // per (b*H + h, group): entry state H^T [Dv][Dk]
};

// --------------------------------------------------------------------------
// Stage 1: per-chunk WY / UT transform.  Grid NC * B*H with the heads running
// fastest, kWyWaves waves: workgroups that run together read whole token rows
// (all heads of a chunk), and a chunk's factors are written about when its
// neighbours' are, in the order in which the scan reads them back.  With the
// chunks fastest a 3-frame call (T = 10560, H = 16) in one pass on inputs that are
// not in the caches took 230 us, with the heads fastest 196; the kernel alone on
// warm inputs is the same.
// --------------------------------------------------------------------------
// LDS: K rows, A (fp32; V rows take its place once the solve is done), T
// (fp32), gates.  52.3 KB on the bf16 path at D = 128: three workgroups per CU.
template <class E, int DK, int DV> struct WyLds {
    static constexpr int PAD = 16 / (int)sizeof(E);
    static constexpr int LDK = DK + PAD;      // K, row-major (token rows)
    static constexpr int LDV = DV + PAD;      // V, row-major
    static constexpr int LDA = kChunk + 4;    // A and T (fp32)
    static constexpr size_t szA = 4 * kChunk * LDA;
    static constexpr size_t szV = sizeof(E) * kChunk * LDV;
    static constexpr size_t oK = 0;
    static constexpr size_t oA = oK + sizeof(E) * kChunk * LDK;  // A, then V
    static constexpr size_t oT = oA + (szA > szV ? szA : szV);
    static constexpr size_t oG = oT + szA;
    static constexpr size_t bytes = oG + 8 * kChunk + 3 * 4 * kChunk;
    // waves per SIMD when as many eight-wave workgroups as fit in 160 KB share
    // a CU (the register budget the kernel is compiled for)
    static constexpr int fit = (int)((160 * 1024) / bytes);
    // (fp32: at most two, its fragments spill in the registers of a third)
    static constexpr int cap = sizeof(E) == 4 && fit > 2 ? 2 : fit;
    static constexpr int waves_per_simd = cap >= 4 ? 8 : (cap < 1 ? 2 : 2 * cap);
};

// Decay ratio e^{g_r - g_s} (s <= r) inside the WY kernel.  The fp32 path
// takes the difference of the fp64 cumulative sums (full precision even when
// the decay over a chunk is huge); the bf16 path takes it from fp32 copies of
// g * log2(e), whose rounding (at most ~1e-3 relative to the ratio when
// |g| ~ 5600, the extreme of a chunk of alpha ~ 0) is far below bf16's.
template <class E>
__device__ __forceinline__ float wy_decay(const double *sg, const float *sgl, int r, int s) {
    constexpr double kLog2e = 1.4426950408889634;
    if constexpr (sizeof(E) == 2)
        return __builtin_amdgcn_exp2f(sgl[r] - sgl[s]);
    else
        return __builtin_amdgcn_exp2f((float)((sg[r] - sg[s]) * kLog2e));
}

constexpr int kWyWaves = 8;

template <class E, int DK, int DV, bool RAW>
__global__ __launch_bounds__(64 * kWyWaves)
__attribute__((amdgpu_waves_per_eu(WyLds<E, DK, DV>::waves_per_simd))) void gdn_wy_kernel(Params<E> p) {
    using L = WyLds<E, DK, DV>;
    using TR = Tr<E>;
    using frag = typename TR::frag;
    constexpr int NWV = kWyWaves, NT = 64 * NWV;
    constexpr int VE = 16 / (int)sizeof(E);       // elements per 16-byte vector
    constexpr int NKV = kChunk * (DK / VE) / NT;   // K vectors per thread
    constexpr int NVV = kChunk * (DV / VE) / NT;   // V vectors per thread
    static_assert(NKV * NT == kChunk * (DK / VE) && NVV * NT == kChunk * (DV / VE), "whole vectors per thread");
    constexpr int NFR = (DK / 64) * 8;             // W fragments per chunk
    constexpr double kLog2e = 1.4426950408889634;
    extern __shared__ __align__(16) unsigned char smem[];
    E *sK = (E *)(smem + L::oK);
    float *sA = (float *)(smem + L::oA);
    E *sV = (E *)(smem + L::oA);                  // V rows, once A is dead
    float *sT = (float *)(smem + L::oT);
    double *sg = (double *)(smem + L::oG);        // g_r
    float *sb = (float *)(sg + kChunk);           // beta_r
    float *sw = sb + kChunk;                      // -beta_r e^{g_r}
    float *sgl = sw + kChunk;                     // g_r log2(e) in fp32 (bf16 path)

    const int c = blockIdx.x / (p.B * p.H), bh = blockIdx.x - c * (p.B * p.H);
    const int b = bh / p.H, h = bh - b * p.H;
    // w is wave-uniform: scalar branches and table lookups
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, li = l & 15,
              lg = l >> 4;
    const int t0 = (p.c0 + c) * kChunk;
    const int nvalid = min(kChunk, p.T - t0);
    const size_t cidx = (size_t)bh * p.NC + c;
    const size_t row0 = ((size_t)b * p.T + t0) * p.H + h;  // token-row index of token t0
    const size_t rstride = (size_t)p.H;                    // token-row stride

    // Gates first (they head the dependency chain), then K rows with 16-byte
    // coalesced loads (padding rows are zero).  The queries (first needed after
    // the A tiles) and V (needed only for U~ at the end) are requested after
    // the first barrier, so that the gate and K requests of all the workgroups
    // starting together are served first.
    float ga = 1.f, gbe = 0.f;  // alpha, beta of token l (wave 0; padding: 1, 0)
    if (w == 0 && l < nvalid) {
        ga = p.alpha[row0 + l * rstride];
        gbe = p.beta[row0 + l * rstride];
    }
    uint4 kreg[NKV], vreg[NVV];
#pragma unroll
    for (int n = 0; n < NKV; ++n) {
        const int idx = tid + NT * n, r = idx / (DK / VE), cv = idx % (DK / VE);
        kreg[n] = make_uint4(0u, 0u, 0u, 0u);
        if (r < nvalid) kreg[n] = *(const uint4 *)(p.k + (row0 + r * rstride) * DK + cv * VE);
    }
    // Fused output: six (token tile rt, s block m) jobs on waves 1..6, run
    // while wave 0 inverts the diagonal blocks: job j = w - 1 is (j, 0) for
    // j < 4 (these also write the tile's Qf) and (j - 2, 1) for j = 4, 5.
    // Q rows of the job's 16 tokens as row fragments (Q[r][32 kb + 8 lg + e],
    // r = 16 rt + li; padded tokens are 0).
    const int qj = w - 1;
    const int qjob_rt = qj < 4 ? qj : qj - 2, qjob_m = qj < 4 ? 0 : 1;
    const bool qjob = w >= 1 && w <= 6;
    const int rq = 16 * qjob_rt + li;
    frag qf[DK / 32];
    // Gates: wave-wide inclusive prefix sum of clamped log alpha in fp64
    // (padding tokens: alpha = 1, beta = 0).
    if (w == 0) {
        const float be = gbe;
        float la = logf(ga);
        la = (la < kLogAlphaMin) ? kLogAlphaMin : la;  // keeps NaN
        double g = (double)la;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const double o = __shfl_up(g, d);
            if (l >= d) g += o;
        }
        const double gC = __shfl(g, kChunk - 1);
        const float eg = __builtin_amdgcn_exp2f((float)(g * kLog2e));
        sg[l] = g;
        sgl[l] = (float)(g * kLog2e);
        sb[l] = be;
        sw[l] = -be * eg;
        p.gf[cidx * kGateRec + l] = __builtin_amdgcn_exp2f((float)((gC - g) * kLog2e));
        if (l == 0) {
            *(double *)(p.gf + cidx * kGateRec + kChunk) = gC;
            p.gf[cidx * kGateRec + kChunk + 2] = expf((float)gC);
        }
    }
#pragma unroll
    for (int n = 0; n < NKV; ++n) {
        const int idx = tid + NT * n, r = idx / (DK / VE), cv = idx % (DK / VE);
        *(uint4 *)(sK + r * L::LDK + cv * VE) = kreg[n];
    }
    lds_barrier();
    if (qjob) {
#pragma unroll
        for (int kb = 0; kb < DK / 32; ++kb)
            qf[kb] = rq < nvalid ? load_frag<E>(p.q + (row0 + rq * rstride) * DK + 32 * kb, lg)
                                 : TR::cat(TR::zero(), TR::zero());
    }
#pragma unroll
    for (int n = 0; n < NVV; ++n) {
        const int idx = tid + NT * n, r = idx / (DV / VE), cv = idx % (DV / VE);
        vreg[n] = make_uint4(0u, 0u, 0u, 0u);
        if (r < nvalid) vreg[n] = *(const uint4 *)(p.v + (row0 + r * rstride) * DV + cv * VE);
    }

    // A = strict_lower(beta_r e^{g_r - g_s} K K^T): the 10 lower 16x16 blocks.
    for (int t = w; t < 10; t += NWV) {
        const int bi = (t >= 6) ? 3 : (t >= 3) ? 2 : (t >= 1) ? 1 : 0;
        const int bj = t - bi * (bi + 1) / 2;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < DK / 32; ++kb)
            acc = TR::mma(load_frag<E>(sK + (16 * bi + li) * L::LDK + 32 * kb, lg),
                          load_frag<E>(sK + (16 * bj + li) * L::LDK + 32 * kb, lg), acc);
        const int s2 = 16 * bj + li;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 16 * bi + 4 * lg + q;
            float val = 0.f;
            if (s2 < r) val = sb[r] * wy_decay<E>(sg, sgl, r, s2) * acc[q];
            sA[r * L::LDA + s2] = val;
        }
    }
    lds_barrier();

    // T = (I + A)^{-1} in fp32.  Wave 0 inverts the four diagonal 16x16 blocks
    // by forward substitution (lane = block * 16 + column) while waves 1..6
    // produce the fused-output score fragments, which need only Q, K and the
    // gates.
    if (w == 0) {
        const int base = 16 * (l >> 4), j = l & 15;
        float x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float *arow = sA + (base + r) * L::LDA + base;
            float acc = (r == j) ? 1.f : 0.f;
#pragma unroll
            for (int s4 = 0; s4 < (r + 3) / 4; ++s4) {
                const f32x4 av = *(const f32x4 *)(arow + 4 * s4);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (4 * s4 + e < r) acc -= av[e] * x[4 * s4 + e];
            }
            x[r] = acc;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) sT[(base + r) * L::LDA + base + j] = x[r];
    } else {
        // Fused output: job (rt, m) writes, for token tile rt,
        //   Qf[rt][kb][lane][e] = e^{g_r} Q[r][32 kb + 8 lg + e]      (m = 0 jobs; RAW: Q, and
        //                         er[r] = e^{g_r})
        //   Pf[rt][m][lane][e]  = e^{g_r - g_s} q_r . k_s (s <= r, else 0), s = 32 m + 8 lg + e,
        // the row fragments (B operands over d, resp. s) of the fused output.
        // P^T tiles take their s rows in P32 order, so a tile pair is one
        // fragment; block m = 1 only matters for r >= 32.
        if (qjob) {
            if (qjob_m == 0) {
                const float er = expf((float)sg[rq]);
                E *Qf = p.Qf + cidx * (size_t)kChunk * DK + l * 8;
#pragma unroll
                for (int kb = 0; kb < DK / 32; ++kb) {
                    frag qs = qf[kb];
                    if constexpr (!RAW)
                        qs = TR::cat(TR::from_f32(TR::to_f32(TR::lo(qs)) * er), TR::from_f32(TR::to_f32(TR::hi(qs)) * er));
                    TR::store8(Qf + (size_t)(qjob_rt * (DK / 32) + kb) * 512, qs);
                }
                if (RAW && lg == 0) p.er[cidx * kChunk + rq] = er;
            }
            E *Pf = p.Pf + cidx * (size_t)kChunk * kChunk + l * 8;
            const int m = qjob_m;
            typename TR::quad pq[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < DK / 32; ++kb)
                    acc = TR::mma(load_frag<E>(sK + (32 * m + p32_row(a, li)) * L::LDK + 32 * kb, lg), qf[kb], acc);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int s2 = 32 * m + 8 * lg + 4 * a + q;
                    const float dec = RAW ? expf((float)(sg[rq] - sg[s2])) : wy_decay<E>(sg, sgl, rq, s2);
                    acc[q] = (s2 <= rq) ? dec * acc[q] : 0.f;
                }
                pq[a] = TR::from_f32(acc);
            }
            TR::store8(Pf + (size_t)(qjob_rt * 2 + m) * 512, TR::cat(pq[0], pq[1]));
        }
    }
    lds_barrier();
    // Off-diagonal blocks by block distance: T_ij = -T_ii sum_{m=j}^{i-1} A_im T_mj.
    for (int dist = 1; dist < 4; ++dist) {
        if (w < 4 - dist) {
            const int j = w, i = w + dist;
            f32x4 X = {0.f, 0.f, 0.f, 0.f};
            for (int m = j; m < i; ++m) {
                const f32x4 a = *(const f32x4 *)(sA + (16 * i + li) * L::LDA + 16 * m + 4 * lg);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    X = mma_f32_k4(a[q], sT[(16 * m + 4 * lg + q) * L::LDA + 16 * j + li], X);
            }
            const f32x4 a = *(const f32x4 *)(sT + (16 * i + li) * L::LDA + 16 * i + 4 * lg);
            f32x4 Y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; ++q) Y = mma_f32_k4(a[q], X[q], Y);
#pragma unroll
            for (int q = 0; q < 4; ++q) sT[(16 * i + 4 * lg + q) * L::LDA + 16 * j + li] = -Y[q];
        }
        lds_barrier();
    }
    // A is dead: V rows take its place (they waited in registers).
#pragma unroll
    for (int n = 0; n < NVV; ++n) {
        const int idx = tid + NT * n, r = idx / (DV / VE), cv = idx % (DV / VE);
        *(uint4 *)(sV + r * L::LDV + cv * VE) = vreg[n];
    }
    // Rows of T diag(c) (c = -beta e^g for -W, beta for U~) as 8-element
    // fragments, formed in registers from fp32 T: T[row][32 sk + 8 lg + e] c_s.
    // The blocks of T above its diagonal 16x16 blocks were never written and
    // are zero; with row = 32 m + p32_row(a, li) and sk = m they are the lanes
    // li < 8 with lg >= 2.
    f32x4 wsc[2][2], bsc[2][2];  // c_s for s = 32 sk + 8 lg + 4 h + q
#pragma unroll
    for (int sk = 0; sk < 2; ++sk)
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            wsc[sk][hh] = *(const f32x4 *)(sw + 32 * sk + 8 * lg + 4 * hh);
            bsc[sk][hh] = *(const f32x4 *)(sb + 32 * sk + 8 * lg + 4 * hh);
        }
    lds_barrier();

    // -W fragments and Ut quads.  Wave w serves the two token tiles with
    // a_s = w & 1 (st = a_s, i.e. m = 0, and st = 2 + a_s, m = 1) and takes the
    // quarter q4 = w >> 1 of their outputs, so it forms the T diag(c) row
    // fragments of its tiles once -- three (m, s block) pairs, T being lower
    // triangular -- and shares the K^T and V fragments of s block 0 between
    // the two tiles.  Every wave issues the same number of MFMAs.
    static_assert(NWV == 8, "two token-tile parities x four quarters");
    const int as = w & 1, q4 = w >> 1;
    frag tw[3], tb[3];  // (m, sk) = (0, 0), (1, 0), (1, 1)
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int m = i > 0 ? 1 : 0, sk = i == 2 ? 1 : 0;
        const float *trow = sT + (32 * m + p32_row(as, li)) * L::LDA + 32 * sk + 8 * lg;
        f32x4 t0 = *(const f32x4 *)trow, t1 = *(const f32x4 *)(trow + 4);
        if (sk == m && lg >= 2 && li < 8) t0 = t1 = f32x4{0.f, 0.f, 0.f, 0.f};
        tw[i] = TR::cat(TR::from_f32(t0 * wsc[sk][0]), TR::from_f32(t1 * wsc[sk][1]));
        tb[i] = TR::cat(TR::from_f32(t0 * bsc[sk][0]), TR::from_f32(t1 * bsc[sk][1]));
    }
    // -W, computed transposed (W^T = K^T (T diag(beta e^g))^T) so that each lane
    // ends up holding the 8 consecutive Dk entries the scan consumes: fragment
    // f = (wave * 4 + st) * 2 + kb, lane (li, lg) =
    // -W[32 m + p32_row(a_s, li)][64 wave + 32 kb + 8 lg + e]  (st = 2 m + a_s).
    constexpr int NWC = NFR / 4;  // (wave, kb) combinations per token tile
    if (q4 < NWC) {
        const int wv = q4 >> 1, kb = q4 & 1, d0 = 64 * wv + 32 * kb;
        f32x4 w0[2], w1[2];  // tiles m = 0 and m = 1
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const frag k0 = tr_frag<E>(sK, L::LDK, 0, d0, true, a, li, lg);
            const frag k1 = tr_frag<E>(sK, L::LDK, 32, d0, true, a, li, lg);
            const f32x4 z = {0.f, 0.f, 0.f, 0.f};
            w0[a] = TR::mma(k0, tw[0], z);
            w1[a] = TR::mma(k1, tw[2], TR::mma(k0, tw[1], z));
        }
        E *Wf = p.W + cidx * (size_t)kChunk * DK + l * 8;
        TR::store8(Wf + ((wv * 4 + as) * 2 + kb) * 512, TR::cat(TR::from_f32(w0[0]), TR::from_f32(w0[1])));
        TR::store8(Wf + ((wv * 4 + 2 + as) * 2 + kb) * 512, TR::cat(TR::from_f32(w1[0]), TR::from_f32(w1[1])));
    }
    // Ut tiles (jt, st) in P32 row order, written as fragment-major quads
    // u = 4 jt + st: lane (li, lg) = Ut[32 m + 8 lg + 4 a_s + q][16 jt + li].
    constexpr int NJ = DV / 16;
    E *Uf = p.Ut + cidx * (size_t)DV * kChunk + l * 4;
#pragma unroll
    for (int j = 0; j < NJ / 4; ++j) {
        const int jt = q4 * (NJ / 4) + j;
        const frag v0 = tr_frag<E>(sV, L::LDV, 0, 16 * jt, false, 0, li, lg);
        const frag v1 = tr_frag<E>(sV, L::LDV, 32, 16 * jt, false, 0, li, lg);
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        TR::store(Uf + (4 * jt + as) * 256, TR::from_f32(TR::mma(tb[0], v0, z)));
        TR::store(Uf + (4 * jt + 2 + as) * 256, TR::from_f32(TR::mma(tb[2], v1, TR::mma(tb[1], v0, z))));
    }
}

// --------------------------------------------------------------------------
// Stage 2: the state recurrence across chunks, H_c = gamma_c H_{c-1} + K_c^T D_c U_c
// with U_c = Ut_c - W_c H_{c-1} and D_c = diag(e^{g_C - g}), i.e.
// H_c = A_c H_{c-1} + B_c with the affine chunk transfer
// A_c = gamma_c I - K_c^T D_c W_c, B_c = K_c^T D_c Ut_c (the token-wise
// counterpart of the paper's S_f = alpha_f P_f S_{f-1} + A_f).  The chunks are
// cut into groups of G; the sequential dependency is reduced to one step per
// group:
//   (T) gdn_chunkscan_kernel<.., SCAN_TRANS>: for every group in parallel, run
//       the recurrence over its chunks from [Phi | Psi] = [I | 0], giving the
//       group transfer Phi_g = prod A_c and the zero-start state Psi_g;
//   (S) gdn_groupscan_kernel: H <- Phi_g H + Psi_g over the groups, recording
//       every group's entry state (and the final state);
//   (O) gdn_chunkscan_kernel<.., SCAN_STATES>: for every group in parallel, run
//       the recurrence from the group's true entry state and form the output.
// With a single group only (O) runs, from state_in, and writes state_out.
//
// gdn_chunkscan_kernel: a workgroup owns 16 * CT state columns of one
// (b, h, group), the state split over four compute waves by rows.  Wave s holds
// the fp32 accumulators of row tiles RT s .. RT s + RT - 1 (RT = Dk / 64) and
// computes token tile s of U = Ut - W H, then its own rows of the update
// H <- gamma H + K^T (diag(e^{g_C - g}) U).  Both products need what the other
// waves made, so a chunk has two phases with a barrier in front of each:
//   B1(c)  H_{c-1} (rounded to E, as MFMA operands) is in LDS
//          phase 1: W H and the conversion of U, written to LDS
//   B2(c)  U_c is in LDS
//          phase 2: the update, the new H written to LDS
// A phase is one LDS round trip, one short chain of MFMAs and a few
// conversions; with the rows on one wave the step was 36 MFMAs and 80 VALU
// instructions in a row on one SIMD while three others had nothing to do.
// NOW output waves read the same H and U operands and form the output of
// 4 / NOW token tiles each: Q~ H in phase 1, + P U and the store in phase 2.
//
// -W and U~t go straight from the workspace to the registers of the wave that
// needs them, four chunks ahead (the fragment-major layout is for this).  The
// key rows are read by all waves, transposed, so two loader waves stream them
// (and the gate records) from the input into a ring of DEPTH LDS slots with
// asynchronous global->LDS copies (1 KB per instruction, lane i's 16 bytes
// landing at +16 i, each row's pieces permuted, see kswz).  The compute waves
// take K(c) into registers in phase 1 of chunk c, so its slot is refilled for
// chunk c + DEPTH from B2(c) on: a copy has DEPTH - 1/2 steps to land.
//
// What bounds a step (T = 3520, D = 128, 55 steps): it takes 0.70 us with 8
// workgroups on the chip (one head), 0.72 with 128 and 0.76 with 256, so the bound
// is inside the CU.  A workgroup takes in 56 KB a step (W, K and Q~ 16 KB each, P 6,
// U~t 2); a bare load of as much in the same pattern takes 0.45 us with 16 to 64
// workgroups and 0.56 with 128 (125 and 100 B/ns into one CU), the compute waves
// alone (a copy of the kernel that leaves the loads out) 0.37: the two overlap only
// in part.  Before, one wave carried all rows of a column tile: 0.56 us of
// dependent MFMAs and VALU a step, 0.72 with the loads.  So where the intake weighs
// as much as the chain the kernel is as fast as before (40 us), and where the chain
// was the limit, faster: fp32 (256 MFMAs of 32 cycles a step and tile, now
// over four SIMDs) T = 3557, H = 16 250 -> 104 us, and 143 with the output in it
// where a kernel of its own took 83 more; the grouped passes of two
// heads at T = 10560 18.4 -> 12 us (transfers) and 22.9 + 9.6 -> 13 us (states,
// which then formed the output in a kernel of its own); D = 64 x 80 heads, with
// two column tiles per workgroup, 307 -> 174 us.
// --------------------------------------------------------------------------
enum { SCAN_TRANS = 0, SCAN_STATES = 1 };

constexpr int kScanSplit = 4;   // compute waves per workgroup

// Operand fragments in LDS that several waves write and read: fragment f of a
// buffer is one value per lane; half a of it (four of its eight elements) comes
// from another accumulator tile than the other half.  bf16: 16 bytes per lane;
// fp32: the halves in planes of 16 bytes per lane.
template <class E> struct Xch;
template <> struct Xch<uint16_t> {
    using TR = Tr<uint16_t>;
    static constexpr int BYTES = 1024;
    static __device__ __forceinline__ void put(unsigned char *b, int f, int a, int l, TR::quad v) {
        *(TR::quad *)(b + f * BYTES + l * 16 + 8 * a) = v;
    }
    static __device__ __forceinline__ void put2(unsigned char *b, int f, int l, TR::quad lo, TR::quad hi) {
        *(TR::frag *)(b + f * BYTES + l * 16) = TR::cat(lo, hi);
    }
    static __device__ __forceinline__ TR::frag get(const unsigned char *b, int f, int l) {
        return *(const TR::frag *)(b + f * BYTES + l * 16);
    }
};
template <> struct Xch<float> {
    using TR = Tr<float>;
    static constexpr int BYTES = 2048;
    static __device__ __forceinline__ void put(unsigned char *b, int f, int a, int l, TR::quad v) {
        *(TR::quad *)(b + f * BYTES + a * 1024 + l * 16) = v;
    }
    static __device__ __forceinline__ void put2(unsigned char *b, int f, int l, TR::quad lo, TR::quad hi) {
        put(b, f, 0, l, lo);
        put(b, f, 1, l, hi);
    }
    static __device__ __forceinline__ TR::frag get(const unsigned char *b, int f, int l) {
        return TR::cat(*(const TR::quad *)(b + f * BYTES + l * 16), *(const TR::quad *)(b + f * BYTES + 1024 + l * 16));
    }
};

template <class E, int DK, int CT, int NOW> struct ScanLds {
    static constexpr int KB = DK / 32;                     // 32-row blocks of the state
    static constexpr int NT = DK / 16;                     // 16-row tiles of the state
    static constexpr int WK = kChunk * DK;                 // elements of -W (and of K) per chunk
    static constexpr int W_BYTES = WK * (int)sizeof(E);
    static constexpr int oD = W_BYTES;                     // in a slot: key rows, gate record
    static constexpr int SLOT = oD + 4 * kGateRec;
    static constexpr int NC_W = W_BYTES / 1024;            // 1 KB copies of -W (and of K)
    static constexpr int HX = CT * KB * Xch<E>::BYTES;     // H_{c-1} operands
    static constexpr int UX = CT * 2 * Xch<E>::BYTES;      // U operands (scaled for the update; as is for the output)
    static constexpr int CAP = 160 * 1024;
    static constexpr int DL = (CAP - HX - UX * (NOW ? 2 : 1)) / SLOT;
    // the loaders wait with DEPTH - 1 younger chunks in flight: vmcnt <= 63
    static constexpr int DVM = 1 + 63 / (NC_W / 2 + 1);
    static constexpr int DEPTH = 4;                        // the compute waves' unroll of four
    static constexpr int oH = DEPTH * SLOT, oU = oH + HX, oUo = oU + UX;
    static constexpr size_t bytes = oUo + (NOW ? UX : 0);
    static_assert(DEPTH <= DL && DEPTH <= DVM, "the ring fits the LDS and its waits the counter");
    static_assert(W_BYTES % 1024 == 0 && SLOT % 16 == 0, "whole 1 KB copies, aligned slots");
};

// Key rows in the scan's LDS ring: row r (a token of the chunk) holds its DK
// elements with the 16-byte granules permuted, granule g stored at g ^ kswz(r).
// The update's A operand is read with transposing reads, whose 16 lanes take
// 4 consecutive rows x 4 consecutive granules: the permutation sends them to
// 16 distinct bank groups.  kswz(r + 4) = kswz(r) for the rows r = 8 i + j,
// j < 4, those reads start from.  fp32 rows are gathered element by element
// and stay in order.
template <class E, int DK> __device__ __forceinline__ int kswz(int r) {
    constexpr int GPR = DK * (int)sizeof(E) / 16;  // granules per row
    if constexpr (sizeof(E) == 4)
        return 0;
    else if constexpr (GPR == 16)
        return 4 * (r & 3);         // 256-byte rows: the 4 rows take disjoint granule quads
    else
        return 4 * ((r >> 1) & 1);  // 128-byte rows: two per bank line, the pairs take disjoint quads
}

// Update A-operand fragment from the ring's key rows Kr (the tr_frag read in
// P32 order, through the permutation): lane (li, lg) receives
// K[row0 + 8 lg + q'][colbase + p32_row(a, li)], q' = 0..7.
template <class E, int DK>
__device__ __forceinline__ typename Tr<E>::frag kt_frag(const E *Kr, int row0, int colbase, int a, int li,
                                                        int lg) {
    if constexpr (sizeof(E) == 2) {
        typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
        const int row = row0 + 8 * lg + (li >> 2);
        const int off = 8 * ((colbase / 8 + (li & 3)) ^ kswz<E, DK>(row)) + 4 * a;
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(Kr + row * DK + off));
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(Kr + (row + 4) * DK + off));
        return Tr<E>::cat(__builtin_bit_cast(u32x2, lo), __builtin_bit_cast(u32x2, hi));
    } else {
        return tr_frag<E>(Kr, DK, row0, colbase, true, a, li, lg);
    }
}

template <int NOW> constexpr int scan_threads() { return (kScanSplit + NOW + 2) * 64; }

template <class E, int DK, int DV, int PHASE, int CT, int NOW, bool RAW>
__global__ __launch_bounds__(scan_threads<NOW>()) void gdn_chunkscan_kernel(Params<E> p) {
    using TR = Tr<E>;
    using frag = typename TR::frag;
    using quad = typename TR::quad;
    using L = ScanLds<E, DK, CT, NOW>;
    using X = Xch<E>;
    static_assert((NOW > 0) == (PHASE == SCAN_STATES), "the state pass forms the output");
    constexpr int D = L::DEPTH, NCW = kScanSplit;
    constexpr int KB = L::KB, NT = L::NT, RT = NT / NCW; // row tiles per compute wave
    constexpr int NWS = sizeof(E) == 4 ? 2 : 4;          // register sets of W and U~t (fp32: no room for four)
    constexpr int WGC = 16 * CT;                         // columns per workgroup
    constexpr int WCOLS = PHASE == SCAN_TRANS ? DK + DV : DV;
    constexpr int NJB = WCOLS / WGC;                     // column blocks per (b, h, group)
    static_assert(CT <= 2 && WCOLS % WGC == 0 && DK % WGC == 0, "column blocks do not straddle Phi and Psi");
    extern __shared__ __align__(16) unsigned char scan_lds[];
    unsigned char *hx = scan_lds + L::oH, *ux = scan_lds + L::oU, *uo = scan_lds + L::oUo;

    // XCD-aware placement: workgroups are dealt round-robin to the 8 XCDs, so
    // id = 8 slot + x runs on XCD x.  The NJB column blocks of one (b, h, group)
    // get consecutive slots of the same XCD and share its L2 for the chunk
    // operands W, K that all of them read.
    const int id = blockIdx.x, x = id & 7, slot = id >> 3;
    const int unit = (slot / NJB) * 8 + x, jb = slot % NJB;
    if (unit >= p.B * p.H * p.NG) return;
    const int bh = unit / p.NG, grp = unit - bh * p.NG;
    const int b = bh / p.H, h = bh - b * p.H;
    const int c_begin = grp * p.G, c_end = min(p.NC, c_begin + p.G);
    // w is wave-uniform: scalar branches and addresses
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, li = l & 15,
              lg = l >> 4;
    const int col0 = WGC * jb;
    const bool is_phi = PHASE == SCAN_TRANS && col0 < DK;
    // first column of this workgroup within the state (Phi columns or Psi / H columns)
    const int jw = (PHASE == SCAN_TRANS && !is_phi) ? col0 - DK : col0;
    const bool has_ut = PHASE == SCAN_STATES || !is_phi;
    // Column of the state that lane li of column tile ct holds.  With two tiles
    // the 32 columns are dealt in P32 order, so that an output wave's lane gets
    // eight consecutive output columns from the pair: one 16-byte store per
    // token, 64 contiguous bytes per token and workgroup, instead of two 8-byte
    // ones.
    auto col = [&](int ct) { return jw + (CT == 2 ? p32_row(ct, li) : 16 * ct + li); };

    if (w >= NCW + NOW) {
        // ---------------- loader waves ----------------
        // A wave needs some 50 cycles to issue a 1 KB copy, so a chunk's copies are
        // dealt to two waves and each issues half of its share in either phase: no
        // phase waits for the issue.  Past the end the loaders still issue the same
        // number of copies (so that the counts the waits rely on are constant),
        // reading the last chunk, into the slot of the missing chunk.
        const int part = w - NCW - NOW;
        constexpr int NS = L::NC_W / 2, NH = NS / 2;     // copies per wave and chunk, and per phase
        {
            // Key rows of chunk c from the input (B, T, H, DK): instruction n,
            // lane l fills LDS granule 64 n + l, i.e. granule (64 n + l) % GPR of
            // row (64 n + l) / GPR, from the row's granule permuted back by kswz.
            // Rows past the sequence's end are read from its last token; their
            // pseudo-values are exactly zero (beta = 0 and zero V and K rows in the
            // WY factors), so they add nothing to the update.
            // A copy's rows are RPC apart from the next one's, so a lane's
            // offset from the copy's first row is the same for all of them.
            constexpr int GPR = DK * (int)sizeof(E) / 16, RPC = 64 / GPR;
            const int lr = l / GPR, lc = 16 * ((l % GPR) ^ kswz<E, DK>(lr));
            const unsigned rs = (unsigned)p.H * DK * (unsigned)sizeof(E), voff = (unsigned)lr * rs + lc;
            const char *kbase = (const char *)(p.k + ((size_t)b * p.T * p.H + h) * DK);
            auto issue = [&](int c, int off, auto half) {
                constexpr int HF = decltype(half)::value;
                const int src = min(c, c_end - 1), t0 = (p.c0 + src) * kChunk, left = p.T - 1 - t0, n0 = NS * part + NH * HF;
                unsigned char *sl = scan_lds + off;
                const char *kc = kbase + (size_t)t0 * rs;
                if (left >= kChunk - 1) {
#pragma unroll
                    for (int n = 0; n < NH; ++n)
                        __builtin_amdgcn_global_load_lds(
                            (const void *)(kc + (size_t)(RPC * (n0 + n)) * rs + voff),
                            (__attribute__((address_space(3))) void *)(sl + 1024 * (n0 + n)), 16, 0, 0);
                } else {
#pragma unroll
                    for (int n = 0; n < NH; ++n)
                        __builtin_amdgcn_global_load_lds(
                            (const void *)(kc + (size_t)min(RPC * (n0 + n) + lr, left) * rs + lc),
                            (__attribute__((address_space(3))) void *)(sl + 1024 * (n0 + n)), 16, 0, 0);
                }
                // the gate record (272 bytes), a copy of its own that both waves
                // issue so that their counts agree
                if (HF == 0 && l < kGateRec / 4)
                    __builtin_amdgcn_global_load_lds(
                        (const void *)(p.gf + ((size_t)bh * p.NC + src) * kGateRec + 4 * l),
                        (__attribute__((address_space(3))) void *)(sl + L::oD), 16, 0, 0);
            };
            const std::integral_constant<int, 0> h0{};
            const std::integral_constant<int, 1> h1{};
#pragma unroll
            for (int i = 0; i < D - 1; ++i) issue(c_begin + i, i * L::SLOT, h0), issue(c_begin + i, i * L::SLOT, h1);
            issue(c_begin + D - 1, (D - 1) * L::SLOT, h0);
            int off = 0, prev = (D - 1) * L::SLOT;           // slots of chunks c and c - 1
            for (int c = c_begin; c < c_end; ++c) {
                wait_vmcnt<(D - 2) * (NS + 1) + NH + 1>();   // K(c) has landed
                lds_only_barrier();                          // B1(c)
                issue(c + D - 1, prev, h1);
                lds_only_barrier();                          // B2(c): K(c) is in registers
                issue(c + D, off, h0);
                prev = off;
                off = off + L::SLOT == D * L::SLOT ? 0 : off + L::SLOT;
            }
        }
        wait_vmcnt<0>();
        lds_only_barrier();                     // ring quiet: the compute waves may reuse it
        if (PHASE == SCAN_TRANS && is_phi) lds_only_barrier();  // matches the N staging barrier
        return;
    }

    if constexpr (NOW > 0) {
        if (w >= NCW) {
            // ---------------- output waves ----------------
            // Wave o forms, for token tiles rt = o + NOW j of each chunk and every
            // column tile,  O^T = H_{c-1}^T Q~^T + U^T P^T  (RAW: H_{c-1}^T Q^T diag(e^g) + U^T P^T):
            //   A operands: the H_{c-1} and U fragments in LDS (B-operand
            //   layout over d, resp. s, which is also the A layout),
            //   B operands: the Qf / Pf row fragments of the chunk.
            // Lane (li, lg) gets columns 4 lg + q of each tile for token 16 rt + li.
            constexpr int RO = 4 / NOW;
            const int o = w - NCW;
            struct Set {
                frag q[RO][KB], p[RO][2];
                float er[RO];                            // RAW: e^{g_r}
            };
            // Operands are requested two chunks ahead, in three register sets
            // used in turn (fp32, with longer steps and larger operands: one
            // ahead, in two sets; past the end: the last chunk's, not used), a part of
            // them at the start of either phase so that neither waits for the
            // issue.  Addresses are a uniform base and a 32-bit lane offset.
            const unsigned lo16 = 16u * l * (sizeof(frag) / 16);
            const char *qp = (const char *)(p.Qf + ((size_t)bh * p.NC + c_begin) * (size_t)kChunk * DK);
            const char *pp = (const char *)(p.Pf + ((size_t)bh * p.NC + c_begin) * (size_t)kChunk * kChunk);
            const float *ep = p.er + ((size_t)bh * p.NC + c_begin) * (size_t)kChunk + li;
            int c_req = c_begin;                         // chunk that qp, pp and ep point at
            auto ld = [&](const char *base, int f) { return TR::load8((const E *)(base + f * (int)sizeof(frag) * 64 + lo16)); };
            auto load_q = [&](Set &st, int kb0, int kb1) {
#pragma unroll
                for (int j = 0; j < RO; ++j) {
#pragma unroll
                    for (int kb = kb0; kb < kb1; ++kb) st.q[j][kb] = ld(qp, (o + NOW * j) * KB + kb);
                    if (RAW && kb0 == 0) st.er[j] = ep[16 * (o + NOW * j)];
                }
            };
            auto load_p = [&](Set &st) {
#pragma unroll
                for (int j = 0; j < RO; ++j) {
                    const int rt = o + NOW * j;
                    st.p[j][0] = ld(pp, rt * 2);
                    // block m = 1 (tokens 32 ..) only matters for rt >= 2
                    if (rt >= 2) st.p[j][1] = ld(pp, rt * 2 + 1);
                }
                if (c_req + 1 < c_end) {
                    ++c_req;
                    qp += (size_t)kChunk * DK * sizeof(E);
                    pp += (size_t)kChunk * kChunk * sizeof(E);
                    ep += kChunk;
                }
            };
            const size_t ostride = (size_t)p.H * DV;     // elements from one token's row to the next one's
            E *obase = p.out + (((size_t)b * p.T + (size_t)(p.c0 + c_begin) * kChunk) * p.H + h) * DV + jw;
            unsigned ooff[RO];
#pragma unroll
            for (int j = 0; j < RO; ++j) ooff[j] = (unsigned)((16 * (o + NOW * j) + li) * ostride + 4 * CT * lg);
            auto chunk = [&](int c, Set &st, Set &nx, auto whole) {
                lds_only_barrier();                      // B1(c)
                frag hb[CT][KB];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int kb = 0; kb < KB; ++kb) hb[ct][kb] = X::get(hx, ct * KB + kb, l);
                __builtin_amdgcn_sched_barrier(0);
                load_q(nx, 0, KB / 2);
                __builtin_amdgcn_sched_barrier(0);
                f32x4 acc[RO][CT];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int j = 0; j < RO; ++j) {
                        acc[j][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int kb = 0; kb < KB; ++kb) acc[j][ct] = TR::mma(hb[ct][kb], st.q[j][kb], acc[j][ct]);
                        if constexpr (RAW) acc[j][ct] *= st.er[j];
                    }
                lds_only_barrier();                      // B2(c)
                frag ub[CT][2];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int m = 0; m < 2; ++m) ub[ct][m] = X::get(uo, ct * 2 + m, l);
                __builtin_amdgcn_sched_barrier(0);
                load_q(nx, KB / 2, KB);
                load_p(nx);
                __builtin_amdgcn_sched_barrier(0);
                const int nvalid = p.T - (p.c0 + c) * kChunk;
#pragma unroll
                for (int j = 0; j < RO; ++j) {
                    const int rt = o + NOW * j;
                    quad oq[CT];
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        acc[j][ct] = TR::mma(ub[ct][0], st.p[j][0], acc[j][ct]);
                        if (rt >= 2) acc[j][ct] = TR::mma(ub[ct][1], st.p[j][1], acc[j][ct]);
                        oq[ct] = TR::from_f32(acc[j][ct]);
                    }
                    if (decltype(whole)::value || 16 * rt + li < nvalid) {
                        if constexpr (CT == 2)
                            TR::store8(obase + ooff[j], TR::cat(oq[0], oq[1]));
                        else
                            TR::store(obase + ooff[j], oq[0]);
                    }
                }
                obase += kChunk * ostride;
            };
            // Whole chunks a few at a time, without a branch (a branch around the
            // stores or out of the loop makes the compiler wait for operands that
            // are not needed yet); the rest, the sequence's last chunk among it,
            // one by one.
            const int c_whole = min(c_end, p.T / kChunk - p.c0);
            int c = c_begin;
            Set s0, s1;
            load_q(s0, 0, KB);
            load_p(s0);
            if constexpr (sizeof(E) == 4) {
                for (; c + 2 <= c_whole; c += 2) {
                    chunk(c, s0, s1, std::true_type{});
                    chunk(c + 1, s1, s0, std::true_type{});
                }
                if (c < c_end) chunk(c, s0, s1, std::false_type{});
                if (c + 1 < c_end) chunk(c + 1, s1, s0, std::false_type{});
            } else {
                Set s2;
                load_q(s1, 0, KB);
                load_p(s1);
                for (; c + 3 <= c_whole; c += 3) {
                    chunk(c, s0, s2, std::true_type{});
                    chunk(c + 1, s1, s0, std::true_type{});
                    chunk(c + 2, s2, s1, std::true_type{});
                }
                if (c < c_end) chunk(c, s0, s2, std::false_type{});
                if (c + 1 < c_end) chunk(c + 1, s1, s0, std::false_type{});
                if (c + 2 < c_end) chunk(c + 2, s2, s1, std::false_type{});
            }
            lds_only_barrier();                          // matches the loaders' last barrier
            return;
        }
    }

    // ---------------- compute waves ----------------
    const int s = w;                                     // token tile and share of the row tiles
    // State H[:, jw + 16 ct + li], row tiles t = RT s + i in P32 order:
    // Hacc[i][ct][q] = H[32 (t / 2) + 8 lg + 4 (t % 2) + q][jw + 16 ct + li].
    f32x4 Hacc[RT][CT];
    auto row0 = [&](int i) {
        const int t = RT * s + i;
        return 32 * (t >> 1) + 8 * lg + 4 * (t & 1);
    };
    if constexpr (PHASE == SCAN_TRANS) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    Hacc[i][ct][q] = (is_phi && row0(i) + q == col(ct)) ? 1.f : 0.f;
    } else if (p.NG > 1) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int i = 0; i < RT; ++i)
                Hacc[i][ct] = *(const f32x4 *)(p.HgT + ((size_t)unit * DV + col(ct)) * DK + row0(i));
    } else if (p.state_in) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    Hacc[i][ct][q] = p.state_in[((size_t)bh * DK + row0(i) + q) * DV + col(ct)];
    } else {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int i = 0; i < RT; ++i) Hacc[i][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    double lgam = 0.0;  // sum of gC over the group (SCAN_TRANS)

    // H rounded to E into LDS, as the B operands over its 32-row blocks
    auto put_h = [&]() {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            quad hq[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i) hq[i] = TR::from_f32(Hacc[i][ct]);
            if constexpr (RT == 2)
                X::put2(hx, ct * KB + s, l, hq[0], hq[1]);
            else
                X::put(hx, ct * KB + (s >> 1), s & 1, l, hq[0]);
        }
    };
    // this wave's U~t quads: tokens 32 m + 8 lg + 4 a + q (s = 2 m + a); requested
    // NWS chunks ahead, ut running over the chunks (past the end: the last one)
    const char *ut = (const char *)(p.Ut + ((size_t)bh * p.NC + c_begin) * (size_t)DV * kChunk) +
                     (size_t)(jw / 16) * 1024 * sizeof(E);
    unsigned uoff[CT];                                   // column c sits in lane c % 16 of tile c / 16
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const int c = col(ct) - jw;
        uoff[ct] = (1024 * (c >> 4) + s * 256 + (16 * lg + (c & 15)) * 4) * (unsigned)sizeof(E);
    }
    int u_left = c_end - 1 - c_begin;                    // chunks after the one ut points at
    auto load_us = [&](quad (&us)[CT]) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
            us[ct] = has_ut ? TR::load((const E *)(ut + uoff[ct])) : TR::zero();
        ut += u_left > 0 ? (size_t)DV * kChunk * sizeof(E) : 0;
        --u_left;
    };
    // -W fragments of token tile s (k block kb of wave-row pair kb / 2), straight
    // from the workspace: no other wave needs them.  Requested NWS chunks ahead,
    // like U~t.
    const char *wp = (const char *)(p.W + ((size_t)bh * p.NC + c_begin) * (size_t)L::WK);
    const unsigned woff = (s * 1024 + l * 8) * (unsigned)sizeof(E);
    auto load_w = [&](frag (&wf)[KB]) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
            wf[kb] = TR::load8((const E *)(wp + ((kb >> 1) * 4096 + (kb & 1) * 512) * sizeof(E) + woff));
        wp += u_left > 0 ? (size_t)L::W_BYTES : 0;
    };
    // One chunk: U = U~t - W H_{c-1} (the workspace holds -W), then
    // H_c = gamma H_{c-1} + K^T (diag(e^{g_C - g}) U).
    // Chunk c_begin + j sits in slot j % D and its W and U~t in set j % NWS, so with
    // four steps in a row every LDS address is a constant.
    auto step = [&](auto j_, quad (&us)[CT], frag (&wf)[KB]) {
        constexpr int J = decltype(j_)::value;
        lds_only_barrier();                              // B1(c)
        const unsigned char *sl = scan_lds + (J % D) * L::SLOT;
        frag hb[KB][CT], kf[RT][2];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) hb[kb][ct] = X::get(hx, ct * KB + kb, l);
        const float *Dl = (const float *)(sl + L::oD);
        const float gam = Dl[kChunk + 2];
        const f32x4 dsc = *(const f32x4 *)(Dl + 32 * (s >> 1) + 8 * lg + 4 * (s & 1));
        if constexpr (PHASE == SCAN_TRANS) lgam += *(const double *)(Dl + kChunk);
        // K^T fragments of the wave's rows: rows d in P32 order 32 (t / 2) +
        // p32_row(t % 2, li), tokens 32 m + 8 lg + e
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const int t = RT * s + i;
                kf[i][m] = kt_frag<E, DK>((const E *)sl, 32 * m, 32 * (t >> 1), t & 1, li, lg);
            }
        f32x4 u[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) u[ct] = TR::to_f32(us[ct]);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) u[ct] = TR::mma(wf[kb], hb[kb][ct], u[ct]);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            X::put(ux, ct * 2 + (s >> 1), s & 1, l, TR::from_f32(u[ct] * dsc));
            if constexpr (NOW > 0) X::put(uo, ct * 2 + (s >> 1), s & 1, l, TR::from_f32(u[ct]));
        }
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) Hacc[i][ct] *= gam;
        lds_only_barrier();                              // B2(c)
        frag uk[2][CT];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) uk[m][ct] = X::get(ux, ct * 2 + m, l);
        load_w(wf);
        load_us(us);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) Hacc[i][ct] = TR::mma(kf[i][m], uk[m][ct], Hacc[i][ct]);
        put_h();
    };
    quad us[NWS][CT];
    frag wf[NWS][KB];
#pragma unroll
    for (int i = 0; i < NWS; ++i) {
        load_w(wf[i]);
        load_us(us[i]);
    }
    put_h();
    int c = c_begin;
    const std::integral_constant<int, 0> j0{};
    const std::integral_constant<int, 1> j1{};
    const std::integral_constant<int, 2> j2{};
    const std::integral_constant<int, 3> j3{};
    for (; c + 4 <= c_end; c += 4) {
        step(j0, us[0 % NWS], wf[0 % NWS]);
        step(j1, us[1 % NWS], wf[1 % NWS]);
        step(j2, us[2 % NWS], wf[2 % NWS]);
        step(j3, us[3 % NWS], wf[3 % NWS]);
    }
    if (c < c_end) step(j0, us[0 % NWS], wf[0 % NWS]);
    if (c + 1 < c_end) step(j1, us[1 % NWS], wf[1 % NWS]);
    if (c + 2 < c_end) step(j2, us[2 % NWS], wf[2 % NWS]);
    lds_only_barrier();  // the loaders have drained: the ring is free

    const size_t gidx = (size_t)bh * p.NG + grp;
    if constexpr (PHASE == SCAN_STATES) {
        if (p.NG == 1 && p.state_out) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        p.state_out[((size_t)bh * DK + row0(i) + q) * DV + col(ct)] = Hacc[i][ct][q];
        }
    } else if (!is_phi) {  // SCAN_TRANS from here on
        // Psi_g^T [Dv][Dk], fp32
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int i = 0; i < RT; ++i)
                *(f32x4 *)(p.PsiT + (gidx * DV + col(ct)) * DK + row0(i)) = Hacc[i][ct];
    } else {
        if (jb == 0 && w == 0 && l == 0) p.lgam[gidx] = lgam;
        // N_g = Phi_g - Gamma_g I, rounded to E, staged in LDS (in the ring
        // memory) as N^T (row e = state column - col0, rows d contiguous) and
        // re-read with the transposing LDS read into the group scan's A-operand
        // fragments: fragment (wave v, row tile t, k block kb), lane (li, lg) =
        //   N[64 v + 32 (t / 2) + p32_row(t % 2, li)][32 kb + 8 lg + e].
        static_assert(PHASE != SCAN_TRANS || WGC % 32 == 0, "the transfer pass writes whole 32-column k blocks");
        constexpr int LDN = DK + 16 / (int)sizeof(E);
        static_assert((int)sizeof(E) * WGC * LDN <= L::oH, "N^T staging");
        const float Gam = expf((float)lgam);
        E *sN = (E *)scan_lds;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const int e = col(ct) - jw;                  // staging row
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                f32x4 n = Hacc[i][ct];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (row0(i) + q == col0 + e) n[q] -= Gam;
                TR::store(sN + e * LDN + row0(i), TR::from_f32(n));
            }
        }
        lds_only_barrier();  // staging written (the loaders take this barrier too)
        const int kb0 = col0 / 32;
        constexpr int NKB = WGC / 32;                       // k blocks in this workgroup
        constexpr int NFRAG = (DK / 64) * 4 * NKB;
        E *Nf = p.Nf + gidx * (size_t)DK * DK + l * 8;
        for (int f = w; f < NFRAG; f += NCW) {
            const int v = f / (4 * NKB), t = (f / NKB) % 4, kk = f % NKB;
            const frag nf = tr_frag<E>(sN, LDN, 32 * kk, 64 * v + 32 * (t >> 1), true, t & 1, li, lg);
            TR::store8(Nf + (size_t)((v * 4 + t) * (DK / 32) + kb0 + kk) * 512, nf);
        }
    }
}

// --------------------------------------------------------------------------
// Group scan: H <- Gamma_g H + N_g H + Psi_g over the groups of one (b, h), in
// 16-column blocks (one workgroup each, four waves splitting the rows, which
// exchange their shares of H each step through LDS).  Records every group's
// entry state H^T for the state stage and writes the final state.  A step is
// short next to the latency of its operands (N_g alone is 32 KB in bf16), so
// they are requested four groups ahead, in four register sets used in turn:
// with one group's notice the step took 1.85 us (bf16, D = 128).
// --------------------------------------------------------------------------
template <class E, int DK, int DV>
__global__ __launch_bounds__(64 * kScanSplit) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gdn_groupscan_kernel(Params<E> p) {
    using TR = Tr<E>;
    using X = Xch<E>;
    using frag = typename TR::frag;
    using quad = typename TR::quad;
    constexpr int RT = DK / 16 / kScanSplit;             // row tiles per wave
    constexpr int NJ = DV / 16;
    constexpr int KB = DK / 32;
    __shared__ __align__(16) unsigned char sH[2][KB * X::BYTES];  // H rounded to E, double-buffered

    const int id = blockIdx.x, x = id & 7, slot = id >> 3;
    const int bh = (slot / NJ) * 8 + x, jt = slot % NJ;
    if (bh >= p.B * p.H) return;
    const int tid = threadIdx.x, s = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, li = l & 15, lg = l >> 4;
    const int j = 16 * jt + li;
    auto row0 = [&](int i) {
        const int t = RT * s + i;
        return 32 * (t >> 1) + 8 * lg + 4 * (t & 1);
    };

    f32x4 Hacc[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            Hacc[i][q] = p.state_in ? p.state_in[((size_t)bh * DK + row0(i) + q) * DV + j] : 0.f;
    struct Set {
        frag nf[RT][KB];
        f32x4 ps[RT];
        double lg;
    };
    auto fetch = [&](int g, Set &o) {                    // past the end: the last group's, not used
        const size_t gidx = (size_t)bh * p.NG + min(g, p.NG - 1);
        const E *Nc = p.Nf + gidx * (size_t)DK * DK + (size_t)RT * s * KB * 512 + l * 8;
#pragma unroll
        for (int i = 0; i < RT; ++i) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) o.nf[i][kb] = TR::load8(Nc + (i * KB + kb) * 512);
            o.ps[i] = *(const f32x4 *)(p.PsiT + (gidx * DV + j) * DK + row0(i));
        }
        o.lg = p.lgam[gidx];
    };
    auto step = [&](int g, Set &o) {
        unsigned char *sh = sH[g & 1];
        float *Hg = p.HgT + (((size_t)bh * p.NG + g) * DV + j) * DK;   // entry state of group g
        quad hq[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            hq[i] = TR::from_f32(Hacc[i]);
            if constexpr (RT == 1) X::put(sh, s >> 1, s & 1, l, hq[0]);
        }
        if constexpr (RT == 2) X::put2(sh, s, l, hq[0], hq[1]);
#pragma unroll
        for (int i = 0; i < RT; ++i) *(f32x4 *)(Hg + row0(i)) = Hacc[i];
        lds_only_barrier();
        const float Gam = expf((float)o.lg);
#pragma unroll
        for (int i = 0; i < RT; ++i) Hacc[i] = Hacc[i] * Gam + o.ps[i];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const frag hb = X::get(sh, kb, l);
#pragma unroll
            for (int i = 0; i < RT; ++i) Hacc[i] = TR::mma(o.nf[i][kb], hb, Hacc[i]);
        }
        fetch(g + 4, o);
    };
    Set o0, o1, o2, o3;
    fetch(0, o0);
    fetch(1, o1);
    fetch(2, o2);
    fetch(3, o3);
    int g = 0;
    for (; g + 4 <= p.NG; g += 4) {
        step(g, o0);
        step(g + 1, o1);
        step(g + 2, o2);
        step(g + 3, o3);
    }
    if (g < p.NG) step(g, o0);
    if (g + 1 < p.NG) step(g + 1, o1);
    if (g + 2 < p.NG) step(g + 2, o2);
    if (p.state_out) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) p.state_out[((size_t)bh * DK + row0(i) + q) * DV + j] = Hacc[i][q];
    }
}

}  // namespace gdn
