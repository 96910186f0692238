// Perturbation-batched contraction (Section II.B, the pair part of the
// E_{G,G} inner sums), recombined into two well-scaled channels per point:
//
//   Y_i = sum_j K_ij X_j,   X_j = [p_j; q_j] (2 x P), K_ij (2 x 2):
//     K_pp = Phi + c_i Phi_g + c_j Phi_g' + c_i c_j Phi_gg'
//     K_pq = R^2 (Phi_g' + c_i Phi_gg')
//     K_qp = R^2 (Phi_g  + c_j Phi_gg')
//     K_qq = R^4 Phi_gg'
//   with p = w rho^x, q = w rho (omega_r rho^x + omega_g gamma^x),
//   c = rho dkappa/drho, Phi_g = -Phi (1/g + 1/s), Phi_g' = -Phi (1/g' + 1/s),
//   Phi_gg' = 2 Phi (1/(g g') + 1/s^2), s = g + g'.
//
// Summed over i and j, X_i^T K_ij X_j equals the paper's
// sum_ij w_i w_j [rho^A_i (f^{rho rho}_ij rho^B_j + f^{rho gamma}_ij gamma^B_j)
//                + gamma^A_i (f^{gamma rho}_ij rho^B_j + f^{gamma gamma}_ij gamma^B_j)]
// without the delta_ij local terms, which the assembly adds.
//
// This is a dense (2N x 2N) x (2N x P) product whose left operand is never
// stored: every (i, j) pair is formed once, in registers, directly in the
// MFMA A-operand layout.  X chunks are staged in LDS and shared by the waves
// of a workgroup (four, or eight for the split-BF16 form with eight or more
// column blocks); every wave owns 16 outer points and all columns of its
// column group, with accumulators in registers.  Three arithmetic modes:
//
//  FP64:   one pair per lane per 16 x 4 block, four v_mfma_f64_16x16x4 per
//          16 columns (K_pp X_p, K_pq X_q into Y_p; K_qp X_p, K_qq X_q into Y_q),
//          or four v_mfma_f64_4x4x4 per 4 columns past the last whole 16.
//  FP32:   the same scheme with v_mfma_f32_16x16x4 and FP32 pair arithmetic.
//  BF16X3: four pairs per lane per 16 x 16 block; the MFMA K index runs over
//          (j, channel), k = 2 (j mod 16) + c, so one v_mfma_f32_16x16x32_bf16
//          contracts K_pp, K_pq (or K_qp, K_qq) of 16 j with both channels of X.
//          Each operand is split as v = hi + lo with hi = bf16(v),
//          lo = bf16(v - hi), and three products hi*hi + hi*lo + lo*hi are
//          accumulated (relative error about 2^-16 per product).
//
// X carries the factor -3/2 of Phi (the perturbation packing scales both
// channels), so the pair arithmetic forms K / (-3/2) with r = 1 / (g g' s) in
// place of Phi.  Using 1/(g g') = s r and
// 1/s = g g' r, each pair needs one reciprocal and
//   A = r (1/g + 1/s),  A' = r (1/g' + 1/s),  Q = 2 r (1/s^2 + 1/(g g')),
//   t1 = c_i Q - A',  t2 = c_j Q - A,
//   K_pp = r - c_i A + c_j t1,  K_pq = R^2 t1,  K_qp = R^2 t2,  K_qq = R^4 Q.
// The mixed modes accumulate at most kFp32Run consecutive j points in FP32 (the MFMA
// accumulators) and then add those sums into the split's FP64 partials; the
// assembly sums the partials over splits in FP64.  So the sums are FP32
// within a tile of kFp32Run points and FP64 across tiles and splits.
#include <type_traits>

#include "dev_common.h"
#include <algorithm>

#include "grid_tile.h"
#include "vv10_internal.h"

namespace vv10 {

namespace {

constexpr int kJC = 32;   // j points per LDS stage

template <int NCB>
constexpr int smem_f64() { return 2 * kJC * (int)sizeof(double4) + kJC * 2 * NCB * 16 * (int)sizeof(double); }

// The four kernel-derivative values of pair (i, j), divided by -3/2 (see the
// file header); a = (x, y, z, omega), (kappa, ., c, .) of each point.
__device__ __forceinline__ void pair_K64(const double4 a0, const double4 a1, const double4 b0,
                                         double bk, double cj, double &kpp, double &kpq,
                                         double &kqp, double &kqq) {
    const double dx = a0.x - b0.x, dy = a0.y - b0.y, dz = a0.z - b0.z;
    const double R2 = __builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz));
    const double gg = __builtin_fma(a0.w, R2, a1.x);
    const double gp = __builtin_fma(b0.w, R2, bk);
    const double s = gg + gp, t = gg * gp;
    const double r = rcp64(t * s);
    const double sr = s * r, is = t * r;                // 1/(g g'), 1/s
    const double A = r * __builtin_fma(gp, sr, is);     // r (1/g + 1/s)
    const double Ap = r * __builtin_fma(gg, sr, is);    // r (1/g' + 1/s)
    const double Q = (r + r) * __builtin_fma(is, is, sr);
    const double ci = a1.z;
    const double t1 = __builtin_fma(ci, Q, -Ap);
    const double t2 = __builtin_fma(cj, Q, -A);
    kpp = __builtin_fma(cj, t1, __builtin_fma(-ci, A, r));
    kpq = R2 * t1;
    kqp = R2 * t2;
    kqq = (R2 * R2) * Q;
}

// FP64 MFMA and FP64 VALU share their multipliers: measured, a 16x16x4 MFMA
// takes 64 cycles of a SIMD, an FMA 4.75, v_rcp_f64 16.5, and none of them
// overlap, so the kernel's time is the sum of both and each instruction of
// the pair arithmetic counts (about 165 cycles per wave and 64 pairs).  The
// columns past a multiple of 16 go by fours on v_mfma_f64_4x4x4 (four blocks:
// 16 rows, 4 columns, 17.3 cycles; the same A operand, and measured bitwise
// the same products as 16x16x4): P = 54 takes 227 cycles per A operand
// instead of 256, P = 18 81 instead of 128 (contraction of the hexamer
// 6.27 -> 5.89 ms, 14.8 -> 13.1 M cycles per XCD; of the dimer 0.119 -> 0.091
// ms).  NQ is a template parameter: tested in the loop, it made the compiler
// copy accumulators behind MFMA waits and cost all of the gain.
// NQ: quads of columns in the last block, 4 (the 16-column form) or fewer.
template <int NCB, bool SCR = false, int NQ = 4>
__device__ __forceinline__ void tile_f64(int64_t npad, int64_t jlen, int32_t Pp,
                                         const double4 *__restrict__ P0,
                                         const double4 *__restrict__ P1,
                                         const double *__restrict__ X, double *__restrict__ Yout,
                                         int64_t itile, int grp, int split, char *smem,
                                         const uint32_t *__restrict__ mask = nullptr) {
    constexpr int NC = NCB * 16, LB = NCB - 1;
    double4 *sA = reinterpret_cast<double4 *>(smem);
    double4 *sB = sA + kJC;
    double *sX = reinterpret_cast<double *>(sB + kJC);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, kq = lane >> 4, mq = lane & 3;
    const int64_t ibase = itile * 64 + wave * 16;
    const int col0 = grp * NC;
    const int64_t jbeg = (int64_t)split * jlen;
    const int64_t jend = min(npad, jbeg + jlen);
    constexpr int kJJUnroll = SCR ? 1 : 2;   // screened: fewer live registers
    const double4 a0 = P0[ibase + m], a1 = P1[ibase + m];
    constexpr int NB = NQ == 4 ? NCB : LB, NT = NQ == 4 ? 0 : NQ;   // blocks, quads
    v4d accp[NB > 0 ? NB : 1], accq[NB > 0 ? NB : 1];
    double tp[NT > 0 ? NT : 1], tq[NT > 0 ? NT : 1];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
        accp[cb] = (v4d){0.0, 0.0, 0.0, 0.0};
        accq[cb] = (v4d){0.0, 0.0, 0.0, 0.0};
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) tp[t] = tq[t] = 0.0;
    for (int64_t j0 = jbeg; j0 < jend; j0 += kJC) {
        __syncthreads();
        if (tid < kJC) {
            sA[tid] = P0[j0 + tid];
            sB[tid] = P1[j0 + tid];
        }
        stage_rows<2 * kJC, NC>(X + j0 * 2 * Pp, Pp, col0, sX);
        __syncthreads();
        // the chunk that holds this wave's outer points leaves out the self pair
        const bool diag = ibase < j0 + kJC && ibase + 16 > j0;
        const int dself = diag ? (int)(ibase - j0) + m - kq : -1;
#pragma unroll kJJUnroll
        for (int jj = 0; jj < kJC; jj += 4) {
            const int jl = jj + kq;
            double kpp, kpq, kqp, kqq;
            pair_K64(a0, a1, sA[jl], sB[jl].x, sB[jl].z, kpp, kpq, kqp, kqq);
            kpp = jj == dself ? 0.0 : kpp;
            const double *xr = sX + (jl * 2) * NC;
            const uint32_t mw = SCR ? mask[((j0 + jj) >> 4) * ((Pp >> 4) / NCB) + grp] : 0u;
#pragma unroll
            for (int cb = 0; cb < NB; ++cb) {
                if (SCR && !((mw >> cb) & 1u)) continue;
                const double xp = xr[cb * 16 + m], xq = xr[NC + cb * 16 + m];
                accp[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(kpp, xp, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(kqp, xp, accq[cb], 0, 0, 0);
                accp[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(kpq, xq, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(kqq, xq, accq[cb], 0, 0, 0);
            }
            if (SCR && NT && !((mw >> LB) & 1u)) continue;
            double xp[NT > 0 ? NT : 1], xq[NT > 0 ? NT : 1];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                xp[t] = xr[LB * 16 + 4 * t + mq];
                xq[t] = xr[NC + LB * 16 + 4 * t + mq];
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                tp[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(kpp, xp[t], tp[t], 0, 0, 0);
                tq[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(kqp, xp[t], tq[t], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                tp[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(kpq, xq[t], tp[t], 0, 0, 0);
                tq[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(kqq, xq[t], tq[t], 0, 0, 0);
            }
        }
    }
    // D layouts (measured on gfx950): 16x16x4, item r of lane l holds row
    // 4 r + l/16, column l%16; 4x4x4, lane l holds row 4 ((l/4)%4) + l/16, column l%4
    double *Yb = Yout + (int64_t)split * npad * 2 * Pp;
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t row = ibase + 4 * r + kq;
            Yb[(row * 2 + 0) * Pp + col0 + cb * 16 + m] = accp[cb][r];
            Yb[(row * 2 + 1) * Pp + col0 + cb * 16 + m] = accq[cb][r];
        }
    const int64_t rowq = ibase + 4 * ((lane >> 2) & 3) + kq;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        Yb[(rowq * 2 + 0) * Pp + col0 + LB * 16 + 4 * t + mq] = tp[t];
        Yb[(rowq * 2 + 1) * Pp + col0 + LB * 16 + 4 * t + mq] = tq[t];
    }
}

// ---------------------------------------------------------------------------
// FP32 MFMA
// ---------------------------------------------------------------------------
// The four kernel-derivative values of pair (i, j), divided by -3/2 (see the
// file header); a = (x, y, z, omega), b = (kappa, ., c, .) of each point.
__device__ __forceinline__ void pair_K(const float4 a0, const float4 a1, const float4 b0,
                                       const float4 b1, float &kpp, float &kpq, float &kqp,
                                       float &kqq) {
    const float dx = a0.x - b0.x, dy = a0.y - b0.y, dz = a0.z - b0.z;
    const float R2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
    const float gg = __builtin_fmaf(a0.w, R2, a1.x);
    const float gp = __builtin_fmaf(b0.w, R2, b1.x);
    const float s = gg + gp, t = gg * gp;
    const float r = rcp32(t * s);
    const float sr = s * r;                           // 1 / (g g')
    const float is = t * r;                           // 1 / s
    const float A = r * __builtin_fmaf(gp, sr, is);   // r (1/g + 1/s)
    const float Ap = r * __builtin_fmaf(gg, sr, is);  // r (1/g' + 1/s)
    const float Q = (r + r) * __builtin_fmaf(is, is, sr);
    const float ci = a1.z, cj = b1.z;
    const float t1 = __builtin_fmaf(ci, Q, -Ap);
    const float t2 = __builtin_fmaf(cj, Q, -A);
    kpp = __builtin_fmaf(cj, t1, __builtin_fmaf(-ci, A, r));
    kpq = R2 * t1;
    kqp = R2 * t2;
    kqq = (R2 * R2) * Q;
}

template <int NCB>
constexpr int smem_f32() { return 2 * kJC * (int)sizeof(float4) + kJC * 2 * NCB * 16 * (int)sizeof(float); }

template <int NCB, bool SCR = false>
__device__ __forceinline__ void tile_f32(int64_t npad, int64_t jlen, int32_t Pp,
                                         const float4 *__restrict__ P0,
                                         const float4 *__restrict__ P1,
                                         const float *__restrict__ X, double *__restrict__ Yout,
                                         int64_t itile, int grp, int split, char *smem,
                                         const uint32_t *__restrict__ mask = nullptr) {
    constexpr int NC = NCB * 16;
    static_assert(kFp32Run % kJC == 0, "FP32 runs end on chunk boundaries");
    float4 *sA = reinterpret_cast<float4 *>(smem);
    float4 *sB = sA + kJC;
    float *sX = reinterpret_cast<float *>(sB + kJC);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, kq = lane >> 4;
    const int64_t ibase = itile * 64 + wave * 16;
    const int col0 = grp * NC;
    const int64_t jbeg = (int64_t)split * jlen;
    const int64_t jend = min(npad, jbeg + jlen);
    constexpr int kJJUnroll = SCR ? 1 : 2;   // screened: fewer live registers
    const float4 a0 = P0[ibase + m], a1 = P1[ibase + m];
    v4f accp[NCB], accq[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        accp[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
        accq[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
    }
    // D layout of the FP32 MFMAs (measured on gfx950): item r of lane l holds
    // row 4 (l/16) + r, column l%16.  The FP32 sums of each run of kFp32Run
    // points go into this split's FP64 partials.
    const PartialRows Yb(Yout, split, npad * 2 * Pp, partials_f32(npad, jlen));
    bool first = true;
    auto flush = [&]() {
        // one base address formed here (the empty asm keeps it from being
        // hoisted out of the loop)
        int64_t off = (ibase + 4 * kq) * 2 * Pp + col0 + m;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float vp[NCB], vq[NCB];
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                vp[cb] = accp[cb][r];
                vq[cb] = accq[cb][r];
            }
            add_row<NCB>(Yb, off + (2 * r + 0) * (int64_t)Pp, vp, first);
            add_row<NCB>(Yb, off + (2 * r + 1) * (int64_t)Pp, vq, first);
        }
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            accp[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
            accq[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
        }
        first = false;
    };
    for (int64_t j0 = jbeg; j0 < jend; j0 += kJC) {
        __syncthreads();
        if (tid < kJC) {
            sA[tid] = P0[j0 + tid];
            sB[tid] = P1[j0 + tid];
        }
        stage_rows<2 * kJC, NC>(X + j0 * 2 * Pp, Pp, col0, sX);
        __syncthreads();
        // the chunk that holds this wave's outer points leaves out the self pair
        const bool diag = ibase < j0 + kJC && ibase + 16 > j0;
        const int dself = diag ? (int)(ibase - j0) + m - kq : -1;
#pragma unroll kJJUnroll
        for (int jj = 0; jj < kJC; jj += 4) {
            const int jl = jj + kq;
            float kpp, kpq, kqp, kqq;
            pair_K(a0, a1, sA[jl], sB[jl], kpp, kpq, kqp, kqq);
            kpp = jj == dself ? 0.f : kpp;
            const float *xr = sX + (jl * 2) * NC + m;
            const uint32_t mw = SCR ? mask[((j0 + jj) >> 4) * ((Pp >> 4) / NCB) + grp] : 0u;
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                if (SCR && !((mw >> cb) & 1u)) continue;
                const float xp = xr[cb * 16];
                accp[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kpp, xp, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kqp, xp, accq[cb], 0, 0, 0);
            }
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                if (SCR && !((mw >> cb) & 1u)) continue;
                const float xq = xr[NC + cb * 16];
                accp[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kpq, xq, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kqq, xq, accq[cb], 0, 0, 0);
            }
        }
        if ((j0 + kJC - jbeg) % kFp32Run == 0 && j0 + kJC < jend) flush();
    }
    flush();
}

// ---------------------------------------------------------------------------
// split-BF16 MFMA
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct Aops {          // A operands of one 16 x 16 pair block (per lane: 4 pairs)
    bf16x8 ph, pl, qh, ql;
};

// Split two FP32 values into packed bf16 hi (round to nearest even) and lo
// (the rounded remainder): returns the packed words (v0 in the low half).
// The low half of hi is widened with a byte permute, which keeps the compiler
// from converting v0 a second time.  Contraction is off so that v - hi is a
// plain subtraction in every kernel that inlines this (a product fused into
// it in one kernel and not in another would break bitwise agreement between
// the single-molecule and batched contractions).
__device__ __forceinline__ void split2(float v0, float v1, uint32_t &hi, uint32_t &lo) {
#pragma clang fp contract(off)
    const bf16x2 h = {(__bf16)v0, (__bf16)v1};
    hi = __builtin_bit_cast(uint32_t, h);
    const float h0 = __uint_as_float(__builtin_amdgcn_perm(0u, hi, 0x01000c0cu));   // hi << 16
    const float h1 = __uint_as_float(hi & 0xffff0000u);
    const bf16x2 l = {(__bf16)(v0 - h0), (__bf16)(v1 - h1)};
    lo = __builtin_bit_cast(uint32_t, l);
}

// One pair of a block in three steps of about equal VALU work, so that a
// caller can place each step between MFMAs: (0) the geometry and its
// reciprocal, (1) the four kernel values of pair_K, (2) their hi/lo split.
// The arithmetic is that of pair_K and split2, operation for operation.
struct PairSteps {
    float R2, gg, gp, s, t, r, kpp, kpq, kqp, kqq;
    __device__ __forceinline__ void geometry(const float4 a0, const float4 a1, const float4 b0,
                                             const float2 b1) {
        const float dx = a0.x - b0.x, dy = a0.y - b0.y, dz = a0.z - b0.z;
        R2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
        gg = __builtin_fmaf(a0.w, R2, a1.x);
        gp = __builtin_fmaf(b0.w, R2, b1.x);
        s = gg + gp;
        t = gg * gp;
        r = rcp32(t * s);
    }
    __device__ __forceinline__ void values(float ci, float cj) {
        const float sr = s * r, is = t * r;
        const float A = r * __builtin_fmaf(gp, sr, is);
        const float Ap = r * __builtin_fmaf(gg, sr, is);
        const float Q = (r + r) * __builtin_fmaf(is, is, sr);
        const float t1 = __builtin_fmaf(ci, Q, -Ap);
        const float t2 = __builtin_fmaf(cj, Q, -A);
        kpp = __builtin_fmaf(cj, t1, __builtin_fmaf(-ci, A, r));
        kpq = R2 * t1;
        kqp = R2 * t2;
        kqq = (R2 * R2) * Q;
    }
};

// Software pipeline per wave, in stages of 32 j points (two 16-point
// blocks) and chunks of one column block (six MFMAs per chunk):
//  * X of a stage (hi and lo, all columns of the group) and the points whose
//    pairs are formed during it are double-buffered in LDS and go there
//    straight from global memory, issued one stage ahead;
//  * a chunk's B operands are read from LDS kAhead chunks before their MFMAs,
//    so that no LDS latency is exposed;
//  * the next block's A operands are formed meanwhile, a twelfth of the
//    block's pair arithmetic after each twelfth of its chunks: one wave's
//    VALU work issues under its own and the other waves' MFMAs;
//  * the barrier that closes a stage stands kAhead chunks before the stage's
//    last MFMAs: every read of the stage's buffer has then been issued, and
//    the chunks that follow cover the first reads of the next one.
// What bounds it (20-water grid, twelve blocks): 72 MFMAs of 16 cycles and 172
// VALU instructions per wave and 16-point block.  The form with the waits
// exposed took 107 M cycles per XCD at 2.05 GHz (matrix cores busy 60 %), this
// one 87 M at 1.88 GHz (73 %): the clock falls as the cycles do, by the card's
// power limit, so only less work would gain more.  Contraction about 50.5 -> 46.3
// ms; at four blocks (hexamer), bound by
// VALU issue, 1.45 -> 1.30 ms.
template <int NCB>
constexpr int smem_bf16x3() { return (4 * NCB + 2) * 64 * (int)sizeof(bf16x8); }

template <int NCB, bool SCR = false, int WAVES = 4>
__device__ __forceinline__ void tile_bf16x3(int64_t npad, int64_t jlen, int32_t Pp,
                                            const float4 *__restrict__ P0,
                                            const float4 *__restrict__ P1,
                                            const bf16x8 *__restrict__ Xhi,
                                            const bf16x8 *__restrict__ Xlo,
                                            double *__restrict__ Yout, int64_t itile, int grp,
                                            int split, char *smem, char *smem2,
                                            const uint32_t *__restrict__ mask = nullptr) {
    constexpr int NC = NCB * 16;
    static_assert(kFp32Run % 64 == 0, "FP32 runs end on stage pairs");
    constexpr int UNITS = NCB * 64;                     // 8-bf16 units per block and array
    constexpr int NT = 64 * WAVES;                      // threads of the workgroup
    constexpr int PER = (2 * UNITS + NT - 1) / NT;      // units per thread, stage and array
    constexpr int kAhead = NCB == 1 ? 1 : 2;
    // a stage buffer: X hi then lo of two blocks, [block][cb][lane], and 32
    // points (64 units of P0, then 64 of P1); the two buffers are distinct LDS arrays, so that
    // the compiler sees that a stage's reads and the loads into the other
    // buffer never alias
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int64_t ibase = itile * (16 * WAVES) + wave * 16;
    const int col0 = grp * NC;
    const int64_t jbeg = (int64_t)split * jlen;
    const int64_t jend = min(npad, jbeg + jlen);
    const float4 a0 = P0[ibase + m], a1 = P1[ibase + m];
    v4f accp[NCB], accq[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        accp[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
        accq[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
    }
    // the FP32 sums of each run of kFp32Run points go into this split's FP64
    // partials (D layout: item r of lane (m, g) is row 4 g + r, column m)
    const PartialRows Yb(Yout, split, npad * 2 * Pp, partials_f32(npad, jlen));
    bool first = true;
    auto flush = [&]() {
        // one base address formed here (the empty asm keeps it from being
        // hoisted out of the loop: 2 x 4 x NCB addresses would stay live)
        int64_t off = (ibase + 4 * g) * 2 * Pp + col0 + m;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float vp[NCB], vq[NCB];
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                vp[cb] = accp[cb][r];
                vq[cb] = accq[cb][r];
            }
            add_row<NCB>(Yb, off + (2 * r + 0) * (int64_t)Pp, vp, first);
            add_row<NCB>(Yb, off + (2 * r + 1) * (int64_t)Pp, vq, first);
        }
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            accp[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
            accq[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
        }
        first = false;
    };
    // A stage's 32 points go into a buffer straight from global memory
    // (buffer_load_dwordx4 ... lds: lane l of a wave writes the 16 bytes at
    // the wave's LDS base + 16 l, so unit e = tid + NT k lands at unit e), in
    // PER pieces of hi and lo and one of points, issued one piece per chunk
    // after the barrier that frees the buffer: issued together they kept the
    // waves from their MFMAs for some 600 cycles a stage.  The source of piece
    // k is the stage's base (uniform, in the descriptor) plus a 32-bit offset
    // fixed over the stages, and the LDS base is uniform, so a piece costs no
    // vector address arithmetic.  The buffer form matters: with a
    // global_load_lds pending the compiler makes every wait on an LDS read a
    // full one (it takes the instruction for a flat access).
    // (first unit of this wave's piece k, uniform; where the waves outnumber
    // the units left, some bring units that another wave brings too)
    auto first_unit = [&](int k) { return (wave * 64 + NT * k) % (2 * UNITS); };
    uint32_t xoff[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = first_unit(k) + lane;
        const int sub = e >= UNITS;
        xoff[k] = (uint32_t)(sub * Pp * 4 + (e - sub * UNITS)) * (uint32_t)sizeof(bf16x8);
    }
    auto to_lds = [](const void *base, uint32_t off, bf16x8 *dst) { load16_lds(base, off, 0, dst); };
    // piece k of the stage at j
    auto load_piece = [&](int k, int64_t j, bf16x8 *buf) {
        if (k == PER) {
            // the points whose pairs are formed during the stage, j + 16 ..
            // j + 47 (clamped: past the grid they are formed but never used):
            // even waves bring P0, odd ones P1, the upper lanes the same again
            const uint32_t left = (uint32_t)min(npad - 1 - j, (int64_t)64);
            to_lds((wave & 1 ? P1 : P0) + j, min(16u + (lane & 31), left) * (uint32_t)sizeof(float4),
                   buf + 4 * UNITS + 64 * (wave & 1));
            return;
        }
        const int e0 = first_unit(k);
        const int64_t base = (j / 16) * Pp * 4 + col0 * 4;
        to_lds(Xhi + base, xoff[k], buf + e0);
        to_lds(Xlo + base, xoff[k], buf + 2 * UNITS + e0);
    };
    // points of this lane's four pairs of a block: (x, y, z, omega), (kappa, c)
    float4 n0[4];
    float2 n1[4];
    auto read_points = [&](const bf16x8 *buf, int sub) {
        const float4 *q = reinterpret_cast<const float4 *>(buf + 4 * UNITS) + 16 * sub + 4 * g;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            n0[jj] = q[jj];
            n1[jj] = make_float2(q[64 + jj].x, q[64 + jj].z);
        }
    };
    // the diagonal block leaves out the self pair: it is pair m mod 4 of lane
    // (m, g = m/4), whose K_pp is cleared (K_pq, K_qp, K_qq vanish there, R = 0);
    // a lane mask selected by a uniform test, as a branch would split the block
    bool self[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) self[jj] = m == 4 * g + jj;
    PairSteps ps;
    uint32_t ph[4], pl[4], qh[4], ql[4];
    // (the empty asm statements keep each step's instructions in its chunk)
    auto step = [&](int k, bool diag) {                 // k = 3 pair + step
        const int jj = k / 3;
        if (k % 3 == 0) {
            ps.geometry(a0, a1, n0[jj], n1[jj]);
            asm volatile("" : "+v"(ps.R2), "+v"(ps.gg), "+v"(ps.gp), "+v"(ps.s), "+v"(ps.t), "+v"(ps.r));
        } else if (k % 3 == 1) {
            ps.values(a1.z, n1[jj].y);
            ps.kpp = diag && self[jj] ? 0.f : ps.kpp;
            asm volatile("" : "+v"(ps.kpp), "+v"(ps.kpq), "+v"(ps.kqp), "+v"(ps.kqq));
        } else {
            split2(ps.kpp, ps.kpq, ph[jj], pl[jj]);
            split2(ps.kqp, ps.kqq, qh[jj], ql[jj]);
            asm volatile("" : "+v"(ph[jj]), "+v"(pl[jj]), "+v"(qh[jj]), "+v"(ql[jj]));
        }
    };
    auto formed = [&]() {
        Aops A;
        A.ph = __builtin_bit_cast(bf16x8, (uint4){ph[0], ph[1], ph[2], ph[3]});
        A.pl = __builtin_bit_cast(bf16x8, (uint4){pl[0], pl[1], pl[2], pl[3]});
        A.qh = __builtin_bit_cast(bf16x8, (uint4){qh[0], qh[1], qh[2], qh[3]});
        A.ql = __builtin_bit_cast(bf16x8, (uint4){ql[0], ql[1], ql[2], ql[3]});
        return A;
    };
    // B operands (hi, lo) of the chunks in flight
    bf16x8 Bh[kAhead + 1], Bl[kAhead + 1];
    // one stage: A holds the operands of its first block on entry and those
    // of the next stage's first block on return
    auto stage = [&](int64_t j0, bf16x8 *cur, bf16x8 *nxt, Aops &A) {
        // screened: a column block whose mask bit is clear skips its MFMAs
        uint32_t mw[2] = {~0u, ~0u};
        if constexpr (SCR)
#pragma unroll
            for (int sub = 0; sub < 2; ++sub)
                mw[sub] = mask[((j0 >> 4) + sub) * ((Pp >> 4) / NCB) + grp];
#pragma unroll
        for (int c = 0; c < 2 * NCB; ++c) {
            const int sub = c / NCB, cb = c - sub * NCB;
            if (c == 2 * NCB - kAhead) {
                __builtin_amdgcn_s_waitcnt(0);   // this wave's LDS loads and reads are done
                __syncthreads();
            }
            // pieces of the next stage (past the last one: that one again)
#pragma unroll
            for (int k = 0; k <= PER; ++k)
                if (c == (k < 2 * NCB - kAhead ? k : 2 * NCB - kAhead - 1))
                    load_piece(k, min(j0 + 32, jend - 32), nxt);
            // (issue priority falls along the stage, so that of the waves of a
            // SIMD the one behind goes first and they reach the barrier together)
            if (WAVES == 8 && (4 * c) % (2 * NCB) < 4) {
                const int q = 4 * c / (2 * NCB);
                if (q == 0) __builtin_amdgcn_s_setprio(3);
                if (q == 1) __builtin_amdgcn_s_setprio(2);
                if (q == 2) __builtin_amdgcn_s_setprio(1);
                if (q == 3) __builtin_amdgcn_s_setprio(0);
            }
            __builtin_amdgcn_sched_barrier(0);
            {
                const int pc = c + kAhead, q = pc % (2 * NCB);
                const bf16x8 *b = (pc < 2 * NCB ? cur : nxt) + q * 64 + lane;
                Bh[kAhead] = b[0];
                Bl[kAhead] = b[2 * UNITS];
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!SCR || ((mw[sub] >> cb) & 1u)) {
                const bf16x8 bh = Bh[0], bl = Bl[0];
                accp[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.ph, bh, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.qh, bh, accq[cb], 0, 0, 0);
                accp[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.pl, bh, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.ql, bh, accq[cb], 0, 0, 0);
                accp[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.ph, bl, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.qh, bl, accq[cb], 0, 0, 0);
            }
#pragma unroll
            for (int k = 0; k < 12; ++k)
                if (k * NCB / 12 == cb) step(k, j0 + 16 * sub + 16 == ibase);
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                Bh[k] = Bh[k + 1];
                Bl[k] = Bl[k + 1];
            }
            __builtin_amdgcn_sched_barrier(0);
            if (cb == NCB - 1) {
                A = formed();
                read_points(sub ? nxt : cur, sub ^ 1);
            }
        }
    };
    bf16x8 *buf0 = reinterpret_cast<bf16x8 *>(smem), *buf1 = reinterpret_cast<bf16x8 *>(smem2);
    Aops A;
#pragma unroll
    for (int k = 0; k <= PER; ++k) load_piece(k, jbeg, buf0);
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        n0[jj] = P0[jbeg + 4 * g + jj];
        n1[jj] = make_float2(P1[jbeg + 4 * g + jj].x, P1[jbeg + 4 * g + jj].z);
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) step(k, jbeg == ibase);
    A = formed();
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
        Bh[k] = buf0[k * 64 + lane];
        Bl[k] = buf0[2 * UNITS + k * 64 + lane];
    }
    read_points(buf0, 0);
    // a split holds a whole number of 32-point stages (jbeg and jlen are
    // multiples of 32, npad of 256)
    int64_t j0 = jbeg;
    for (; j0 + 64 <= jend; j0 += 64) {
        stage(j0, buf0, buf1, A);
        stage(j0 + 32, buf1, buf0, A);
        if ((j0 + 64 - jbeg) % kFp32Run == 0 && j0 + 64 < jend) flush();
    }
    if (j0 < jend) stage(j0, buf0, buf1, A);
    flush();
}

// One workgroup per (i tile, column group, j split): blockIdx = (tile, group, split).
// SCR: skip the (16-point, 16-column) blocks that the screening mask marks
// inactive (the MFMA work only; the kernel tile is still formed).
// FP64: the last group's last block holds NQ quads of columns (4: all 16).
template <int NCB, bool SCR, int NQ>
__global__ __launch_bounds__(256, 2) void k_contract_f64(int64_t npad, int64_t jlen, int32_t Pp,
                                                         const double4 *__restrict__ P0,
                                                         const double4 *__restrict__ P1,
                                                         const double *__restrict__ X,
                                                         double *__restrict__ Yout,
                                                         const uint32_t *__restrict__ mask) {
    __shared__ __attribute__((aligned(16))) char smem[smem_f64<NCB>()];
    if (NQ == 4 || blockIdx.y + 1 == gridDim.y)
        tile_f64<NCB, SCR, NQ>(npad, jlen, Pp, P0, P1, X, Yout, blockIdx.x, blockIdx.y, blockIdx.z,
                               smem, mask);
    else
        tile_f64<NCB, SCR>(npad, jlen, Pp, P0, P1, X, Yout, blockIdx.x, blockIdx.y, blockIdx.z,
                           smem, mask);
}

template <int NCB, bool SCR>
__global__ __launch_bounds__(256, 2) void k_contract_f32(int64_t npad, int64_t jlen, int32_t Pp,
                                                         const float4 *__restrict__ P0,
                                                         const float4 *__restrict__ P1,
                                                         const float *__restrict__ X,
                                                         double *__restrict__ Yout,
                                                         const uint32_t *__restrict__ mask) {
    __shared__ __attribute__((aligned(16))) char smem[smem_f32<NCB>()];
    tile_f32<NCB, SCR>(npad, jlen, Pp, P0, P1, X, Yout, blockIdx.x, blockIdx.y, blockIdx.z, smem,
                       mask);
}

// Waves (16 outer points each) of the split-BF16 kernels, by column blocks:
// from eight blocks on, eight waves share each staged X (two per SIMD; their
// accumulators leave room for no more), below four waves, whose workgroups
// then fill the SIMDs with three waves each or more, two at seven blocks (eight
// waves at four column blocks: 1.46 against 1.29-1.30 ms on the hexamer).
template <int NCB>
constexpr int bf16_waves() { return NCB >= kWideMinNcb ? 8 : 4; }

template <int NCB, bool SCR>
__global__ __launch_bounds__(64 * bf16_waves<NCB>(), 8 / bf16_waves<NCB>()) void k_contract_bf16x3(int64_t npad, int64_t jlen, int32_t Pp,
                                                            const float4 *__restrict__ P0,
                                                            const float4 *__restrict__ P1,
                                                            const bf16x8 *__restrict__ Xhi,
                                                            const bf16x8 *__restrict__ Xlo,
                                                            double *__restrict__ Yout,
                                                            const uint32_t *__restrict__ mask) {
    __shared__ __attribute__((aligned(16))) char smem[smem_bf16x3<NCB>()];
    __shared__ __attribute__((aligned(16))) char smem2[smem_bf16x3<NCB>()];   // the other stage
    tile_bf16x3<NCB, SCR, bf16_waves<NCB>()>(npad, jlen, Pp, P0, P1, Xhi, Xlo, Yout,
                                             blockIdx.x, blockIdx.y, blockIdx.z, smem, smem2,
                                             mask);
}

template <int NCB, bool SCR>
hipError_t run_mode(vv10_plan *p, const Workspace &ws) {
    dim3 grid((unsigned)(p->npad / 64), (unsigned)ws.ngroups, (unsigned)ws.jsplit);
    const uint32_t *mask = SCR ? ws.mask : nullptr;
    if (p->prec == VV10_FP64) {
        if constexpr (NCB <= 8) {
            // quads of columns in the last block (a block past the columns,
            // which uneven groups leave, takes the 16-column form on zeros)
            const int left = ws.P - (ws.Pp - 16);
            const int nq = left > 0 ? (left + 3) / 4 : 4;
            auto go = [&](auto q) {
                k_contract_f64<NCB, SCR, decltype(q)::value><<<grid, 256, 0, p->stream>>>(
                    p->npad, ws.jlen, ws.Pp, p->P0, p->P1, static_cast<const double *>(ws.X),
                    static_cast<double *>(ws.Ypart), mask);
            };
            if (nq == 1) go(std::integral_constant<int, 1>{});
            else if (nq == 2) go(std::integral_constant<int, 2>{});
            else if (nq == 3) go(std::integral_constant<int, 3>{});
            else go(std::integral_constant<int, 4>{});
        } else {
            return hipErrorInvalidValue;
        }
    } else if (p->prec == VV10_MIXED_FP32) {
        k_contract_f32<NCB, SCR><<<grid, 256, 0, p->stream>>>(
            p->npad, ws.jlen, ws.Pp, p->P0f, p->P1f, static_cast<const float *>(ws.X),
            static_cast<double *>(ws.Ypart), mask);
    } else {
        const bf16x8 *xh = static_cast<const bf16x8 *>(ws.X);
        const bf16x8 *xl = xh + (size_t)p->npad * ws.Pp * 2 / 8;
        constexpr int W = bf16_waves<NCB>();
        dim3 gridb((unsigned)(p->npad / (16 * W)), (unsigned)ws.ngroups, (unsigned)ws.jsplit);
        k_contract_bf16x3<NCB, SCR><<<gridb, 64 * W, 0, p->stream>>>(
            p->npad, ws.jlen, ws.Pp, p->P0f, p->P1f, xh, xl, static_cast<double *>(ws.Ypart), mask);
    }
    return hipGetLastError();
}

template <int NCB>
hipError_t run(vv10_plan *p, const Workspace &ws, bool screen) {
    return screen ? run_mode<NCB, true>(p, ws) : run_mode<NCB, false>(p, ws);
}

template <int NCB>
int occupancy_f64() {
    int nb = 0;
    if constexpr (NCB <= 8) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_contract_f64<NCB, false, 4>, 256, 0) !=
            hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
    }
    return nb;
}

template <typename F>
auto dispatch_ncb(int ncb, F &&f) -> decltype(f(std::integral_constant<int, 1>{})) {
    switch (ncb) {
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 7: return f(std::integral_constant<int, 7>{});
        case 8: return f(std::integral_constant<int, 8>{});
        case 9: return f(std::integral_constant<int, 9>{});
        case 10: return f(std::integral_constant<int, 10>{});
        case 11: return f(std::integral_constant<int, 11>{});
        case 12: return f(std::integral_constant<int, 12>{});
        default: return decltype(f(std::integral_constant<int, 1>{})){};
    }
}

// ---------------------------------------------------------------------------
// Persistent batched kernels: a fixed grid of workgroups pulls work items
// from an integer counter, one list and counter per kernel, each list
// largest first.  A contraction item is (molecule, i tile, column group,
// j split); a grid item is one grid-pass tile of one molecule for one atom
// group (the grid-position intermediates and the pair integrals).  Every
// item writes its own output slab, so the results do not depend on which
// workgroup ran which item.
// ---------------------------------------------------------------------------
// Two forms each: one for every column count that the list may hold, and one for
// lists of at most kNarrowNcb column blocks (clusters of up to eight waters),
// whose smaller register allocation (160, 104 and 162 VGPRs for 250, 198 and
// 189) leaves room for one or two waves more per SIMD.  Two dozen clusters of
// 1 to 6 waters with 600 points an atom, per run: FP32 7.70 -> 6.70 ms,
// split-BF16 4.15 -> 4.08 (the clock falls with the waits); a dozen in FP64 6.66
// -> 6.13 (5.75 with the column quads).  With a limit of four, 16 clusters of up to eight waters took FP32
// 6.50 ms against 5.78 and split-BF16 3.27 against 3.22; with seven, 14 clusters of
// up to nine waters took FP32 5.00 ms against 5.39, but FP64 10.5 against 8.8 and
// split-BF16 3.36 against 2.79 (accumulators moved to AGPRs, one wave per SIMD).
constexpr int kNarrowNcb = 5;
template <int PREC>
struct PersistentTraits;
template <>
struct PersistentTraits<VV10_FP64> {
    static constexpr int kMaxNcb = 8;
    template <int MAX>
    static constexpr int smem() { return smem_f64<MAX>(); }
    static constexpr int kWaves = 4;
    static constexpr int kNarrowPerEu = 3;
};
template <>
struct PersistentTraits<VV10_MIXED_FP32> {
    static constexpr int kMaxNcb = 12;
    template <int MAX>
    static constexpr int smem() { return smem_f32<MAX>(); }
    static constexpr int kWaves = 4;
    static constexpr int kNarrowPerEu = 4;
};
template <>
struct PersistentTraits<VV10_MIXED_BF16X3> {
    // four waves: the eight-wave form of the standalone kernel (32-point
    // stages, X straight into two LDS buffers) spilled 32 registers here
    // when every column count shared one register allocation and was slower
    // on the 64-cluster batch (2.95 s per launch against 2.86 s); molecules
    // with kWideMinNcb or more blocks per group run it in a kernel of their
    // own (k_contract_persistent_wide), so this one serves the narrower
    // counts only, whose smaller register allocation leaves room for more
    // waves per SIMD
    static constexpr int kMaxNcb = kWideMinNcb - 1;
    static constexpr int kWaves = 4;
    template <int MAX>
    static constexpr int smem() { return smem_bf16x3<MAX>(); }
    static constexpr int kNarrowPerEu = 3;
};

template <int PREC, int NCB>
__device__ __forceinline__ void run_item(const BatchMol &d, const BatchItem &it, char *smem,
                                         char *smem2) {
    if constexpr (PREC == VV10_FP64) {
        // quads of columns in the last group's last block, as the standalone
        // kernel (FP64 batch of a dozen clusters of 1 to 6 waters 6.15 -> 5.75 ms)
        const int left = 3 * d.n_atom - (d.Pp - 16);
        const bool last = (it.grp + 1) * 16 * NCB == d.Pp && left > 0;
        const int nq = last ? (left + 3) / 4 : 4;
        auto go = [&](auto q) __attribute__((always_inline)) {
            tile_f64<NCB, false, decltype(q)::value>(
                d.npad, d.jlen, d.Pp, global_as<double4>(d.P0), global_as<double4>(d.P1),
                global_as<double>(d.X), global_ptr(static_cast<double *>(d.Ypart)), it.itile, it.grp, it.split, smem);
        };
        if (nq == 1) go(std::integral_constant<int, 1>{});
        else if (nq == 2) go(std::integral_constant<int, 2>{});
        else if (nq == 3) go(std::integral_constant<int, 3>{});
        else go(std::integral_constant<int, 4>{});
    } else if constexpr (PREC == VV10_MIXED_FP32) {
        tile_f32<NCB>(d.npad, d.jlen, d.Pp, global_as<float4>(d.P0), global_as<float4>(d.P1),
                      global_as<float>(d.X), global_ptr(static_cast<double *>(d.Ypart)), it.itile, it.grp, it.split, smem);
    } else {
        const bf16x8 *xh = global_as<bf16x8>(d.X);
        tile_bf16x3<NCB, false, PersistentTraits<PREC>::kWaves>(
            d.npad, d.jlen, d.Pp, global_as<float4>(d.P0), global_as<float4>(d.P1), xh,
            xh + d.npad * d.Pp * 2 / 8, global_ptr(static_cast<double *>(d.Ypart)), it.itile, it.grp, it.split, smem, smem2);
    }
}

// Grid items of a batch: a workgroup pulls one grid tile of one molecule and
// atom group at a time (with the pair integrals, as the Hessian
// call forms them).  A kernel of its own keeps the grid pass's register
// allocation (and the standalone grid kernel's waves per SIMD), where the
// contraction kernels' allocations would hold it to two waves per SIMD.
// The pointers of a molecule's record are marked as global ones here and in the
// contraction's kernels: taken for flat ones, their accesses needed vector
// address registers, and this kernel spilled 9 or 10 (now none).  Eight clusters
// of 2 to 30 waters, 1500 points an atom, split-BF16: contractions 51.3 + 194.9 ->
// 50.9 + 193.3 ms, grid items 58.4 and 58.6; six of 3 to 30 with 1000 points in
// FP64, contraction 537 -> 528 ms.
template <int PREC>
__global__ __launch_bounds__(64 * kGridWaves) __attribute__((amdgpu_waves_per_eu(PREC == VV10_FP64 ? 3 : 4))) void k_grid_persistent(
    const BatchMol *__restrict__ mols, const BatchItem *__restrict__ items, int32_t n_items,
    int32_t *__restrict__ counter) {
    using T = std::conditional_t<PREC == VV10_FP64, double, float>;
    using T4 = std::conditional_t<PREC == VV10_FP64, double4, float4>;
    __shared__ GridLds<T4> lds;
    __shared__ int32_t next;
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(counter, 1);
        __syncthreads();
        const int32_t k = __builtin_amdgcn_readfirstlane(next);   // uniform: item data in SGPRs
        __syncthreads();
        if (k >= n_items) break;          // every workgroup leaves once the list is drained
        const BatchItem it = items[k];
        const BatchMol d = mols[it.mol];

        // grid_unit orders its LDS writes after the previous reads itself
        grid_unit<T, T4, true, false>(d.n_atom, d.Pp, d.bgroups, d.npad, global_ptr(d.seg),
                                      global_ptr(d.tile_i0), global_ptr(d.tile_n),
                                      global_ptr(d.tile_atom), global_as<T4>(d.P0),
                                      global_as<T4>(d.P1), global_ptr(d.Pd), global_ptr(d.Z),
                                      nullptr, global_ptr(d.Dpart), global_ptr(d.Igrp), it.itile,
                                      it.grp, d.whole, lds);
    }
}

template <int PREC, int MAX>
__global__ __launch_bounds__(64 * PersistentTraits<PREC>::kWaves,
                             MAX <= kNarrowNcb ? PersistentTraits<PREC>::kNarrowPerEu : 2) void k_contract_persistent(
    const BatchMol *__restrict__ mols, const BatchItem *__restrict__ items, int32_t n_items,
    int32_t *__restrict__ counter) {
    constexpr int kSmem = PersistentTraits<PREC>::template smem<MAX>();
    __shared__ __attribute__((aligned(16))) char smem[kSmem];
    // the second stage buffer of the split-BF16 form (a one-byte dummy otherwise)
    __shared__ __attribute__((aligned(16))) char smem2[PREC == VV10_MIXED_BF16X3 ? kSmem : 1];
    __shared__ int32_t next;
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(counter, 1);
        __syncthreads();
        const int32_t k = __builtin_amdgcn_readfirstlane(next);   // uniform: item data in SGPRs
        __syncthreads();
        if (k >= n_items) break;          // every workgroup leaves once the list is drained
        const BatchItem it = items[k];
        const BatchMol d = mols[it.mol];
        switch (d.ncb) {
#define VV10_CASE(c) \
    case c:          \
        if constexpr (c <= MAX) run_item<PREC, c>(d, it, smem, smem2); \
        break;
            VV10_CASE(1) VV10_CASE(2) VV10_CASE(3) VV10_CASE(4) VV10_CASE(5) VV10_CASE(6)
            VV10_CASE(7) VV10_CASE(8) VV10_CASE(9) VV10_CASE(10) VV10_CASE(11) VV10_CASE(12)
#undef VV10_CASE
            default: break;
        }
        __syncthreads();                   // LDS is reused by the next item
    }
}

// Wide items of a split-BF16 batch (eight to twelve column blocks): the
// eight-wave form of the standalone kernel (128-point i tiles, 32-point
// stages with X straight into two LDS buffers) pulls them from a list and a
// counter of its own.  Only these column counts share its register
// allocation, which keeps the form's two waves per SIMD without spills
// (every column count in one kernel spilled it).
__global__ __launch_bounds__(512, 1) void k_contract_persistent_wide(
    const BatchMol *__restrict__ mols, const BatchItem *__restrict__ items, int32_t n_items,
    int32_t *__restrict__ counter) {
    static_assert(bf16_waves<kWideMinNcb>() == 8 && bf16_waves<12>() == 8,
                  "wide items run the eight-wave form");
    __shared__ __attribute__((aligned(16))) char smem[smem_bf16x3<12>()];
    __shared__ __attribute__((aligned(16))) char smem2[smem_bf16x3<12>()];
    __shared__ int32_t next;
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(counter, 1);
        __syncthreads();
        const int32_t k = __builtin_amdgcn_readfirstlane(next);   // uniform: item data in SGPRs
        __syncthreads();
        if (k >= n_items) break;          // every workgroup leaves once the list is drained
        const BatchItem it = items[k];
        const BatchMol d = mols[it.mol];
        const bf16x8 *xh = global_as<bf16x8>(d.X);
        const bf16x8 *xl = xh + d.npad * d.Pp * 2 / 8;
        const float4 *p0 = global_as<float4>(d.P0);
        const float4 *p1 = global_as<float4>(d.P1);
        double *y = global_ptr(static_cast<double *>(d.Ypart));
        switch (d.ncb) {
#define VV10_CASE(c)                                                                         \
    case c:                                                                                  \
        tile_bf16x3<c, false, 8>(d.npad, d.jlen, d.Pp, p0, p1, xh, xl, y, it.itile, it.grp, \
                                 it.split, smem, smem2);                                     \
        break;
            VV10_CASE(8) VV10_CASE(9) VV10_CASE(10) VV10_CASE(11) VV10_CASE(12)
#undef VV10_CASE
            default: break;
        }
        __syncthreads();                   // LDS is reused by the next item
    }
}

__global__ void k_zero_counter(int32_t *c) { *c = 0; }

__global__ __launch_bounds__(64) void k_batch_buffers(int32_t n_mol, const int64_t *__restrict__ off,
                                                      BatchBuffers all, BatchBuffers *__restrict__ dst) {
    const int32_t m = blockIdx.x * 64 + threadIdx.x;
    if (m >= n_mol) return;
    const int64_t rx = off[2 * m], h = off[2 * m + 1];
    dst[m] = {all.rho_x + rx, all.grad_rho_x + 3 * rx, all.energy + m, all.hess + h};
}

// The grid pass (with the pair integrals) and the contraction of a small call
// as one launch: workgroups b < ngrid are grid units, the others contraction
// tiles, which need nothing from each other.  A grid of a few hundred units
// leaves part of the chip idle by itself; the tiles fill it.  A Hessian call of
// one water (N 1500, FP64) 153 -> 133 us, of two (N 4200) 267 -> 248 in FP64,
// 230 -> 214 in FP32, 205 -> 185 in split-BF16; of four (N 12000, 2256 units)
// 1243 -> 1225 and 573 -> 555; of five (N 16500, 4050 units) 2680 -> 2671 and 977 ->
// 941, past the line.  The six of N 18000 (5184 units) lose 0.6 % in FP64 and the
// hexamer (N 27000, 7776 units), whose tiles run with the grid pass's registers
// here, 7.09 -> 7.18 ms: at ten units a CU the line is on the safe side.
constexpr int kTogetherNcb = 4, kTogetherUnitsPerCu = 10;
template <int PREC, int NCB, int NQ>
__global__ __launch_bounds__(256, PREC == VV10_FP64 || (PREC == VV10_MIXED_BF16X3 && NCB > 2) ? 3 : 4) void k_grid_contract(
    int32_t ngrid, int32_t ntiles, int32_t bgroups, bool whole, int32_t n_atom, int64_t npad, int64_t jlen,
    int32_t Pp, const int64_t *__restrict__ seg, const int32_t *__restrict__ tile_i0,
    const int32_t *__restrict__ tile_n, const int32_t *__restrict__ tile_atom,
    const void *__restrict__ P0v, const void *__restrict__ P1v, const double4 *__restrict__ Pd,
    const void *__restrict__ Xv, double *__restrict__ Z, double *__restrict__ Dpart,
    double *__restrict__ Igrp, double *__restrict__ Yout) {
    using T = std::conditional_t<PREC == VV10_FP64, double, float>;
    using T4 = std::conditional_t<PREC == VV10_FP64, double4, float4>;
    constexpr int kTile = PREC == VV10_FP64 ? smem_f64<NCB>()
                          : PREC == VV10_MIXED_FP32 ? smem_f32<NCB>() : smem_bf16x3<NCB>();
    constexpr int kSmem = std::max<int>(kTile, sizeof(GridLds<T4>));
    __shared__ __attribute__((aligned(16))) char smem[kSmem];
    // the second stage buffer of the split-BF16 form (a one-byte dummy otherwise)
    __shared__ __attribute__((aligned(16))) char smem2[PREC == VV10_MIXED_BF16X3 ? kTile : 1];
    const T4 *P0 = static_cast<const T4 *>(P0v), *P1 = static_cast<const T4 *>(P1v);
    const int b = blockIdx.x;
    if (b < ngrid) {
        const int grp = b / ntiles;
        grid_unit<T, T4, true, false>(n_atom, Pp, bgroups, npad, seg, tile_i0, tile_n, tile_atom,
                                      P0, P1, Pd, Z, nullptr, Dpart, Igrp, b - grp * ntiles, grp, whole,
                                      *reinterpret_cast<GridLds<T4> *>(smem));
        return;
    }
    const int it = (int)(npad / 64), k = b - ngrid, split = k / it, itile = k - split * it;
    if constexpr (PREC == VV10_FP64)
        tile_f64<NCB, false, NQ>(npad, jlen, Pp, P0, P1, static_cast<const double *>(Xv), Yout,
                                 itile, 0, split, smem);
    else if constexpr (PREC == VV10_MIXED_FP32)
        tile_f32<NCB>(npad, jlen, Pp, P0, P1, static_cast<const float *>(Xv), Yout, itile, 0,
                      split, smem);
    else
        tile_bf16x3<NCB, false, 4>(npad, jlen, Pp, P0, P1, static_cast<const bf16x8 *>(Xv),
                                   static_cast<const bf16x8 *>(Xv) + npad * Pp * 2 / 8, Yout, itile,
                                   0, split, smem, smem2);
}

template <int PREC, int NCB, int NQ>
void grid_contract_launch(vv10_plan *p, const Workspace &ws) {
    const int32_t ngrid = p->ntiles * ws.bgroups;
    const unsigned blocks = (unsigned)(ngrid + p->npad / 64 * ws.jsplit);
    const void *P0 = PREC == VV10_FP64 ? (const void *)p->P0 : p->P0f;
    const void *P1 = PREC == VV10_FP64 ? (const void *)p->P1 : p->P1f;
    k_grid_contract<PREC, NCB, NQ><<<blocks, 256, 0, p->stream>>>(
        ngrid, p->ntiles, ws.bgroups, p->whole, p->n_atom, p->npad, ws.jlen, ws.Pp, p->d_seg, p->d_tile_i0,
        p->d_tile_n, p->d_tile_atom, P0, P1, p->P1, ws.X, ws.Z, ws.Dpart, ws.Igrp,
        static_cast<double *>(ws.Ypart));
}

template <int NCB>
void grid_contract_mode(vv10_plan *p, const Workspace &ws) {
    if (p->prec == VV10_MIXED_FP32) return grid_contract_launch<VV10_MIXED_FP32, NCB, 4>(p, ws);
    if (p->prec == VV10_MIXED_BF16X3) return grid_contract_launch<VV10_MIXED_BF16X3, NCB, 4>(p, ws);
    const int left = ws.P - (ws.Pp - 16), nq = left > 0 ? (left + 3) / 4 : 4;
    if (nq == 1) grid_contract_launch<VV10_FP64, NCB, 1>(p, ws);
    else if (nq == 2) grid_contract_launch<VV10_FP64, NCB, 2>(p, ws);
    else if (nq == 3) grid_contract_launch<VV10_FP64, NCB, 3>(p, ws);
    else grid_contract_launch<VV10_FP64, NCB, 4>(p, ws);
}

// ---------------------------------------------------------------------------
// Fused split-BF16 contraction for weights that move with the nuclei (one
// column group of at most four blocks): the pair geometry of each (i, j) is
// formed once for the main 2 x 2 kernel and for the three weight rows
// Y_pv, Y_qv, Y_vv of the weight contraction (weights.hip).  A stage is a
// 32-point j block: the main contraction takes it as two 16-point
// sub-blocks, the weight contraction as one K of 32 whose order follows the
// same lanes' pairs, k = 8 g + e for the point 4 g + e (e < 4) or
// 16 + 4 g + e - 4 (e >= 4) of the block, which is the order in which the
// weight packing stores v.
// ---------------------------------------------------------------------------
// Two pairs of a block in four steps, so that a caller can place each step
// between MFMAs: (0) the geometries and reciprocals, (1) the four main values
// and the three weight values (r - c_i A, -R^2 A, r) of each pair, divided by
// -3/2, (2) the hi/lo split of the main values, (3) that of the weight values
// (two pairs share a word).  The main values are those of pair_K.
struct PairStepsW {
    float R2[2], gg[2], gp[2], s[2], t[2], r[2], k[2][7];
    __device__ __forceinline__ void geometry(int u, const float4 a0, const float4 a1,
                                             const float4 b0, const float2 b1) {
        const float dx = a0.x - b0.x, dy = a0.y - b0.y, dz = a0.z - b0.z;
        R2[u] = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
        gg[u] = __builtin_fmaf(a0.w, R2[u], a1.x);
        gp[u] = __builtin_fmaf(b0.w, R2[u], b1.x);
        s[u] = gg[u] + gp[u];
        t[u] = gg[u] * gp[u];
        r[u] = rcp32(t[u] * s[u]);
    }
    // self: the self pair, whose K_pp and rows r - c_i A and r are left out
    // (the others vanish there)
    __device__ __forceinline__ void values(int u, float ci, float cj, bool self) {
        const float sr = s[u] * r[u];
        const float is = t[u] * r[u];
        const float A = r[u] * __builtin_fmaf(gp[u], sr, is);
        const float Ap = r[u] * __builtin_fmaf(gg[u], sr, is);
        const float Q = (r[u] + r[u]) * __builtin_fmaf(is, is, sr);
        const float t1 = __builtin_fmaf(ci, Q, -Ap);
        const float t2 = __builtin_fmaf(cj, Q, -A);
        const float base = __builtin_fmaf(-ci, A, r[u]);
        const float kpp = __builtin_fmaf(cj, t1, base);
        k[u][0] = self ? 0.f : kpp;
        k[u][1] = R2[u] * t1;                       // kpq
        k[u][2] = R2[u] * t2;                       // kqp
        k[u][3] = (R2[u] * R2[u]) * Q;              // kqq
        k[u][4] = self ? 0.f : base;                // kpv
        k[u][5] = -R2[u] * A;                       // kqv
        k[u][6] = self ? 0.f : r[u];                // kvv
    }
};

// LDS units (16 B) of a stage: main hi and lo of two 16-point blocks, weight
// hi and lo of the 32-point block (NCB x 64 units each), 64 units each of P0, P1.
template <int NCB>
constexpr int units_bf16x3_w() { return (6 * NCB + 2) * 64; }

// Pipelined as tile_bf16x3, in chunks of one column block: NCB chunks of the
// first 16-point block (six MFMAs), NCB of the second, NCB of the weight rows
// (nine).  During the first NCB chunks the pairs of the second block are
// formed, during the others those of the next stage's first block; the weight
// rows' operands consist of both halves, so the half formed a stage ahead
// waits in registers.  With the operands formed at the stage's start, the
// staged data through registers and the reads next to their MFMAs the weighted
// hexamer took 2.31 ms at 2.0 GHz, now 2.05 ms at 1.93 GHz.
template <int NCB>
__global__ __launch_bounds__(256, 2) void k_contract_bf16x3_w(
    int64_t npad, int64_t jlen, int32_t Pp, const float4 *__restrict__ P0,
    const float4 *__restrict__ P1, const bf16x8 *__restrict__ Xhi, const bf16x8 *__restrict__ Xlo,
    const bf16x8 *__restrict__ Vhi, const bf16x8 *__restrict__ Vlo, double *__restrict__ Yout,
    double *__restrict__ Ywout) {
    static_assert(kFp32Run % 64 == 0, "FP32 runs end on stage pairs");
    constexpr int C = 3 * NCB;                  // chunks of a stage
    constexpr int kAhead = NCB == 1 ? 1 : 2;
    constexpr int PER = (6 * NCB + 3) / 4;      // 64-unit pieces per wave and stage
    __shared__ __attribute__((aligned(16))) bf16x8 buf0[units_bf16x3_w<NCB>()];
    __shared__ __attribute__((aligned(16))) bf16x8 buf1[units_bf16x3_w<NCB>()];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int64_t ibase = (int64_t)blockIdx.x * 64 + wave * 16;
    const int64_t jbeg = (int64_t)blockIdx.z * jlen;
    const int64_t jend = min(npad, jbeg + jlen);
    const float4 a0 = P0[ibase + m], a1 = P1[ibase + m];
    v4f accp[NCB], accq[NCB], awp[NCB], awq[NCB], awv[NCB];
    auto clear = [&]() {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            accp[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
            accq[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
            awp[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
            awq[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
            awv[cb] = (v4f){0.f, 0.f, 0.f, 0.f};
        }
    };
    clear();
    // the FP32 sums of each run of kFp32Run points go into this split's
    // partials (D layout: item r of lane l holds row 4 (l/16) + r, column l%16)
    const PartialRows Yb(Yout, blockIdx.z, npad * 2 * Pp, partials_f32(npad, jlen));
    const PartialRows Yw(Ywout, blockIdx.z, npad * 3 * Pp, partials_f32(npad, jlen));
    bool first = true;
    auto flush = [&]() {
        // base addresses formed here (the empty asm keeps them from being
        // hoisted out of the loop)
        int64_t ob = (ibase + 4 * g) * 2 * Pp + m, ow = (ibase + 4 * g) * 3 * Pp + m;
        asm volatile("" : "+v"(ob), "+v"(ow));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float v[5][NCB];
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                v[0][cb] = accp[cb][r];
                v[1][cb] = accq[cb][r];
                v[2][cb] = awp[cb][r];
                v[3][cb] = awq[cb][r];
                v[4][cb] = awv[cb][r];
            }
            add_row<NCB>(Yb, ob + (2 * r + 0) * (int64_t)Pp, v[0], first);
            add_row<NCB>(Yb, ob + (2 * r + 1) * (int64_t)Pp, v[1], first);
            add_row<NCB>(Yw, ow + (3 * r + 0) * (int64_t)Pp, v[2], first);
            add_row<NCB>(Yw, ow + (3 * r + 1) * (int64_t)Pp, v[3], first);
            add_row<NCB>(Yw, ow + (3 * r + 2) * (int64_t)Pp, v[4], first);
        }
        clear();
        first = false;
    };
    auto to_lds = [](const void *base, uint32_t off, bf16x8 *dst) { load16_lds(base, off, 0, dst); };
    // piece k: 64 units of one array and column block (where the waves
    // outnumber the pieces left, some bring one that another wave brings too);
    // its source at j = 0 and the units from one 16-point block to the next,
    // in SGPRs
    const bf16x8 *src[PER];
    int64_t blk[PER];
    int unit[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int q = (wave + 4 * k) % (6 * NCB), arr = q / NCB, cb = q - arr * NCB;
        const bf16x8 *x = Xhi;
        if (arr >= 2) x = Xlo;
        if (arr == 4) x = Vhi;
        if (arr == 5) x = Vlo;
        src[k] = x + (arr < 4 ? (arr & 1) * Pp * 4 : 0) + cb * 64;
        blk[k] = arr < 4 ? 4 * Pp : 2 * Pp;
        unit[k] = q * 64;
    }
    const float4 *psrc = P0;
    if (wave & 1) psrc = P1;
    const int punit = (6 * NCB + (wave & 1)) * 64;
    // piece k (the points: k = PER) of the stage at j
    auto load_piece = [&](int k, int64_t j, bf16x8 *buf) __attribute__((always_inline)) {
        if (k == PER) {
            const uint32_t left = (uint32_t)min(npad - 1 - j, (int64_t)64);
            to_lds(psrc + j, min(16u + (lane & 31), left) * (uint32_t)sizeof(float4), buf + punit);
        } else {
            to_lds(src[k] + (j / 16) * blk[k], lane * (uint32_t)sizeof(bf16x8), buf + unit[k]);
        }
    };
    // points of this lane's four pairs of a block: (x, y, z, omega), (kappa, c)
    float4 n0[4];
    float2 n1[4];
    auto read_points = [&](const bf16x8 *buf, int sub) {
        const float4 *q = reinterpret_cast<const float4 *>(buf + 6 * NCB * 64) + 16 * sub + 4 * g;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            n0[jj] = q[jj];
            n1[jj] = make_float2(q[64 + jj].x, q[64 + jj].z);
        }
    };
    // the diagonal block leaves out the self pair: pair m mod 4 of lane (m, g = m/4)
    bool self[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) self[jj] = m == 4 * g + jj;
    PairStepsW ps;
    uint32_t ph[4], pl[4], qh[4], ql[4];             // main words being formed
    uint32_t wf[6][2];                               // weight words being formed (ph, pl, qh, ql, vh, vl)
    // step k of eight: pairs 2 (k / 4) and 2 (k / 4) + 1 (the empty asm
    // statements keep each step's instructions in its chunk)
    auto step = [&](int k, bool diag) {
        const int e = 2 * (k / 4);
        if (k % 4 == 0) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                ps.geometry(u, a0, a1, n0[e + u], n1[e + u]);
                asm volatile("" : "+v"(ps.R2[u]), "+v"(ps.gg[u]), "+v"(ps.gp[u]), "+v"(ps.s[u]),
                             "+v"(ps.t[u]), "+v"(ps.r[u]));
            }
        } else if (k % 4 == 1) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                ps.values(u, a1.z, n1[e + u].y, diag && self[e + u]);
                asm volatile("" : "+v"(ps.k[u][0]), "+v"(ps.k[u][1]), "+v"(ps.k[u][2]),
                             "+v"(ps.k[u][3]), "+v"(ps.k[u][4]), "+v"(ps.k[u][5]), "+v"(ps.k[u][6]));
            }
        } else if (k % 4 == 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                split2(ps.k[u][0], ps.k[u][1], ph[e + u], pl[e + u]);
                split2(ps.k[u][2], ps.k[u][3], qh[e + u], ql[e + u]);
                asm volatile("" : "+v"(ph[e + u]), "+v"(pl[e + u]), "+v"(qh[e + u]), "+v"(ql[e + u]));
            }
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                split2(ps.k[0][4 + c], ps.k[1][4 + c], wf[2 * c][e / 2], wf[2 * c + 1][e / 2]);
                asm volatile("" : "+v"(wf[2 * c][e / 2]), "+v"(wf[2 * c + 1][e / 2]));
            }
        }
    };
    auto formed = [&]() {
        Aops A;
        A.ph = __builtin_bit_cast(bf16x8, (uint4){ph[0], ph[1], ph[2], ph[3]});
        A.pl = __builtin_bit_cast(bf16x8, (uint4){pl[0], pl[1], pl[2], pl[3]});
        A.qh = __builtin_bit_cast(bf16x8, (uint4){qh[0], qh[1], qh[2], qh[3]});
        A.ql = __builtin_bit_cast(bf16x8, (uint4){ql[0], ql[1], ql[2], ql[3]});
        return A;
    };
    Aops A;                       // main operands of the block at hand
    uint32_t wa[6][2];            // weight words of the stage's first half
    bf16x8 W[6];                  // weight operands of the stage
    bf16x8 Bh[kAhead + 1], Bl[kAhead + 1];
    // B operands of chunk c: block 0, block 1, weight rows
    auto unit_hi = [](int c) { return c < 2 * NCB ? c : c + 2 * NCB; };
    auto unit_lo = [](int c) { return c < 2 * NCB ? c + 2 * NCB : c + 3 * NCB; };
    auto stage = [&](int64_t j0, bf16x8 *cur, bf16x8 *nxt) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int part = c / NCB, cb = c - part * NCB;
            if (c == C - kAhead) {
                __builtin_amdgcn_s_waitcnt(0);   // this wave's LDS loads and reads are done
                __syncthreads();
            }
            // pieces of the next stage (past the last one: that one again)
#pragma unroll
            for (int k = 0; k <= PER; ++k)
                if (c == (k < C - kAhead ? k : C - kAhead - 1))
                    load_piece(k, min(j0 + 32, jend - 32), nxt);
            __builtin_amdgcn_sched_barrier(0);
            {
                const int pc = c + kAhead, q = pc % C;
                const bf16x8 *b = (pc < C ? cur : nxt) + lane;
                Bh[kAhead] = b[unit_hi(q) * 64];
                Bl[kAhead] = b[unit_lo(q) * 64];
            }
            __builtin_amdgcn_sched_barrier(0);
            const bf16x8 bh = Bh[0], bl = Bl[0];
            if (part < 2) {
                accp[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.ph, bh, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.qh, bh, accq[cb], 0, 0, 0);
                accp[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.pl, bh, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.ql, bh, accq[cb], 0, 0, 0);
                accp[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.ph, bl, accp[cb], 0, 0, 0);
                accq[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.qh, bl, accq[cb], 0, 0, 0);
            } else {
                awp[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[0], bh, awp[cb], 0, 0, 0);
                awq[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[2], bh, awq[cb], 0, 0, 0);
                awv[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[4], bh, awv[cb], 0, 0, 0);
                awp[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[1], bh, awp[cb], 0, 0, 0);
                awq[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[3], bh, awq[cb], 0, 0, 0);
                awv[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[5], bh, awv[cb], 0, 0, 0);
                awp[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[0], bl, awp[cb], 0, 0, 0);
                awq[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[2], bl, awq[cb], 0, 0, 0);
                awv[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[4], bl, awv[cb], 0, 0, 0);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (part == 0 && k * NCB / 8 == cb) step(k, j0 + 16 == ibase);
                if (part > 0 && k * 2 * NCB / 8 == c - NCB) step(k, j0 + 32 == ibase);
            }
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                Bh[k] = Bh[k + 1];
                Bl[k] = Bl[k + 1];
            }
            __builtin_amdgcn_sched_barrier(0);
            if (c == NCB - 1) {
                A = formed();
#pragma unroll
                for (int k = 0; k < 6; ++k)
                    W[k] = __builtin_bit_cast(bf16x8, (uint4){wa[k][0], wa[k][1], wf[k][0], wf[k][1]});
                read_points(cur, 1);
            }
            if (c == C - 1) {
                A = formed();
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    wa[k][0] = wf[k][0];
                    wa[k][1] = wf[k][1];
                }
                read_points(nxt, 0);
            }
        }
    };
#pragma unroll
    for (int k = 0; k <= PER; ++k) load_piece(k, jbeg, buf0);
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        n0[jj] = P0[jbeg + 4 * g + jj];
        n1[jj] = make_float2(P1[jbeg + 4 * g + jj].x, P1[jbeg + 4 * g + jj].z);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) step(k, jbeg == ibase);
    A = formed();
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        wa[k][0] = wf[k][0];
        wa[k][1] = wf[k][1];
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
        Bh[k] = buf0[unit_hi(k) * 64 + lane];
        Bl[k] = buf0[unit_lo(k) * 64 + lane];
    }
    read_points(buf0, 0);
    int64_t j0 = jbeg;
    for (; j0 + 64 <= jend; j0 += 64) {
        stage(j0, buf0, buf1);
        stage(j0 + 32, buf1, buf0);
        if ((j0 + 64 - jbeg) % kFp32Run == 0 && j0 + 64 < jend) flush();
    }
    if (j0 < jend) stage(j0, buf0, buf1);
    flush();
}

template <int NCB>
hipError_t run_weighted(vv10_plan *p, const Workspace &ws, const WeightWork &ww) {
    dim3 grid((unsigned)(p->npad / 64), 1u, (unsigned)ws.jsplit);
    const bf16x8 *xh = static_cast<const bf16x8 *>(ws.X);
    const bf16x8 *xl = xh + (size_t)p->npad * ws.Pp * 2 / 8;
    const bf16x8 *vh = static_cast<const bf16x8 *>(ww.Xv);
    const bf16x8 *vl = vh + (size_t)p->npad * ws.Pp / 8;
    k_contract_bf16x3_w<NCB><<<grid, 256, 0, p->stream>>>(
        p->npad, ws.jlen, ws.Pp, p->P0f, p->P1f, xh, xl, vh, vl, static_cast<double *>(ws.Ypart),
        static_cast<double *>(ww.Ypart));
    return hipGetLastError();
}

}  // namespace

// The mixed modes' counts are fixed numbers, not what the built kernels reach
// (split-BF16 now holds three workgroups at three and four blocks and two at
// seven): the split count that follows from them decides where the FP32 runs end,
// so a result would otherwise change in its last FP32 digits whenever a compiler
// allocates a register more or a kernel is rewritten.
int contract_blocks_per_cu(vv10_precision prec, int ncb) {
    static constexpr int f32_slots[13] = {0, 8, 8, 8, 6, 5, 5, 4, 4, 3, 3, 3, 3};
    if (ncb < 1 || ncb > max_ncb(prec)) return 0;
    if (prec == VV10_MIXED_FP32) return f32_slots[ncb];
    if (prec == VV10_MIXED_BF16X3) return ncb <= 4 ? 4 : (ncb < kWideMinNcb ? 3 : 2);
    return dispatch_ncb(ncb, [](auto c) { return occupancy_f64<decltype(c)::value>(); });
}

hipError_t launch_contract(vv10_plan *p, const Workspace &ws, bool screen) {
    if (ws.ncb < 1 || ws.ncb > max_ncb(p->prec)) return hipErrorInvalidValue;
    return dispatch_ncb(ws.ncb, [&](auto c) { return run<decltype(c)::value>(p, ws, screen); });
}

bool grid_contract_together(const vv10_plan *p, const Workspace &ws) {
    return ws.ngroups == 1 && ws.ncb <= kTogetherNcb &&
           (int64_t)p->ntiles * ws.bgroups <= kTogetherUnitsPerCu * (int64_t)p->num_cu;
}

hipError_t launch_grid_contract(vv10_plan *p, const Workspace &ws) {
    if (!grid_contract_together(p, ws)) return hipErrorInvalidValue;
    if (ws.ncb == 1) grid_contract_mode<1>(p, ws);
    else if (ws.ncb == 2) grid_contract_mode<2>(p, ws);
    else if (ws.ncb == 3) grid_contract_mode<3>(p, ws);
    else grid_contract_mode<4>(p, ws);
    return hipGetLastError();
}

bool fused_weighted_contract(const vv10_plan *p, const Workspace &ws) {
    return p->prec == VV10_MIXED_BF16X3 && ws.ngroups == 1 && ws.ncb <= 4;
}

hipError_t launch_contract_weighted(vv10_plan *p, const Workspace &ws, const WeightWork &ww) {
    if (!fused_weighted_contract(p, ws)) return hipErrorInvalidValue;
    switch (ws.ncb) {
        case 1: return run_weighted<1>(p, ws, ww);
        case 2: return run_weighted<2>(p, ws, ww);
        case 3: return run_weighted<3>(p, ws, ww);
        case 4: return run_weighted<4>(p, ws, ww);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace vv10

namespace vv10 {

int persistent_waves(vv10_precision prec) {
    if (prec == VV10_FP64) return PersistentTraits<VV10_FP64>::kWaves;
    if (prec == VV10_MIXED_FP32) return PersistentTraits<VV10_MIXED_FP32>::kWaves;
    return PersistentTraits<VV10_MIXED_BF16X3>::kWaves;
}

namespace {

using PersistentKernel = void (*)(const BatchMol *, const BatchItem *, int32_t, int32_t *);

template <int PREC>
PersistentKernel persistent_form(int max_ncb) {
    if (max_ncb <= kNarrowNcb) return k_contract_persistent<PREC, kNarrowNcb>;
    return k_contract_persistent<PREC, PersistentTraits<PREC>::kMaxNcb>;
}

PersistentKernel persistent_kernel(vv10_precision prec, int max_ncb) {
    if (prec == VV10_FP64) return persistent_form<VV10_FP64>(max_ncb);
    if (prec == VV10_MIXED_FP32) return persistent_form<VV10_MIXED_FP32>(max_ncb);
    return persistent_form<VV10_MIXED_BF16X3>(max_ncb);
}

}  // namespace

int persistent_blocks_per_cu(vv10_precision prec, int max_ncb) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, reinterpret_cast<const void *>(persistent_kernel(prec, max_ncb)),
            64 * persistent_waves(prec), 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return nb;
}

int persistent_wide_blocks_per_cu() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_contract_persistent_wide, 512, 0) !=
        hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return nb;
}
hipError_t launch_batch_buffers(int32_t n_mol, const int64_t *off, const BatchBuffers &all,
                                BatchBuffers *dst, hipStream_t stream) {
    k_batch_buffers<<<(unsigned)((n_mol + 63) / 64), 64, 0, stream>>>(n_mol, off, all, dst);
    return hipGetLastError();
}
hipError_t launch_contract_persistent_wide(const BatchMol *mols, const BatchItem *items,
                                           int32_t n_items, int32_t *counter, int n_blocks,
                                           hipStream_t stream) {
    k_zero_counter<<<1, 1, 0, stream>>>(counter);
    k_contract_persistent_wide<<<n_blocks, 512, 0, stream>>>(mols, items, n_items, counter);
    return hipGetLastError();
}
int persistent_grid_blocks_per_cu(vv10_precision prec) {
    int nb = 0;
    hipError_t e;
    if (prec == VV10_FP64)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_grid_persistent<VV10_FP64>, 64 * kGridWaves, 0);
    else if (prec == VV10_MIXED_FP32)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_grid_persistent<VV10_MIXED_FP32>, 64 * kGridWaves, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_grid_persistent<VV10_MIXED_BF16X3>, 64 * kGridWaves, 0);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return nb;
}
hipError_t launch_grid_persistent(vv10_precision prec, const BatchMol *mols,
                                  const BatchItem *items, int32_t n_items, int32_t *counter,
                                  int n_blocks, hipStream_t stream) {
    k_zero_counter<<<1, 1, 0, stream>>>(counter);
    if (prec == VV10_FP64)
        k_grid_persistent<VV10_FP64><<<n_blocks, 64 * kGridWaves, 0, stream>>>(mols, items, n_items, counter);
    else if (prec == VV10_MIXED_FP32)
        k_grid_persistent<VV10_MIXED_FP32><<<n_blocks, 64 * kGridWaves, 0, stream>>>(mols, items, n_items, counter);
    else
        k_grid_persistent<VV10_MIXED_BF16X3><<<n_blocks, 64 * kGridWaves, 0, stream>>>(mols, items, n_items, counter);
    return hipGetLastError();
}
hipError_t launch_contract_persistent(vv10_precision prec, int max_ncb, const BatchMol *mols,
                                      const BatchItem *items, int32_t n_items, int32_t *counter,
                                      int n_blocks, hipStream_t stream) {
    k_zero_counter<<<1, 1, 0, stream>>>(counter);
    persistent_kernel(prec, max_ncb)<<<n_blocks, 64 * persistent_waves(prec), 0, stream>>>(
        mols, items, n_items, counter);
    return hipGetLastError();
}

}  // namespace vv10
