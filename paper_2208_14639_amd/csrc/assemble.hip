// Hessian assembly (Section II.B, nine-term split).  All FP64.
//
// 1. k_resp, one wave per point i, lanes over the perturbations x:
//      Y = sum of the contraction's j-split partials (split order, FP64)
//          plus the self pair j = i, which the contraction leaves out:
//          Y_p += K_pp(i, i) p_i in FP64
//      Yr = Y_p + rho omega_r Y_q + loc_rho,   Yg = rho omega_g Y_q + loc_gamma
//    (the paper's inner sums sum_j w_j (f^{rho rho}_ij rho^x_j + f^{rho gamma}_ij gamma^x_j)
//    and sum_j w_j (f^{gamma rho}_ij rho^x_j + f^{gamma gamma}_ij gamma^x_j); the local parts are
//    the delta_ij terms, written as derivatives along the perturbation:
//      dk = kappa_r rho^x, dw = omega_r rho^x + omega_g gamma^x,
//      loc_rho   = U dk + W dw + rho^x (kappa_r U + omega_r W)
//                + rho (A kappa_r dk + B (kappa_r dw + omega_r dk) + C omega_r dw)
//                + rho (kappa_rr rho^x U + (omega_rr rho^x + omega_rg gamma^x) W)
//      loc_gamma = rho^x omega_g W + rho (B omega_g dk + C omega_g dw)
//                + rho (omega_rg rho^x + omega_gg gamma^x) W),
//    the grid channels Zr = Z_p + rho omega_r Z_q, Zg = rho omega_g Z_q (the
//    own-atom slot filled by translational invariance, a wave reduction over
//    the other atoms' slots), and R = w (Yr + 2 Zr, Yg + 2 Zg), written over Y.
//    Optional outputs: Yr, Yg (response rows) and Yr + Zr, Yg + Zg (the
//    grid-level coefficients of the Fock nuclear derivative).
//    With weight derivatives w^x (weights that move with the nuclei) the
//    weight contraction's (Y_pv, Y_qv, Y_vv) and the grid channel
//    Ze = E^{xgr} (own slot by invariance again) add
//      Wr = Y_pv + rho omega_r Y_qv,  Wg = rho omega_g Y_qv
//      R += (2 w Wr + 2 w^x f^rho, 2 w Wg + 2 w^x f^gamma),
//      Rw = rho (Y_vv + 2 Ze)     (right factor of the w^x rows),
//    and Wr, Wg to the Fock coefficients (F^A_w without its first line).
// 2. k_gemm: per slice s of points, Hpart[s][l][m] = sum_i L_i^T R_i with
//    L = (rho^x, gamma^x) on FP64 MFMA, so that sum_s Hpart[s] = E_GG + 2 E_{G,gr}
//    (E_GG without the rho^{AB} term); row Pp of each slice holds the gradient
//    part E_G = sum_i w_i (f^rho_i rho^x_i + f^gamma_i gamma^x_i).  With
//    weight derivatives a second GEMM over the rows L = w^x, R = Rw adds
//    E_ww + 2 E_{w,gr} (E_ww = sum_i w^A_i rho_i E^{Bw}_i, symmetric) and, in
//    row Pp, E_w = sum_i w^x_i rho_i (beta + E_i); the R terms above add
//    2 E_{G,w}.  Symmetrised, this is the nine-term split without the
//    caller's rho^{AB} and w^{AB} sums.
// 3. k_sums: Hsum = sum_s Hpart[s] in a fixed order (the w^x slices after
//    the others), and the E_{gr,gr} tile sums of a_i D^B_i reduced per atom
//    pair.
// 4. k_finish: H = sym(Hsum) + sym(E_{gr,gr}), sym(M) = (M + M^T)/2, with the
//    diagonal blocks of E_{gr,gr} from translational invariance, and the
//    gradient E_G + E_gr, E_gr = sum_{i in A} a_i E^{Agr}_i
//    = -sum_{B != A} sum_{i in A} a_i E^{Bgr}_i.
#include <algorithm>
#include <type_traits>

#include "dev_common.h"
#include "vv10_internal.h"

namespace vv10 {

namespace {

// Per-point quantities of the same-point (delta_ij) terms.
struct PointFields {
    double w, r, omr, omg, kar, omrr, omrg, omgg, karr, U, W, A, B, C;
};

__device__ __forceinline__ PointFields point_fields(const double *__restrict__ F,
                                                    const double *__restrict__ I, int64_t npad,
                                                    int64_t i) {
    PointFields f;
    f.w = F[F_W * npad + i];
    f.r = F[F_RHO * npad + i];
    f.omr = F[F_OMR * npad + i];
    f.omg = F[F_OMG * npad + i];
    f.kar = F[F_KAR * npad + i];
    f.omrr = F[F_OMRR * npad + i];
    f.omrg = F[F_OMRG * npad + i];
    f.omgg = F[F_OMGG * npad + i];
    f.karr = F[F_KARR * npad + i];
    f.U = I[I_U * npad + i];
    f.W = I[I_W * npad + i];
    f.A = I[I_A * npad + i];
    f.B = I[I_B * npad + i];
    f.C = I[I_C * npad + i];
    return f;
}

// Yr, Yg of one point and perturbation from the contraction's channel sums
// (yp, yq) and the perturbation values (rx = rho^x, gx = gamma^x).
__device__ __forceinline__ void point_response(const PointFields &f, double rx, double gx,
                                               double yp, double yq, double &Yr, double &Yg) {
    const double dk = f.kar * rx;
    const double dw = f.omr * rx + f.omg * gx;
    const double loc_r = f.U * dk + f.W * dw + rx * (f.kar * f.U + f.omr * f.W)
                       + f.r * (f.A * f.kar * dk + f.B * (f.kar * dw + f.omr * dk) + f.C * f.omr * dw)
                       + f.r * (f.karr * rx * f.U + (f.omrr * rx + f.omrg * gx) * f.W);
    const double loc_g = rx * f.omg * f.W + f.r * (f.B * f.omg * dk + f.C * f.omg * dw)
                       + f.r * (f.omrg * rx + f.omgg * gx) * f.W;
    Yr = yp + f.r * f.omr * yq + loc_r;
    Yg = f.r * f.omg * yq + loc_g;
}

// Inputs of the weight-derivative terms (all null without weight derivatives).
template <typename T>
struct WeightIn {
    const T *Ypart;        // [S][npad][3][Pp] (Y_pv, Y_qv, Y_vv) partials
    const double *Lw;      // [npad][Pp] w^x
    const double *Ze;      // [npad][Pp] E^{xgr} (own slot not written)
    double *Rw;            // [npad][Pp] output
};

// One wave per point; the partials are [S][npad][2][Pp], FP64 or, in the mixed
// modes with splits of one FP32 run, the FP32 sums themselves (with one split
// they are FP64 and alias Y, read before R is written in place).
template <typename T, bool WT>
__global__ __launch_bounds__(256) void k_resp(
    int64_t n, int64_t npad, int32_t P, int32_t Pp, int32_t S, const int32_t *__restrict__ atom_of,
    const double4 *__restrict__ P1, const double *__restrict__ F, const double *__restrict__ I,
    const double *__restrict__ L, const T *Ypart, double *Y, const double *__restrict__ Z, WeightIn<T> wt,
    double *__restrict__ resp_rho, double *__restrict__ resp_gamma, double *__restrict__ fock_rho,
    double *__restrict__ fock_gamma) {
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (i >= n) return;
    const PointFields f = point_fields(F, I, npad, i);
    const int A = atom_of[i];
    // the self pair, left out of the contraction: K_pp p_i (and for the
    // weight rows (Phi + c Phi_g) v_i, Phi v_i), in FP64
    const double4 pd = P1[i];
    const double kself = self_kpp(pd.x, pd.z);
    const SelfPair sq = self_pair(pd.x);
    const double kself_pv = sq.phi + pd.z * sq.phig, kself_vv = sq.phi;
    const double *z0 = Z + (i * 2 + 0) * Pp, *z1 = Z + (i * 2 + 1) * Pp;
    const double *ze = WT ? wt.Ze + i * Pp : nullptr;

    // own-atom slot: -sum over the other atoms' slots of the same direction
    double own0[3] = {0.0, 0.0, 0.0}, own1[3] = {0.0, 0.0, 0.0}, own2[3] = {0.0, 0.0, 0.0};
    for (int x0 = 0; x0 < P; x0 += 64) {
        const int x = x0 + lane;
        const bool use = x < P && x / 3 != A;
        const double v0 = use ? z0[x] : 0.0, v1 = use ? z1[x] : 0.0;
        const double v2 = (WT && use) ? ze[x] : 0.0;
        const int a = x % 3;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            own0[d] -= wave_sum(a == d ? v0 : 0.0);
            own1[d] -= wave_sum(a == d ? v1 : 0.0);
            if (WT) own2[d] -= wave_sum(a == d ? v2 : 0.0);
        }
    }

    const int64_t len = npad * 2 * Pp;
    for (int x = lane; x < Pp; x += 64) {
        double *y0 = Y + (i * 2 + 0) * Pp + x;
        double *y1 = Y + (i * 2 + 1) * Pp + x;
        if (x >= P) {
            *y0 = 0.0;
            *y1 = 0.0;
            if (WT) wt.Rw[i * Pp + x] = 0.0;
            continue;
        }
        const int64_t o = (i * 2) * Pp + x;
        double yp = (double)Ypart[o], yq = (double)Ypart[o + Pp];
        for (int s = 1; s < S; ++s) {
            yp += (double)Ypart[s * len + o];
            yq += (double)Ypart[s * len + o + Pp];
        }
        yp += kself * (f.w * L[o]);
        double Yr, Yg;
        point_response(f, L[o], L[o + Pp], yp, yq, Yr, Yg);
        const int a = x % 3;
        const bool self = x / 3 == A;
        const double o0 = a == 0 ? own0[0] : (a == 1 ? own0[1] : own0[2]);
        const double o1 = a == 0 ? own1[0] : (a == 1 ? own1[1] : own1[2]);
        const double zp = self ? o0 : z0[x];
        const double zq = self ? o1 : z1[x];
        const double Zr = zp + f.r * f.omr * zq, Zg = f.r * f.omg * zq;
        double Wr = 0.0, Wg = 0.0;
        if (WT) {
            const int64_t lw = npad * 3 * Pp, ow = (i * 3) * Pp + x;
            double ypv = (double)wt.Ypart[ow], yqv = (double)wt.Ypart[ow + Pp];
            double yvv = (double)wt.Ypart[ow + 2 * Pp];
            for (int s = 1; s < S; ++s) {
                ypv += (double)wt.Ypart[s * lw + ow];
                yqv += (double)wt.Ypart[s * lw + ow + Pp];
                yvv += (double)wt.Ypart[s * lw + ow + 2 * Pp];
            }
            const double vself = wt.Lw[i * Pp + x] * f.r;   // v_i = w^x_i rho_i
            ypv += kself_pv * vself;
            yvv += kself_vv * vself;
            const double o2 = a == 0 ? own2[0] : (a == 1 ? own2[1] : own2[2]);
            const double zev = self ? o2 : ze[x];
            const double wx = wt.Lw[i * Pp + x];
            Wr = ypv + f.r * f.omr * yqv;
            Wg = f.r * f.omg * yqv;
            *y0 = f.w * (Yr + 2.0 * Zr + 2.0 * Wr) + 2.0 * wx * F[F_FR * npad + i];
            *y1 = f.w * (Yg + 2.0 * Zg + 2.0 * Wg) + 2.0 * wx * F[F_FG * npad + i];
            wt.Rw[i * Pp + x] = f.r * (yvv + 2.0 * zev);
        } else {
            *y0 = f.w * (Yr + 2.0 * Zr);
            *y1 = f.w * (Yg + 2.0 * Zg);
        }
        if (resp_rho) resp_rho[(int64_t)x * n + i] = Yr;
        if (resp_gamma) resp_gamma[(int64_t)x * n + i] = Yg;
        if (fock_rho) fock_rho[(int64_t)x * n + i] = Yr + Zr + Wr;
        if (fock_gamma) fock_gamma[(int64_t)x * n + i] = Yg + Zg + Wg;
    }
}

// Trial-density response: f^{rho,t}_i = Yr, f^{gamma,t}_i = Yg of
// point_response for every trial column t (the perturbation packing wrote
// L = (rho^t, 2 grad rho . grad rho^t), which carries the factor 2 of the
// gamma terms).  32 points x 64 columns per workgroup, transposed through
// LDS so that the [n_t][N] outputs are written along points.
constexpr int TRI = 32, TRX = 64;
template <typename T>
__global__ __launch_bounds__(256) void k_trial_resp(
    int64_t n, int64_t npad, int32_t P, int32_t Pp, int32_t S, const double4 *__restrict__ P1,
    const double *__restrict__ F, const double *__restrict__ I, const double *__restrict__ L,
    const T *__restrict__ Ypart, double *__restrict__ f_rho_t, double *__restrict__ f_gamma_t) {
    __shared__ double sR[TRI][TRX + 1], sG[TRI][TRX + 1];
    const int tid = threadIdx.x, tx = tid & 63, ty = tid >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * TRI;
    const int x = blockIdx.y * TRX + tx;
    const int64_t len = npad * 2 * Pp;
    for (int rr = ty; rr < TRI; rr += 4) {
        const int64_t i = i0 + rr;
        double Yr = 0.0, Yg = 0.0;
        if (i < n && x < P) {
            const int64_t o = (i * 2) * Pp + x;
            double yp = (double)Ypart[o], yq = (double)Ypart[o + Pp];
            for (int s = 1; s < S; ++s) {
                yp += (double)Ypart[s * len + o];
                yq += (double)Ypart[s * len + o + Pp];
            }
            // the self pair, left out of the contraction (FP64)
            const double4 pd = P1[i];
            yp += self_kpp(pd.x, pd.z) * (F[F_W * npad + i] * L[o]);
            point_response(point_fields(F, I, npad, i), L[o], L[o + Pp], yp, yq, Yr, Yg);
        }
        sR[rr][tx] = Yr;
        sG[rr][tx] = Yg;
    }
    __syncthreads();
    const int il = tid & (TRI - 1);
    for (int c = tid / TRI; c < TRX; c += 256 / TRI) {
        const int xx = blockIdx.y * TRX + c;
        const int64_t i = i0 + il;
        if (xx < P && i < n) {
            f_rho_t[(int64_t)xx * n + i] = sR[il][c];
            f_gamma_t[(int64_t)xx * n + i] = sG[il][c];
        }
    }
}

// Hpart[s] (rows 0..Pp-1) = sum over the rows k of slice s of L[k][l] R[k][m];
// row Pp = sum_k L[k][l] wf[k].  NCH = 2: rows k = 2 i + c of (rho^x, gamma^x)
// with wf[2i + c] = w_i (f^rho_i, f^gamma_i); NCH = 1: rows k = i of w^x with
// wf[i] = rho_i (beta + E_i).
// Workgroup (tl, tm, s): output tile of NB x NB 16-column blocks; its eight
// waves take consecutive eighths of the slice, each on v_mfma_f64_16x16x4
// with L and R read straight from memory (A = L^T, B = R, K over rows).  NB
// divides the blocks of Pp evenly, so that few MFMAs run on padding (two
// blocks: four MFMAs a step where a fixed 4 x 4 tile ran sixteen); two waves
// per SIMD, so that one's loads are in flight under the other's MFMAs.
// Against four waves of a fixed 4 x 4 tile: the dimer (Pp 32) 15 -> 8 us, nine
// waters (Pp 96) 51 -> 29, the hexamer (64) 26 -> 22, twenty waters (192) 719
// -> 434 us, 41 TFLOP/s (also from the tiles of a slice sharing one die's L2).
constexpr int kGemmWaves = 8;
inline int gemm_blocks(int nblk) {      // 16-column blocks per tile side
    const int tiles = (nblk + 3) / 4;
    return (nblk + tiles - 1) / tiles;
}
template <int NCH, int NB>
__global__ __launch_bounds__(64 * kGemmWaves) void k_gemm(int64_t n, int64_t npad, int64_t slice,
                                                          int32_t Pp, int32_t tiles, int32_t S,
                                                          const double *__restrict__ F,
                                                          const double *__restrict__ L,
                                                          const double *__restrict__ R,
                                                          double *__restrict__ Hpart) {
    constexpr int W = 16 * NB, HALF = kGemmWaves / 2;
    __shared__ double sT[HALF][W * W + W];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ll = lane & 15, kk = lane >> 4;
    // workgroups b, b + 8, ... run on one die: with a multiple of 8 slices,
    // all tiles of a slice go to one, whose L2 then holds the slice's rows once
    const int T2 = tiles * tiles, b = blockIdx.x;
    const int s = S % 8 == 0 ? b % 8 + 8 * (b / 8 / T2) : b / T2;
    const int tile = S % 8 == 0 ? b / 8 % T2 : b % T2;
    const int tl = tile / tiles, tm = tile - tl * tiles;
    const int l0 = tl * W, m0 = tm * W;
    const bool grad = tm == 0;
    const int nlb = min(NB, (Pp - l0) / 16), nmb = min(NB, (Pp - m0) / 16);   // Pp % 16 == 0
    const int64_t rows = NCH * n;
    const int64_t sb = min(rows, (int64_t)s * slice * NCH), se = min(rows, sb + slice * NCH);
    const int64_t q = (se - sb + kGemmWaves - 1) / kGemmWaves;
    const int64_t rb = min(se, sb + wave * q), re = min(se, rb + q);
    v4d acc[NB][NB];
    double gacc[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a) {
        gacc[a] = 0.0;
#pragma unroll
        for (int c = 0; c < NB; ++c) acc[a][c] = (v4d){0.0, 0.0, 0.0, 0.0};
    }
    // several k steps per iteration, their loads issued before their MFMAs; the
    // MFMAs of each accumulator run in k order.  As many as the loop's registers
    // hold: four blocks a side take two steps (twenty waters 434 us; one step 500,
    // four, which spill in the loop, 484).  The 24 registers that they do spill
    // are in the reduction below, once a workgroup.
    constexpr int ST = NB <= 2 ? 8 : NB == 3 ? 4 : 2;
    for (int64_t k00 = rb; k00 < re; k00 += 4 * ST) {
        // loads without branches, from clamped in-range addresses (finite
        // values); rows past the slice and columns past Pp are zeroed by a
        // multiplication, so that no load waits for another
        double av[ST][NB], bv[ST][NB], wa[ST], wb[ST];
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            const int64_t k = k00 + 4 * st + kk;
            const bool ok = k < re;
            const int64_t kr = ok ? k : rb;
            const double on = ok ? 1.0 : 0.0;
#pragma unroll
            for (int a = 0; a < NB; ++a)
                av[st][a] = L[kr * Pp + min(l0 + 16 * a, Pp - 16) + ll] * (a < nlb ? on : 0.0);
#pragma unroll
            for (int c = 0; c < NB; ++c)
                bv[st][c] = R[kr * Pp + min(m0 + 16 * c, Pp - 16) + ll] * (c < nmb ? on : 0.0);
            if (NCH == 2) {
                const int64_t pt = kr >> 1;
                wa[st] = F[F_W * npad + pt] * on;
                wb[st] = F[((kr & 1) ? F_FG : F_FR) * npad + pt];
            } else {
                wa[st] = F[F_F0 * npad + kr] * on;
                wb[st] = 1.0;
            }
        }
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            const double wf = NCH == 2 ? wa[st] * wb[st] : wa[st];
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int c = 0; c < NB; ++c)
                    acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[st][a], bv[st][c], acc[a][c],
                                                                     0, 0, 0);
            if (grad)
#pragma unroll
                for (int a = 0; a < NB; ++a) gacc[a] = __builtin_fma(av[st][a], wf, gacc[a]);
        }
    }
    // gradient: sum the four k lanes of each column
#pragma unroll
    for (int a = 0; a < NB; ++a) {
        gacc[a] += __shfl_xor(gacc[a], 16, 64);
        gacc[a] += __shfl_xor(gacc[a], 32, 64);
    }
    // D layout of v_mfma_f64_16x16x4 (measured on gfx950): item r of lane l
    // holds row 4 r + l/16, column l%16 of the 16 x 16 block.  The upper four
    // waves' sums are added to the lower four's, those then in wave order.
    auto row = [&](int a, int r) { return sT[wave % HALF] + (16 * a + 4 * r + kk) * W + ll; };
    auto put = [&]() {
#pragma unroll
        for (int a = 0; a < NB; ++a) {
#pragma unroll
            for (int c = 0; c < NB; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) row(a, r)[16 * c] = acc[a][c][r];
            if (kk == 0) sT[wave % HALF][W * W + 16 * a + ll] = gacc[a];
        }
    };
    if (wave >= HALF) put();
    __syncthreads();
    if (wave < HALF) {
#pragma unroll
        for (int a = 0; a < NB; ++a) {
#pragma unroll
            for (int c = 0; c < NB; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[a][c][r] += row(a, r)[16 * c];
            if (kk == 0) gacc[a] += sT[wave % HALF][W * W + 16 * a + ll];
            mem_order();                // one row of blocks' loads at a time
        }
        put();
    }
    __syncthreads();
    double *H = Hpart + (int64_t)s * (Pp + 1) * Pp;
    for (int e = tid; e < W * W + (grad ? W : 0); e += 64 * kGemmWaves) {
        double v = sT[0][e];
#pragma unroll
        for (int w = 1; w < HALF; ++w) v += sT[w][e];
        const int rr = e / W, cc = e - rr * W;
        if (rr < W) {
            if (l0 + rr < Pp && m0 + cc < Pp) H[(int64_t)(l0 + rr) * Pp + m0 + cc] = v;
        } else if (l0 + cc < Pp) {
            H[(int64_t)Pp * Pp + l0 + cc] = v;
        }
    }
}

template <int NCH>
void gemm_launch(const vv10_plan *p, const Workspace &ws, const double *L, const double *R,
                 double *Hpart) {
    const int nblk = ws.Pp / 16, nb = gemm_blocks(nblk), tiles = (nblk + nb - 1) / nb;
    const int64_t slice = (p->n + ws.gsplit - 1) / ws.gsplit;
    auto go = [&](auto c) {
        k_gemm<NCH, decltype(c)::value><<<(unsigned)(tiles * tiles * ws.gsplit), 64 * kGemmWaves, 0,
                                          p->stream>>>(p->n, p->npad, slice, ws.Pp, tiles,
                                                       ws.gsplit, p->F, L, R, Hpart);
    };
    if (nb == 1) go(std::integral_constant<int, 1>{});
    else if (nb == 2) go(std::integral_constant<int, 2>{});
    else if (nb == 3) go(std::integral_constant<int, 3>{});
    else go(std::integral_constant<int, 4>{});
}

// Workgroups b < nh: Hsum[e] = sum_s Hpart[s][e], e < len = (Pp + 1) Pp, over
// the S slices of Hpart and then the S2 slices of H2: 64 entries each, 16 waves
// per 64 entries, each over a sixteenth of the slices, so that the few
// workgroups of a small Hessian keep enough loads in flight; the waves' sums
// are added in wave order.
// Workgroups b >= nh: DS[A][B][c] = sum over the tiles t of atom A of
// Dpart[t][B][c] (tile order), one thread each.  Two independent reductions of
// a few us, bound by latency: one launch instead of two.
constexpr int kSumWaves = 16;
__global__ __launch_bounds__(64 * kSumWaves) void k_sums(
    int64_t len, int S, const double *__restrict__ Hpart, int S2, const double *__restrict__ H2,
    double *__restrict__ Hsum, int nh, int32_t n_atom, const int32_t *__restrict__ tile_first,
    const double *__restrict__ Dpart, double *__restrict__ DS) {
    __shared__ double part[kSumWaves][64];
    if ((int)blockIdx.x >= nh) {
        const int64_t k = (int64_t)(blockIdx.x - nh) * (64 * kSumWaves) + threadIdx.x;
        if (k >= (int64_t)n_atom * n_atom * 9) return;
        const int A = (int)(k / (9LL * n_atom));
        const int rem = (int)(k - (int64_t)A * 9 * n_atom);   // B * 9 + c
        // the own-atom slot (B = A) is never formed by the grid pass (its terms
        // follow from translational invariance in k_finish): zero, not read
        if (rem / 9 == A) {
            DS[k] = 0.0;
            return;
        }
        double v = 0.0;
#pragma unroll 8
        for (int t = tile_first[A]; t < tile_first[A + 1]; ++t)
            v += Dpart[(int64_t)t * n_atom * 9 + rem];
        DS[k] = v;
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t e = (int64_t)blockIdx.x * 64 + lane;
    const int St = S + S2;
    const int q = (St + kSumWaves - 1) / kSumWaves;
    const int sb = min(St, wave * q), se = min(St, sb + q);
    double a = 0.0;
    if (e < len)
#pragma unroll 16
        for (int s = sb; s < se; ++s)
            a += s < S ? Hpart[(int64_t)s * len + e] : H2[(int64_t)(s - S) * len + e];
    part[wave][lane] = a;
    __syncthreads();
    if (wave == 0 && e < len) {
        double t = part[0][lane];
#pragma unroll
        for (int w = 1; w < kSumWaves; ++w) t += part[w][lane];
        Hsum[e] = t;
    }
}

__device__ __forceinline__ int sym_index(int a, int b) {
    if (a == b) return a;                 // xx, yy, zz
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    return lo == 0 ? (hi == 1 ? 3 : 4) : 5;   // xy, xz, yz
}

// E_{gr,gr}[(A,a)][(B,b)] = DS[A][B][(a,b)] for B != A; the diagonal blocks
// are -sum_{C != A} DS[A][C][(a,b)] (translational invariance).  The D sums
// are symmetric in the atom pair and formed for A < B only.
__device__ __forceinline__ double dsym(int32_t n_atom, const double *__restrict__ DS, int A, int B,
                                       int c) {
    const int lo = A < B ? A : B, hi = A < B ? B : A;
    return DS[((int64_t)lo * n_atom + hi) * 9 + c];
}

__device__ __forceinline__ double egrgr(int32_t n_atom, const double *__restrict__ DS, int A, int B,
                                        int c) {
    if (A != B) return dsym(n_atom, DS, A, B, c);
    // every load issued (the C = A entry is read and discarded), so that
    // they are in flight together
    double v = 0.0;
#pragma unroll 8
    for (int C = 0; C < n_atom; ++C) {
        const double d = dsym(n_atom, DS, A, C, c);
        v -= C != A ? d : 0.0;
    }
    return v;
}

// Threads k < P^2: hess[l][m]; threads P^2 <= k < P^2 + P: grad[k - P^2].
__global__ __launch_bounds__(256) void k_finish(int32_t n_atom, int32_t P, int32_t Pp,
                                                const double *__restrict__ Hsum,
                                                const double *__restrict__ DS,
                                                double *hess, double *__restrict__ grad,
                                                const BatchBuffers *__restrict__ io) {
    if (io) hess = global_ptr(io->hess);
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t PP = (int64_t)P * P;
    if (k < PP) {
        if (!hess) return;
        const int l = (int)(k / P), m = (int)(k % P);
        const int A = l / 3, a = l % 3, B = m / 3, b = m % 3;
        const int c = sym_index(a, b);
        const double glm = egrgr(n_atom, DS, A, B, c), gml = egrgr(n_atom, DS, B, A, c);
        hess[k] = 0.5 * (Hsum[(int64_t)l * Pp + m] + Hsum[(int64_t)m * Pp + l]) + 0.5 * (glm + gml);
    } else if (grad && k < PP + P) {
        const int x = (int)(k - PP);
        const int A = x / 3, a = x % 3;
        double gr = 0.0;
        // sum_{i in A} a_i E^{Bgr}_i, formed for B > A; for B < A it is
        // minus the (B, A) sum (a_i e_ij symmetric, d_ij = -d_ji)
#pragma unroll 8
        for (int B = 0; B < n_atom; ++B) {
            const double d = B > A ? DS[((int64_t)A * n_atom + B) * 9 + 6 + a]
                                   : -DS[((int64_t)B * n_atom + A) * 9 + 6 + a];
            gr -= B != A ? d : 0.0;
        }
        grad[x] = Hsum[(int64_t)Pp * Pp + x] + gr;
    }
}

}  // namespace

namespace {

// Gradient (Section II.A, first form of the grid part): for x = 3 A + a,
//   grad[x] = sum_i w_i (f^rho_i rho^x_i + f^gamma_i gamma^x_i)
//           [+ sum_i w^x_i rho_i (beta + E_i)]
//           - sum_{B > A} sum_{tiles t of A} Gpart[t][B][a]
//           + sum_{B < A} sum_{tiles t of B} Gpart[t][A][a]
// (the tile sums are antisymmetric in the atom pair; the pass forms B > A),
// gamma^x = 2 grad rho . grad rho^x; w^x (optional) with the owner slot from
// Wown.  The point sums run over S slices of the points, one workgroup per
// (atom, slice) for the atom's three directions, whose per-point fields it
// reads once: bound by the 32 N P bytes of the derivatives.  The
// hexamer (47 MB): 13.0 + 4.6 us, against 48 with one workgroup per x.
// Grids of at most kGradOneSlice points take one slice, whose workgroups add the
// tile sums as well: the second launch costs more than the slices save there (a
// kept plan of one water, N 150: 8.7 -> 5.9 us; of four, N 720: 8.7 -> 6.2).
// Fixed-order tree reductions throughout.
constexpr int kGradSlices = 32, kGradOneSlice = 1024;

// This lane's share of the tile sums of x = 3 A + a: -sum_{B != A} sum_{t in A}
// Gpart[t][B]; the pass forms B > A, and a B < A term is minus the (B, A) one,
// i.e. +Gpart[t][A] over the tiles t of B.
__device__ __forceinline__ double tile_terms(int32_t n_atom, int A, int a, int lane,
                                             const int32_t *__restrict__ tile_first,
                                             const double *__restrict__ Gpart) {
    double v = 0.0;
    const int t0 = tile_first[A], nt = tile_first[A + 1] - t0;
#pragma unroll 8
    for (int k = lane; k < (n_atom - A - 1) * nt; k += 64) {
        const int B = A + 1 + k / nt, t = t0 + k % nt;
        v -= Gpart[((int64_t)t * n_atom + B) * 3 + a];
    }
#pragma unroll 8
    for (int t = lane; t < t0; t += 64) v += Gpart[((int64_t)t * n_atom + A) * 3 + a];
    return v;
}

// ONE: one slice, a workgroup per direction x (three times as many), grad is
// written; else the slice's sums go to part.
template <bool ONE>
__global__ __launch_bounds__(256) void k_gradient_points(int64_t n, int64_t npad, int64_t slice,
                                                         int32_t n_atom,
                                                         const int32_t *__restrict__ atom_of,
                                                         const double *__restrict__ F,
                                                         const double *__restrict__ rho_x,
                                                         const double *__restrict__ grad_rho_x,
                                                         const double *__restrict__ w_x,
                                                         const double *__restrict__ Wown,
                                                         const int32_t *__restrict__ tile_first,
                                                         const double *__restrict__ Gpart,
                                                         double *__restrict__ part,
                                                         double *__restrict__ grad) {
    constexpr int ND = ONE ? 1 : 3;     // directions of the workgroup
    __shared__ double red[ND][4];
    const int tid = threadIdx.x;
    const int A = ONE ? blockIdx.x / 3 : blockIdx.x, a0 = ONE ? blockIdx.x % 3 : 0;
    double tiles = 0.0;                 // of the first wave
    if (ONE && tid < 64) tiles = tile_terms(n_atom, A, a0, tid, tile_first, Gpart);
    const int64_t end = min(n, (int64_t)(blockIdx.y + 1) * slice);
    double s[ND] = {};
#pragma unroll 2
    for (int64_t i = (int64_t)blockIdx.y * slice + tid; i < end; i += 256) {
        const double w = F[F_W * npad + i], fr = w * F[F_FR * npad + i];
        const double fg = 2.0 * (w * F[F_FG * npad + i]);
        const double gx = F[F_GX * npad + i], gy = F[F_GY * npad + i], gz = F[F_GZ * npad + i];
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            const int a = a0 + k;
            const int64_t o = (int64_t)(3 * A + a) * n + i;
            const double *d = grad_rho_x + 3 * o;
            s[k] += fr * rho_x[o] + fg * (gx * d[0] + gy * d[1] + gz * d[2]);
            if (w_x) {
                const double wx = atom_of[i] == A ? Wown[i * 3 + a] : w_x[o];
                s[k] += wx * F[F_F0 * npad + i];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < ND; ++k) {
        s[k] = wave_sum(s[k]);
        if ((tid & 63) == 0) red[k][tid >> 6] = s[k];
    }
    if (ONE && tid < 64) tiles = wave_sum(tiles);
    __syncthreads();
    if (tid < ND) {
        const double v = red[tid][0] + red[tid][1] + red[tid][2] + red[tid][3];
        if (ONE) grad[3 * A + a0] = v + tiles;
        else part[(int64_t)blockIdx.y * 3 * n_atom + 3 * A + tid] = v;
    }
}

// The slices' point sums and the tile sums: one wave per x.
__global__ __launch_bounds__(64) void k_gradient(int32_t n_atom, int S,
                                                 const int32_t *__restrict__ tile_first,
                                                 const double *__restrict__ part,
                                                 const double *__restrict__ Gpart,
                                                 double *__restrict__ grad) {
    const int lane = threadIdx.x, x = blockIdx.x, A = x / 3, a = x % 3;
    double v = 0.0;
    for (int s = lane; s < S; s += 64) v += part[(int64_t)s * 3 * n_atom + x];
    v += tile_terms(n_atom, A, a, lane, tile_first, Gpart);
    v = wave_sum(v);
    if (lane == 0) grad[x] = v;
}

}  // namespace

// Slices of k_gradient_points: their sums go where the atom groups' partial
// integrals were (gw.Igrp, [bgroups][3][npad], which the potential has added).
static int gradient_slices(const vv10_plan *p) {
    if (p->n <= kGradOneSlice) return 1;
    const int64_t room = (int64_t)p->gw.bgroups * p->npad / p->n_atom;
    return (int)std::max<int64_t>(1, std::min<int64_t>({kGradSlices, room, (p->n + 255) / 256}));
}

hipError_t launch_gradient(vv10_plan *p, const double *rho_x, const double *grad_rho_x,
                           const double *w_x, double *grad) {
    if (w_x) {
        const hipError_t e = launch_weight_own(p, w_x, p->wown);
        if (e != hipSuccess) return e;
    }
    const int S = gradient_slices(p);
    const int64_t slice = (p->n + S - 1) / S;
    double *part = p->gw.Igrp;
    if (p->n <= kGradOneSlice) {
        k_gradient_points<true><<<(unsigned)(3 * p->n_atom), 256, 0, p->stream>>>(
            p->n, p->npad, slice, p->n_atom, p->atom_of, p->F, rho_x, grad_rho_x, w_x, p->wown, p->d_tile_first,
            p->gw.Gpart, part, grad);
        return hipGetLastError();
    }
    k_gradient_points<false><<<dim3((unsigned)p->n_atom, (unsigned)S), 256, 0, p->stream>>>(
        p->n, p->npad, slice, p->n_atom, p->atom_of, p->F, rho_x, grad_rho_x, w_x, p->wown,
        p->d_tile_first, p->gw.Gpart, part, grad);
    k_gradient<<<(unsigned)(3 * p->n_atom), 64, 0, p->stream>>>(p->n_atom, S, p->d_tile_first, part,
                                                                p->gw.Gpart, grad);
    return hipGetLastError();
}

hipError_t launch_trial_response(vv10_plan *p, double *f_rho_t, double *f_gamma_t) {
    const Workspace &ws = p->rws;
    dim3 grid((unsigned)((p->n + TRI - 1) / TRI), (unsigned)((ws.P + TRX - 1) / TRX));
    auto go = [&](auto *ypart) {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(ypart)>>;
        k_trial_resp<T><<<grid, 256, 0, p->stream>>>(
            p->n, p->npad, ws.P, ws.Pp, ws.jsplit, p->P1, p->F, p->Ir, ws.L, ypart, f_rho_t,
            f_gamma_t);
    };
    if (partial_elem(p->prec, p->npad, ws.jlen) == sizeof(float)) go(static_cast<const float *>(ws.Ypart));
    else go(static_cast<const double *>(ws.Ypart));
    return hipGetLastError();
}

hipError_t launch_assemble(vv10_plan *p, const vv10_nuclear_outputs &out, bool weighted,
                           const BatchBuffers *io) {
    const Workspace &ws = p->ws;
    const WeightWork &ww = p->ww;
    const int64_t n = p->n;
    double *hess = out.hess, *grad = out.grad;
    {
        const unsigned nb = (unsigned)((n + 3) / 4);
        auto go = [&](auto *ypart) {
            using T = std::remove_const_t<std::remove_pointer_t<decltype(ypart)>>;
            const WeightIn<T> wt = {static_cast<const T *>(ww.Ypart), ww.Lw, ww.Ze, ww.Rw};
            if (weighted)
                k_resp<T, true><<<nb, 256, 0, p->stream>>>(
                    n, p->npad, ws.P, ws.Pp, ws.jsplit, p->atom_of, p->P1, p->F, p->I, ws.L, ypart,
                    ws.Y, ws.Z, wt, out.resp_rho, out.resp_gamma, out.fock_rho, out.fock_gamma);
            else
                k_resp<T, false><<<nb, 256, 0, p->stream>>>(
                    n, p->npad, ws.P, ws.Pp, ws.jsplit, p->atom_of, p->P1, p->F, p->I, ws.L, ypart,
                    ws.Y, ws.Z, wt, out.resp_rho, out.resp_gamma, out.fock_rho, out.fock_gamma);
        };
        if (partial_elem(p->prec, p->npad, ws.jlen) == sizeof(float)) go(static_cast<const float *>(ws.Ypart));
        else go(static_cast<const double *>(ws.Ypart));
    }
    if (!hess && !grad && !io) return hipGetLastError();
    gemm_launch<2>(p, ws, ws.L, ws.Y, ws.Hpart);
    if (weighted) gemm_launch<1>(p, ws, ww.Lw, ww.Rw, ww.Hpart);
    {
        const int64_t len = (int64_t)(ws.Pp + 1) * ws.Pp;
        const int64_t nds = (int64_t)p->n_atom * p->n_atom * 9;
        const int nh = (int)((len + 63) / 64), nd = (int)((nds + 64 * kSumWaves - 1) / (64 * kSumWaves));
        k_sums<<<(unsigned)(nh + nd), 64 * kSumWaves, 0, p->stream>>>(
            len, ws.gsplit, ws.Hpart, weighted ? ws.gsplit : 0, ww.Hpart, ws.Hsum, nh, p->n_atom,
            p->d_tile_first, ws.Dpart, ws.DS);
    }
    const int64_t nt = (int64_t)ws.P * ws.P + ws.P;
    k_finish<<<(unsigned)((nt + 255) / 256), 256, 0, p->stream>>>(p->n_atom, ws.P, ws.Pp, ws.Hsum,
                                                                  ws.DS, hess, grad, io);
    return hipGetLastError();
}

}  // namespace vv10
