// Pair kernel: the inner integrals of Section II.A (E_i, U_i, W_i) and,
// in Hessian mode, those of Section II.B (A_i, B_i, C_i):
//   E_i = sum_j a_j Phi_ij
//   U_i = -sum_j a_j Phi_ij h_ij,           h = 1/(g+g') + 1/g
//   W_i = -sum_j a_j Phi_ij R^2 h_ij
//   {A,B,C}_i = sum_j 2 a_j Phi_ij (R^2)^{0,1,2} m_ij,
//                                        m = 1/(g+g')^2 + 1/((g+g')g) + 1/g^2
// with a_j = w_j rho_j and every j (j = i included: its term is added in
// FP64, the loops run over j != i).  One lane owns one
// outer point i; j points stream through LDS and are read as wave-wide
// broadcasts.  All 1/g, 1/g', 1/(g+g') come from one reciprocal
// r = 1/(g g' (g+g')); the loop sums p = a_j r times h, R^2 h and
// m (R^2)^{0,1,2} (m = h^2 - 1/((g+g') g)), and the constant factors
// (a_j Phi = -3/2 p) are applied to the sums.
#include <algorithm>

#include "dev_common.h"
#include "vv10_internal.h"

namespace vv10 {

namespace {

constexpr int JC = 256;   // j points staged per block step; wave w takes [64 w, 64 w + 64)
// Workgroups that the j splits aim at.  The pass is bound by VALU issue (91 %
// busy); with 2048, one round of resident workgroups, the few that are left
// over ran a second one alone: hexamer 0.360 -> 0.330 ms in FP32 and 0.717 ->
// 0.662 in FP64, 17 waters (N = 101949) 4.50 -> 4.14 in FP32; 4096: 0.334,
// 0.683 and 4.27; 16384: 0.330, 0.670 and 4.23.
constexpr int kPairBlocks = 8192;

// Sums of one wave's 64 j of an LDS chunk.  SELF: the chunk holds the
// outer points themselves (lane l's own point at jj = jself), whose pair is
// left out (added in FP64 at the end).
template <typename T, typename T4, bool HESS, bool SELF>
__device__ __forceinline__ void pair_run(const T4 a0, const T4 a1, const T4 *s0, const T4 *s1,
                                         int jbeg, int jself, T *c) {
#pragma unroll 8
    for (int jj = jbeg; jj < jbeg + 64; ++jj) {
        const T4 b0 = s0[jj], b1 = s1[jj];
        const T dx = a0.x - b0.x, dy = a0.y - b0.y, dz = a0.z - b0.z;
        const T R2 = dx * dx + dy * dy + dz * dz;
        const T g = a0.w * R2 + a1.x;
        const T gp = b0.w * R2 + b1.x;
        const T s = g + gp, t = g * gp;
        T r;
        if constexpr (sizeof(T) == 8) r = rcp64(t * s); else r = rcp32(t * s);
        T pj = b1.y * r;
        if (SELF) pj = jj == jself ? T(0) : pj;
        T ig, is, h;
        if constexpr (sizeof(T) == 8 && !HESS) {
            h = (gp * r) * (s + g);   // 1/g + 1/s without forming either
        } else {
            ig = gp * (s * r);
            is = t * r;
            h = ig + is;
        }
        const T ph = pj * h;
        c[0] += pj;
        c[1] += ph;
        c[2] += ph * R2;
        if (HESS) {
            const T pm = pj * (h * h - is * ig);
            const T pmR2 = pm * R2;
            c[3] += pm;
            c[4] += pmR2;
            c[5] += pmR2 * R2;
        }
    }
}

// One workgroup = 4 waves sharing 64 outer points (one per lane); each wave
// takes a quarter of every 256-point j chunk, and the four partial sums are
// added in wave order at the end.  blockIdx.y selects a contiguous j range
// (a split); splits write partial integrals [split][6][npad] that
// k_potential (E, U, W) or k_sum_integrals (all six) adds in split order.  Mixed mode evaluates in FP32 and
// adds each 64-point run into FP64 accumulators.  The self pair is left out
// of the loops; the split that holds the outer points adds it in FP64 from
// the FP64 point data Pd (kappa, a = w rho).
template <typename T, typename T4, bool HESS>
__global__ __launch_bounds__(256) void k_pair(int64_t npad, int64_t jlen,
                                              const T4 *__restrict__ P0,
                                              const T4 *__restrict__ P1,
                                              const double4 *__restrict__ Pd,
                                              double *__restrict__ Ipart) {
    __shared__ T4 s0[JC], s1[JC];
    __shared__ double red[4][6][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t tb = (int64_t)blockIdx.x * 64;
    const int64_t i = tb + lane;
    const int64_t jbeg = (int64_t)blockIdx.y * jlen;
    const int64_t jend = min(npad, jbeg + jlen);
    const T4 a0 = P0[i], a1 = P1[i];
    double E = 0, U = 0, W = 0, A = 0, B = 0, C = 0;
    for (int64_t j0 = jbeg; j0 < jend; j0 += JC) {
        __syncthreads();
        s0[threadIdx.x] = P0[j0 + threadIdx.x];
        s1[threadIdx.x] = P1[j0 + threadIdx.x];
        __syncthreads();
        T c[6] = {0, 0, 0, 0, 0, 0};
        if (j0 + 64 * wave == tb)   // this wave's run holds the outer points
            pair_run<T, T4, HESS, true>(a0, a1, s0, s1, 64 * wave, 64 * wave + lane, c);
        else
            pair_run<T, T4, HESS, false>(a0, a1, s0, s1, 64 * wave, 0, c);
        E += (double)c[0];
        U += (double)c[1];
        W += (double)c[2];
        if (HESS) {
            A += (double)c[3];
            B += (double)c[4];
            C += (double)c[5];
        }
    }
    red[wave][0][lane] = E;
    red[wave][1][lane] = U;
    red[wave][2][lane] = W;
    red[wave][3][lane] = A;
    red[wave][4][lane] = B;
    red[wave][5][lane] = C;
    __syncthreads();
    const int nout = HESS ? 6 : 3;
    // self pair (W, B, C have a factor R^2 and get none): E += a Phi,
    // U += -a Phi h, A += 2 a Phi m
    const bool own = tb >= jbeg && tb < jend;
    double self[6] = {0, 0, 0, 0, 0, 0};
    if (own) {
        const double4 pd = Pd[i];
        const SelfPair q = self_pair(pd.x);
        self[0] = pd.y * q.phi;
        self[1] = -pd.y * q.phi * q.h;
        self[3] = 2.0 * pd.y * q.phi * q.m;
    }
    for (int k = wave; k < nout; k += 4) {
        const double sc = k == 0 ? -1.5 : (k < 3 ? 1.5 : -3.0);   // E; U, W; A, B, C
        const double v = sc * (red[0][k][lane] + red[1][k][lane] + red[2][k][lane] + red[3][k][lane]);
        Ipart[((int64_t)blockIdx.y * NI + k) * npad + i] = v + self[k];
    }
}

// I[k][i] = sum over splits of Ipart[s][k][i], in split order.
__global__ __launch_bounds__(256) void k_sum_integrals(int64_t npad, int nout, int S,
                                                       const double *__restrict__ Ipart,
                                                       double *__restrict__ I) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)nout * npad) return;
    const int k = (int)(e / npad);
    const int64_t i = e - (int64_t)k * npad;
    double a = 0.0;
#pragma unroll 8
    for (int s = 0; s < S; ++s) a += Ipart[((int64_t)s * NI + k) * npad + i];
    I[k * npad + i] = a;
}

// a += q[s step], and with R = 2 b += q[s step + row], over s < S in order, the
// loads of T partials issued together.  The last T are loaded without branches
// (past the end the last one again, added as zero): in a loop of their own they
// cost a wait each (18 groups of the hexamer, kernel 19.3 -> 13.8 us; 36 of 12
// waters, N 7200, 26.5 -> 16.6; 90 of 30, N 5400, 72 -> 25).  T follows S, as a
// load of nothing still takes its turn (three groups of one water by fours 7.9 us,
// by eights 8.8).
template <int T, int R>
__device__ __forceinline__ void add_parts_by(const double *__restrict__ q, int64_t step, int64_t row,
                                             int S, double &a, double &b) {
    for (int s0 = 0; s0 < S; s0 += T) {
        double u[T], v[T];
#pragma unroll
        for (int k = 0; k < T; ++k) {
            const double *p = q + min(s0 + k, S - 1) * step;
            u[k] = p[0];
            if (R == 2) v[k] = p[row];
        }
#pragma unroll
        for (int k = 0; k < T; ++k) {
            a += s0 + k < S ? u[k] : 0.0;
            if (R == 2) b += s0 + k < S ? v[k] : 0.0;
        }
    }
}

template <int R>
__device__ __forceinline__ void add_parts(const double *__restrict__ q, int64_t step, int64_t row,
                                          int S, double &a, double &b) {
    if (S > 8) add_parts_by<16, R>(q, step, row, S, a, b);
    else if (S > 4) add_parts_by<8, R>(q, step, row, S, a, b);
    else add_parts_by<4, R>(q, step, row, S, a, b);
}

// Potential and energy terms (Section II.A):
//   f^rho_i = beta + E_i + rho_i (kappa_r U_i + omega_r W_i)
//   f^gamma_i = rho_i omega_g W_i
//   energy = sum_i a_i (beta + E_i/2), reduced per block in a fixed order; the
// block that finishes last adds the block sums, in block order.
// 256 points per block.  With partial integrals, 768 threads: thread 256 r + t
// adds rows k0 + r (and k0 + 3 + r) of point t over the splits, in order, so
// that even a small grid keeps all its loads in flight.  Latency bounds it:
// one launch in place of three (sum, potential, energy) takes 7.3 us
// in the place of 13.3 for six rows of the dimer (N 4200, six atom groups).
__global__ __launch_bounds__(768) void k_potential(int64_t n, int64_t npad, double beta,
                                                   IntegralParts ip,
                                                   const double4 *__restrict__ P1,
                                                   double *__restrict__ F, double *__restrict__ I,
                                                   double *__restrict__ f_rho,
                                                   double *__restrict__ f_gamma, double *epart,
                                                   uint32_t *counter, double *energy,
                                                   const int32_t *__restrict__ valid,
                                                   const BatchBuffers *__restrict__ io) {
    __shared__ double sI[3][256];
    __shared__ double s[256];
    __shared__ bool last;
    if (valid && *valid != 0) return;   // invalid inputs: no output is written
    const int t = threadIdx.x & 255, r = threadIdx.x >> 8;
    const int64_t i = (int64_t)blockIdx.x * 256 + t;
    // issued ahead of the sums, which they do not depend on
    double rh = 0.0, kar = 0.0, omr = 0.0, omg = 0.0, ai = 0.0;
    if (r == 0 && i < n) {
        rh = F[F_RHO * npad + i];
        kar = F[F_KAR * npad + i];
        omr = F[F_OMR * npad + i];
        omg = F[F_OMG * npad + i];
        ai = P1[i].y;
    }
    if (ip.nk > 0) {
        if (i < n) {
            const int64_t step = (int64_t)ip.rows * npad;
            const double *q = ip.part + (int64_t)(ip.k0 + r) * npad + i;
            double a = 0.0, b = 0.0;
            if (ip.nk == 6) {
                add_parts<2>(q, step, 3 * npad, ip.S, a, b);
                I[(r + 3) * npad + i] = b;
            } else {
                add_parts<1>(q, step, 0, ip.S, a, b);
            }
            I[(ip.k0 + r) * npad + i] = a;
            sI[r][t] = ip.k0 == 0 ? a : I[r * npad + i];
        }
    } else if (i < n) {
        for (int k = 0; k < 3; ++k) sI[k][t] = I[k * npad + i];
    }
    __syncthreads();
    if (r == 0) {
        double e = 0.0;
        if (i < n) {
            const double Ei = sI[I_E][t], Ui = sI[I_U][t], Wi = sI[I_W][t];
            const double fr = beta + Ei + rh * (kar * Ui + omr * Wi);
            const double fg = rh * omg * Wi;
            F[F_FR * npad + i] = fr;
            F[F_FG * npad + i] = fg;
            F[F_F0 * npad + i] = rh * (beta + Ei);
            if (f_rho) f_rho[i] = fr;
            if (f_gamma) f_gamma[i] = fg;
            e = ai * (beta + 0.5 * Ei);
        }
        s[t] = e;
    }
    auto tree = [&]() {                 // s[0] = sum of s[0..256)
        __syncthreads();
        for (int off = 128; off > 0; off >>= 1) {
            if (threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
            __syncthreads();
        }
    };
    tree();
    if (threadIdx.x == 0) {
        // The block sum is exchanged into place: once its old value is back the
        // sum is at the device's point of coherence, and only then is the block
        // counted (the count waits for the value).  A release fence instead
        // would write back this die's whole L2, which the molecules of a batch
        // share (4.20 -> 4.19 ms there).
        double old = __hip_atomic_exchange(&epart[blockIdx.x], s[0], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" : "+v"(old) : : "memory");
        __builtin_amdgcn_s_waitcnt(0);
        const uint32_t before =
            __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = before + 1 == gridDim.x;
        if (last) *counter = 0;         // as the next call finds it
    }
    __syncthreads();
    if (!last) return;
    if (r == 0) {
        double a = 0.0;
        // each thread sums a contiguous run so the order is fixed
        const int64_t nb = gridDim.x, per = (nb + 255) / 256;
        for (int64_t k = t * per; k < min(nb, (int64_t)(t + 1) * per); ++k)
            a += __hip_atomic_load(&epart[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s[t] = a;
    }
    tree();
    if (threadIdx.x == 0) (io ? global_ptr(io->energy) : energy)[0] = s[0];
}

}  // namespace

namespace {

// j points of each of S splits (whole chunks).
int64_t pair_jlen(int64_t npad, int S) { return ((npad / S + JC - 1) / JC) * JC; }

}  // namespace

int pair_splits(int64_t npad, int32_t n_atom) {
    const int64_t blocks = npad / 64;
    int S = (int)std::min<int64_t>(16, std::max<int64_t>(1, (kPairBlocks + blocks - 1) / blocks));
    // a grid that fits vv10_energy_potential_noalloc's scratch without
    // partials keeps fitting (about 268 bytes a point and 4 an atom besides
    // them), and both paths split alike
    const int64_t scratch = VV10_NOALLOC_SCRATCH_BYTES, rest = 268 * npad + 4 * (int64_t)n_atom;
    if (rest <= scratch)
        while (S > 1 && rest + 8 * NI * S * npad > scratch - (1 << 20)) --S;
    while (S > 1 && npad / S < JC) --S;
    // no empty split: whole chunks a split can cover the grid with fewer (the
    // dimer, N 4200, 17 chunks: two a split, nine of sixteen splits)
    const int64_t jlen = pair_jlen(npad, S);
    return (int)((npad + jlen - 1) / jlen);
}

namespace {

void pair_launch(vv10_plan *p, bool six, double *I_out, IntegralParts *parts) {
    const int S = pair_splits(p->npad, p->n_atom);
    const int64_t jlen = pair_jlen(p->npad, S);
    dim3 grid((unsigned)(p->npad / 64), (unsigned)S);
    double *Ipart = S == 1 ? I_out : p->Ipart;
    if (p->prec == VV10_FP64) {
        if (six)
            k_pair<double, double4, true><<<grid, 256, 0, p->stream>>>(p->npad, jlen, p->P0, p->P1,
                                                                       p->P1, Ipart);
        else
            k_pair<double, double4, false><<<grid, 256, 0, p->stream>>>(p->npad, jlen, p->P0, p->P1,
                                                                        p->P1, Ipart);
    } else {
        if (six)
            k_pair<float, float4, true><<<grid, 256, 0, p->stream>>>(p->npad, jlen, p->P0f, p->P1f,
                                                                     p->P1, Ipart);
        else
            k_pair<float, float4, false><<<grid, 256, 0, p->stream>>>(p->npad, jlen, p->P0f, p->P1f,
                                                                      p->P1, Ipart);
    }
    *parts = S > 1 ? IntegralParts{Ipart, S, NI, 0, six ? 6 : 3} : IntegralParts{};
}

}  // namespace

hipError_t launch_pair_integrals(vv10_plan *p, IntegralParts *parts) {
    pair_launch(p, false, p->I, parts);
    return hipGetLastError();
}

hipError_t launch_pair_integrals6(vv10_plan *p, double *I_out) {
    IntegralParts parts;
    pair_launch(p, true, I_out, &parts);
    if (parts.nk > 0) {
        const int64_t tot = (int64_t)parts.nk * p->npad;
        k_sum_integrals<<<(unsigned)((tot + 255) / 256), 256, 0, p->stream>>>(p->npad, parts.nk,
                                                                              parts.S, parts.part, I_out);
    }
    return hipGetLastError();
}

hipError_t launch_potential(vv10_plan *p, const IntegralParts &parts, double *energy,
                            double *f_rho, double *f_gamma, const int32_t *valid,
                            const BatchBuffers *io) {
    const int64_t nb = p->npad / 256;
    double *epart = p->red;               // [nb] partials, then the energy at red[nb]
    k_potential<<<(unsigned)nb, parts.nk > 0 ? 768 : 256, 0, p->stream>>>(
        p->n, p->npad, p->beta, parts, p->P1, p->F, p->I, f_rho, f_gamma, epart, energy_counter(p),
        energy ? energy : p->red + nb, valid, io);
    return hipGetLastError();
}

}  // namespace vv10
