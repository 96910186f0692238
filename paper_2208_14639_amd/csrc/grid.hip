// The grid pass (Section II.B grid-position intermediates) and the gradient
// pass's grid sums; the unit of the grid pass (four waves) is in grid_tile.h.
#include <algorithm>

#include "grid_tile.h"

namespace vv10 {

namespace {

// The grid pass as one workgroup per (tile, atom group): blockIdx = (tile, group).
template <typename T, typename T4, bool INTS, bool ZE>
__global__ __launch_bounds__(64 * kGridWaves) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 1))) void k_grid(
    int32_t n_atom, int32_t Pp, int32_t bgroups, bool whole, int64_t npad, const int64_t *__restrict__ seg,
    const int32_t *__restrict__ tile_i0, const int32_t *__restrict__ tile_n,
    const int32_t *__restrict__ tile_atom, const T4 *__restrict__ P0,
    const T4 *__restrict__ P1, const double4 *__restrict__ Pd, double *__restrict__ Z,
    double *__restrict__ Ze, double *__restrict__ Dpart, double *__restrict__ Ipart) {
    __shared__ GridLds<T4> lds;
    grid_unit<T, T4, INTS, ZE>(n_atom, Pp, bgroups, npad, seg, tile_i0, tile_n, tile_atom, P0, P1,
                               Pd, Z, Ze, Dpart, Ipart, blockIdx.x, blockIdx.y, whole, lds);
}

// Gradient pass (Section II.A): the pair integrals E, U, W of every outer
// point (over all j) and, per tile t of outer points (atom A) and atom
// B > A, Gpart[t][B][a] = sum_{i in t} a_i E^{Bgr}_{i,a} (B <= A: not written),
// from which the grid part of the gradient follows,
// E_gr = -sum_{B != A} sum_{i in A} a_i E^{Bgr}_i (translational invariance),
// the B < A terms being minus the (B, A) ones.
// The layout (four waves a unit; grid sums of the hexamer 0.27 -> 0.21 ms in
// FP32) and the scaled sums are those of k_grid: E^{Bgr}_i = 3 sum_j p T d.
// Without INTS (the plan already holds E, U, W) only the grid sums are formed.
// LDS for three sums a wave, not the nine of k_grid, leaves room for more of its
// workgroups (sums alone, hexamer in FP32 0.20 -> 0.19 ms; 40 waters with 60 points
// an atom in FP64 66 -> 47 us, with whole atoms a wave).
// W: waves of a workgroup; one where whole atoms a wave and no integrals leave
// them nothing to share, so that a wave without an atom B > A holds no LDS, and an
// atom each for as many as 16384 waves (30 waters with 60 points an atom in FP64 31
// -> 24 us, 20 with 200 points 132 -> 115).
template <typename T, typename T4, bool INTS, int W>
__global__ __launch_bounds__(64 * W) void k_grid_grad(
    int32_t n_atom, int32_t bgroups, bool whole, int64_t npad, const int64_t *__restrict__ seg,
    const int32_t *__restrict__ tile_i0, const int32_t *__restrict__ tile_n,
    const int32_t *__restrict__ tile_atom, const T4 *__restrict__ P0,
    const T4 *__restrict__ P1, const double4 *__restrict__ Pd, double *__restrict__ Gpart,
    double *__restrict__ Ipart) {
    __shared__ GridLds<T4, 3, W> lds;
    const int t = blockIdx.x, grp = blockIdx.y, lane = threadIdx.x & 63;
    const int wave = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    T4 *sA = lds.a[wave], *sB = lds.b[wave];
    const int A = tile_atom[t];
    const int nt = tile_n[t];
    const bool live = lane < nt;
    const int64_t i = (int64_t)tile_i0[t] + (live ? lane : 0);
    const T4 a0 = P0[i], a1 = P1[i];
    const double ai = live ? (double)a1.y : 0.0;
    const T oi = a0.w;
    double pint[3] = {};
    const GridDeal deal(W == 1 || whole, wave, grp, bgroups, W);
    for (int B = deal.B0; B < n_atom; B += deal.Bstep) {
        const int64_t jb = seg[B], je = seg[B + 1];
        double acc[3] = {};
        // the tile sums are antisymmetric in (A, B) (a_i e_ij symmetric,
        // d_ij = -d_ji): formed for B > A only, the assembly takes the B < A
        // ones from the (B, A) sums; B <= A still adds to the pair integrals
        const bool gsum = B > A;
        if (!INTS && !gsum) continue;
        for (int64_t j0 = jb + deal.j0; j0 < je; j0 += deal.jstep) {
            wave_lds_sync();
            const int64_t j = j0 + lane;
            sA[lane] = P0[j < je ? j : jb];
            sB[lane] = P1[j < je ? j : jb];
            wave_lds_sync();
            const int cnt = (int)min((int64_t)TG, je - j0);
            T pc[3] = {}, c[3] = {};
            if (!gsum) {
                // the chunk of the tile's own points leaves out the self pair
                const int jself = (B == A && j0 == tile_i0[t]) ? lane : -1;
#pragma unroll 4
                for (int jj = 0; jj < cnt; ++jj) {
                    const PairGeo<T> q = pair_geo<T>(a0, a1, sA[jj], sB[jj]);
                    const T pj = jj == jself ? T(0) : q.p;
                    const T ph = pj * q.h;
                    pc[0] += pj;
                    pc[1] += ph;
                    pc[2] += ph * q.R2;
                }
            } else {
#pragma unroll 4
                for (int jj = 0; jj < cnt; ++jj) {
                    const T4 b0 = sA[jj];
                    const PairGeo<T> q = pair_geo<T>(a0, a1, b0, sB[jj]);
                    if (INTS) {
                        const T ph = q.p * q.h;
                        pc[0] += q.p;
                        pc[1] += ph;
                        pc[2] += ph * q.R2;
                    }
                    const T e = q.p * (oi * q.ig + b0.w * q.igp + (oi + b0.w) * q.is);
                    c[0] += e * (b0.x - a0.x);
                    c[1] += e * (b0.y - a0.y);
                    c[2] += e * (b0.z - a0.z);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) acc[k] += (double)c[k];
            }
            if (INTS)
#pragma unroll
                for (int k = 0; k < 3; ++k) pint[k] += (double)pc[k];
        }
        if (!gsum) continue;
        deal.template put<3>(lds.red, lane, acc);
        double *gp = Gpart + ((int64_t)t * n_atom + B) * 3;
#pragma unroll 1
        for (int x = deal.x0; x < deal.x1; ++x) {
            const double tot = wave_sum(ai * 3.0 * deal.sum(lds.red, x, lane));
            if (lane == 0) gp[x] = tot;
        }
    }
    if constexpr (INTS) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 3; ++k) lds.red[wave][k][lane] = pint[k];
        __syncthreads();
        if (live && wave < 3) {
            double v = (wave == 0 ? -1.5 : 1.5) * waves_sum(lds.red, wave, lane);
            // self pair in FP64 (group of the own atom): E += a Phi, U += -a Phi h
            if (A % bgroups == grp && wave < 2) {
                const double4 pd = Pd[i];
                const SelfPair q = self_pair(pd.x);
                v += pd.y * q.phi * (wave == 0 ? 1.0 : -q.h);
            }
            Ipart[((int64_t)grp * 3 + wave) * npad + i] = v;
        }
    }
}

}  // namespace

template <bool INTS, bool ZE>
void grid_terms_launch(vv10_plan *p, double *Ze) {
    const Workspace &ws = p->ws;
    dim3 grid((unsigned)p->ntiles, (unsigned)ws.bgroups);
    if (p->prec == VV10_FP64)
        k_grid<double, double4, INTS, ZE><<<grid, 64 * kGridWaves, 0, p->stream>>>(
            p->n_atom, ws.Pp, ws.bgroups, p->whole, p->npad, p->d_seg, p->d_tile_i0, p->d_tile_n,
            p->d_tile_atom, p->P0, p->P1, p->P1, ws.Z, Ze, ws.Dpart, ws.Igrp);
    else
        k_grid<float, float4, INTS, ZE><<<grid, 64 * kGridWaves, 0, p->stream>>>(
            p->n_atom, ws.Pp, ws.bgroups, p->whole, p->npad, p->d_seg, p->d_tile_i0, p->d_tile_n,
            p->d_tile_atom, p->P0f, p->P1f, p->P1, ws.Z, Ze, ws.Dpart, ws.Igrp);
}

template <bool INTS>
void grid_terms_mode(vv10_plan *p, double *Ze) {
    if (Ze) grid_terms_launch<INTS, true>(p, Ze);
    else grid_terms_launch<INTS, false>(p, Ze);
}

template <bool INTS, int W>
void grid_grad_launch(vv10_plan *p, int32_t groups) {
    const GradWork &gw = p->gw;
    dim3 grid((unsigned)p->ntiles, (unsigned)groups);
    if (p->prec == VV10_FP64)
        k_grid_grad<double, double4, INTS, W><<<grid, 64 * W, 0, p->stream>>>(
            p->n_atom, groups, p->whole, p->npad, p->d_seg, p->d_tile_i0, p->d_tile_n, p->d_tile_atom,
            p->P0, p->P1, p->P1, gw.Gpart, gw.Igrp);
    else
        k_grid_grad<float, float4, INTS, W><<<grid, 64 * W, 0, p->stream>>>(
            p->n_atom, groups, p->whole, p->npad, p->d_seg, p->d_tile_i0, p->d_tile_n, p->d_tile_atom,
            p->P0f, p->P1f, p->P1, gw.Gpart, gw.Igrp);
}

hipError_t launch_grid_terms(vv10_plan *p, double *Ze, int ints_from) {
    if (ints_from >= NI) grid_terms_mode<false>(p, Ze);
    else grid_terms_mode<true>(p, Ze);
    return hipGetLastError();
}

hipError_t launch_grid_grad(vv10_plan *p, bool ints) {
    if (ints) grid_grad_launch<true, kGridWaves>(p, p->gw.bgroups);
    else if (p->whole) grid_grad_launch<false, 1>(p, std::min(p->n_atom, 1 + 16384 / p->ntiles));
    else grid_grad_launch<false, kGridWaves>(p, p->gw.bgroups);
    return hipGetLastError();
}

}  // namespace vv10
