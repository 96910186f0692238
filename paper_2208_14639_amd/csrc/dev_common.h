// Device helpers shared by the VV10 kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>

namespace vv10 {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// 1/x in FP64: the hardware estimate r0 (relative error at most 2^-24.3,
// measured over 35 decades) refined by one third-order step,
// r0 (1 + e + e^2) with e = 1 - x r0, whose error e^3 lies far below an ulp
// (one FMA fewer than two Newton steps).  Used only for x > 0 and finite.
__device__ __forceinline__ double rcp64(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, __builtin_fma(e, e, e), r);
}

// A pointer that a kernel read from memory, known to be to global memory (the
// compiler sees that of kernel arguments alone and would use flat accesses, whose
// 64-bit addresses take vector registers).
template <typename T>
__device__ __forceinline__ T *global_ptr(T *p) {
    return (T *)(__attribute__((address_space(1))) T *)reinterpret_cast<uintptr_t>(p);
}
// A molecule's operand in the type that its mode holds it in.
template <typename T>
__device__ __forceinline__ const T *global_as(const void *p) {
    return global_ptr(static_cast<const T *>(p));
}

// Barrier for the compiler only: the memory accesses before it are issued
// before those after it.
__device__ __forceinline__ void mem_order() { asm volatile("" ::: "memory"); }

// The partial sums of one j split of a mixed contraction.  A split of at most
// one FP32 run stores its FP32 sums as they are (f32: half the bytes written
// here and read by the assembly, no value changed: hexamer, nine splits, step
// 2.28 -> 2.23 ms, with moving weights 3.36 -> 3.31); a longer one adds its runs
// into FP64.
struct PartialRows {
    double *y;
    bool f32;
    // split: rows of width elements each (all splits back to back)
    __device__ __forceinline__ PartialRows(double *all, int64_t split, int64_t elems, bool single)
        : y(single ? reinterpret_cast<double *>(reinterpret_cast<float *>(all) + split * elems)
                   : all + split * elems),
          f32(single) {}
};

// Adds one tile row's FP32 sums v[0..N) into its partials at off, off + 16,
// ..., off + 16 (N - 1) (N column blocks of 16); first: written, not read.
// Each partial element has a single writer (one lane of one workgroup), so a
// plain read-add-write suffices and the order of the additions, and the
// result, are fixed.  The row's loads are issued together before the adds
// (one wait per row), and rows are added one at a time so that their loads
// do not all occupy registers at once.
template <int N>
__device__ __forceinline__ void add_row(const PartialRows &p, int64_t off, const float *v, bool first) {
    double *y = p.y + off;
    if (p.f32) {
        float *yf = reinterpret_cast<float *>(p.y) + off;
#pragma unroll
        for (int k = 0; k < N; ++k) yf[16 * k] = v[k];
    } else if (first) {
#pragma unroll
        for (int k = 0; k < N; ++k) y[16 * k] = (double)v[k];
    } else {
        double t[N];
#pragma unroll
        for (int k = 0; k < N; ++k) t[k] = y[16 * k];
#pragma unroll
        for (int k = 0; k < N; ++k) y[16 * k] = t[k] + (double)v[k];
    }
    mem_order();
}

// 16 bytes a lane from base + off + soff (soff wave-uniform) into LDS at dst
// (wave-uniform) + 16 lane.  The wait is the caller's.
__device__ __forceinline__ void load16_lds(const void *base, uint32_t off, uint32_t soff, void *dst) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, -1, 0x00027000),
        reinterpret_cast<__attribute__((address_space(3))) void *>(reinterpret_cast<uintptr_t>(dst)),
        16, off, soff, 0, 0);
}

// ROWS rows of Pp columns from X, columns [col0, col0 + NC), into LDS by a
// workgroup of four waves; the caller's barrier follows.  With one column group
// (Pp = NC) they are contiguous and go there straight, 1 KiB per wave and load,
// for a scalar addition each; otherwise through registers, whose row and column
// arithmetic takes 13 of 46 VALU instructions per 64 pairs of the FP32
// contraction, which share the lanes of its matrix instructions (nine waters,
// six blocks: 2.98 -> 2.81 ms; the FP64 response of the hexamer 5.67 -> 5.53).
// One block in FP32 stays with the registers: four loads a chunk, a wave each,
// whose wait nothing hides (response to 16 densities at N 9600: 215 us, straight
// into LDS 218).
template <int ROWS, int NC, typename T>
__device__ __forceinline__ void stage_rows(const T *__restrict__ X, int32_t Pp, int col0, T *sX) {
    constexpr int U = NC * (int)sizeof(T) / 16;       // 16-byte units of a row
    constexpr int LOADS = ROWS * U / 64;
    static_assert(ROWS * U % 64 == 0, "whole loads");
    if (Pp == NC && (sizeof(T) == 8 || NC > 16)) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
        for (int k = 0; k < (LOADS + 3) / 4; ++k) {
            const int off = (wave + 4 * k) * 1024;
            if (LOADS % 4 == 0 || wave + 4 * k < LOADS)
                load16_lds(X, (threadIdx.x & 63) * 16, off, reinterpret_cast<char *>(sX) + off);
        }
        __builtin_amdgcn_s_waitcnt(0);
    } else {
        for (int e = threadIdx.x; e < ROWS * U; e += 256) {
            const int row = e / U, cc = e - row * U;
            reinterpret_cast<float4 *>(sX)[e] =
                reinterpret_cast<const float4 *>(X + (int64_t)row * Pp + col0)[cc];
        }
    }
}

// 1/x in FP32 (hardware estimate, about 1 ulp).
__device__ __forceinline__ float rcp32(float x) { return __builtin_amdgcn_rcpf(x); }

// The self pair j = i of the inner sums (R = 0, so g = g' = kappa and
// s = g + g' = 2 kappa), in FP64.  Every pair loop, in every mode, leaves
// the self pair out and the kernel that finishes a sum adds it from these
// values: on a coarse grid the self term of a point with a large weight can
// dominate its row, and in FP32 or split-BF16 its rounding would then
// dominate the row's error.
//   phi = Phi_ii, h = 1/s + 1/g, m = 1/s^2 + 1/(s g) + 1/g^2,
//   phig = dPhi/dg = -Phi (1/g + 1/s), phigg = d2Phi/dg dg' = 2 Phi (1/(g g') + 1/s^2).
struct SelfPair {
    double phi, h, m, phig, phigg;
};

__device__ __forceinline__ SelfPair self_pair(double kappa) {
    const double ig = 1.0 / kappa, is = 0.5 * ig;
    SelfPair q;
    q.phi = -1.5 * ig * ig * is;
    q.h = is + ig;
    q.m = is * is + is * ig + ig * ig;
    q.phig = -q.phi * (ig + is);
    q.phigg = 2.0 * q.phi * (ig * ig + is * is);
    return q;
}

// K_pp of the self pair (the p-channel kernel value; K_pq, K_qp, K_qq carry a
// factor R^2 and vanish): Phi + c Phi_g + c Phi_g' + c^2 Phi_gg' with c = rho dkappa/drho.
__device__ __forceinline__ double self_kpp(double kappa, double c) {
    const SelfPair q = self_pair(kappa);
    return q.phi + 2.0 * c * q.phig + c * c * q.phigg;
}

// A mask that clears one bf16 of four packed words: word `word`, its high
// half if `high`, its low half otherwise; all ones when `mine` is false.
__device__ __forceinline__ uint4 bf16_clear_mask(bool mine, int word, bool high) {
    const uint32_t k = high ? 0x0000ffffu : 0xffff0000u;
    return (uint4){mine && word == 0 ? k : 0xffffffffu, mine && word == 1 ? k : 0xffffffffu,
                   mine && word == 2 ? k : 0xffffffffu, mine && word == 3 ? k : 0xffffffffu};
}

template <typename V>
__device__ __forceinline__ V bf16_apply_mask(V v, uint4 k) {
    uint4 u = __builtin_bit_cast(uint4, v);
    u.x &= k.x;
    u.y &= k.y;
    u.z &= k.z;
    u.w &= k.w;
    return __builtin_bit_cast(V, u);
}

// Sum over the 64 lanes of a wave in a fixed butterfly order; every lane
// receives the same total.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

}  // namespace vv10
