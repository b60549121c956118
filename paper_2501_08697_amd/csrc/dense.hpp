// Small dense FP64 linear algebra on the GPU; see dense.hip.
#pragma once

#include "common.hpp"

namespace apw {

constexpr int kSmallSub = 1024;  // largest order of the one-CU kernels (their LDS arrays)
constexpr int kMaxSub = 4096;    // largest eigen-problem order handled on the device
constexpr int kMaxChol = 1024;   // largest Cholesky order (the explicit inverse holds a column in registers)
constexpr int kLargeHeevMin = 257;   // orders from here on take the multi-CU eigensolver (dense_large.hip)
constexpr int kLargeCholMin = 137;   // orders from here on take the blocked multi-CU Cholesky

// Sum over a wavefront, the same value in every lane (all 64 lanes active; fixed order). The
// partners at distance 1, 2, 4 and 8 come by DPP, those at 16 and 32 by the row swaps, all in
// the vector unit: a shuffle goes through the LDS unit, and its latency, twelve times per sum,
// was most of the serial chains that use this (one column of the tridiagonal reduction at
// n = 256 8.4 us with shuffles, 7.3 so).
template <int CTRL> __device__ __forceinline__ double dpp_add(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v = dpp_add<0x141>(v);   // row_half_mirror: the other quad of eight lanes
    v = dpp_add<0x140>(v);   // row_mirror: the other eight lanes of a row
    unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    v = __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
        __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
    b = __builtin_bit_cast(unsigned long long, v);
    lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}

// G (n x n, row-major, ld) Hermitian positive definite: lower triangle := L with
// G = L L^H; Linv (ldi) := L^{-1}. *info_dev = 0 or k + 1 for a failed pivot.
// scratch: potrf_scratch_bytes(n) bytes of device memory (unused for small n).
int potrf_inv(int n, z64 *G, int ld, z64 *Linv, int ldi, int *info_dev, void *scratch, hipStream_t st);
size_t potrf_scratch_bytes(int n);

size_t heev_scratch_bytes(int n);

// Lowest nw eigenpairs of the Hermitian A (n x n, row-major, ld; destroyed):
// w[0..nw) ascending; coef[j*ldc + i] = i-th component of the j-th eigenvector.
int heev_lowest(int n, z64 *A, int ld, int nw, double *w, z64 *coef, int ldc, void *scratch, hipStream_t st);

}  // namespace apw
