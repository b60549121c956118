// Building blocks of the Cholesky factorisation in one work-group: panels of 16 columns in
// registers and 16 x 16 tile products on the FP64 matrix cores (v_mfma_f64_16x16x4f64).
//
// A factorisation column by column waits for two barriers and a pass through LDS per column:
// 1.25 us each, 160 us at n = 128. Here a wavefront factors a panel without a barrier (a row
// per lane, the pivot row's values by v_readlane), and the trailing matrix takes sixteen
// columns at once: three barriers per sixteen columns. What bounds it is the chain of pivots of a
// panel (square root, reciprocal, the updates of fifteen columns): n = 128 in LDS 160 -> 79 us.
#pragma once

#include "common.hpp"

namespace apw {

constexpr int kCholPanel = 16;

__device__ __forceinline__ double lane_value(double v, int l) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Columns [k0, k0 + 16) of the lower triangle of an n x n matrix, by one wavefront: lanes 0-15
// hold the diagonal block (every wavefront of a panel factors it again, so none waits for
// another), lanes 16-63 the rows r0 .. r0 + 47 below it, which become L. at(i, j), j <= i < n, is
// the element in LDS. All wavefronts of the panel call load, then a barrier orders their reads
// before the first store. Returns 0, or q + 1 when the pivot of column k0 + q is not positive.
struct CholPanel {
    z64 x[kCholPanel];
    int row;
    template <class At> __device__ __forceinline__ void load(At at, int n, int k0, int r0) {
        const int lane = threadIdx.x & 63;
        row = lane < kCholPanel ? k0 + lane : r0 + lane - kCholPanel;
#pragma unroll
        for (int q = 0; q < kCholPanel; ++q) {
            x[q] = z64{0.0, 0.0};
            if (row < n && k0 + q <= row) x[q] = at(row, k0 + q);
            else if (lane == q) x[q] = z64{1.0, 0.0};   // past the matrix: identity rows
        }
    }
    // Q: columns factored, at least those the matrix has from k0 on (a 4 x 4 matrix waits for 4
    // pivots, not 16: 8 us against 11, timed by events).
    template <int Q> __device__ __forceinline__ int factor() {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const double d = lane_value(x[q].re, q);
            if (!(d > 0.0) || !isfinite(d)) return q + 1;
            const double l = sqrt(d), inv = 1.0 / l;
            x[q] = lane == q ? z64{l, 0.0} : z64{x[q].re * inv, x[q].im * inv};
#pragma unroll
            for (int c = q + 1; c < Q; ++c) {
                const z64 b = z64{lane_value(x[q].re, c), lane_value(x[q].im, c)};
                x[c] = x[c] - cmulc(x[q], b);
            }
        }
        return 0;
    }
    // diag: also store the diagonal block (one wavefront of the panel does)
    template <class At> __device__ __forceinline__ void store(At at, int n, int k0, bool diag) const {
        const int lane = threadIdx.x & 63;
        if (row >= n || (lane < kCholPanel && !diag)) return;
#pragma unroll
        for (int q = 0; q < kCholPanel; ++q)
            if (k0 + q <= row) at(row, k0 + q) = x[q];
    }
};

typedef double cd4 __attribute__((ext_vector_type(4)));

// One 16 x 16 tile by one wavefront: out(i, j, sum over k < 4 KS of a(i, k) b(k, j)). a(i, k) and
// b(k, j) are read with i, j = lane % 16 and k = lane / 16 + 4 s; of the result a lane holds column
// j = lane % 16, rows i = lane / 16 + 4 e.
template <int KS, class FA, class FB, class FO> __device__ __forceinline__ void tile_product(FA a, FB b, FO out) {
    const int lane = threadIdx.x & 63, r = lane & 15, h = lane >> 4;
    cd4 re = {0.0, 0.0, 0.0, 0.0}, im = re;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const z64 x = a(r, h + 4 * s), y = b(h + 4 * s, r);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, y.re, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, y.im, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.im, y.im, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.im, y.re, im, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) out(h + 4 * e, r, z64{re[e], im[e]});
}

// The lower triangle of an n x n matrix in LDS becomes L, by a work-group of at least
// ceil((n - 16) / 48) wavefronts. Returns 0, or k + 1 for the first pivot that is not positive
// (the same in every thread).
template <class At> __device__ int chol_lds(At at, int n) {
    const int wv = threadIdx.x >> 6, nwv = blockDim.x >> 6;
    __shared__ int failed;
    if (threadIdx.x == 0) failed = 0;
    for (int k0 = 0; k0 < n; k0 += kCholPanel) {
        const int k1 = k0 + kCholPanel, r0 = k1 + wv * 48;
        const bool mine = wv == 0 || r0 < n;
        CholPanel p;
        if (mine) p.load(at, n, k0, r0);
        __syncthreads();
        if (mine) {
            const int left = n - k0;
            const int bad = left <= 4 ? p.factor<4>() : left <= 8 ? p.factor<8>() : p.factor<kCholPanel>();
            if (bad == 0) p.store(at, n, k0, wv == 0);
            else if (threadIdx.x == 0) failed = k0 + bad;
        }
        __syncthreads();
        if (failed) return failed;
        const int nt = (n - k1 + 15) / 16;   // trailing tiles per side
        for (int t = wv; t < nt * (nt + 1) / 2; t += nwv) {
            int ti = 0;
            while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
            const int i0 = k1 + 16 * ti, j0 = k1 + 16 * (t - ti * (ti + 1) / 2);
            tile_product<kCholPanel / 4>(
                [&](int i, int k) { return at(min(i0 + i, n - 1), k0 + k); },
                [&](int k, int j) {
                    const z64 v = at(min(j0 + j, n - 1), k0 + k);
                    return z64{v.re, -v.im};
                },
                [&](int i, int j, z64 v) {
                    if (i0 + i < n && j0 + j <= i0 + i) at(i0 + i, j0 + j) = at(i0 + i, j0 + j) - v;
                });
        }
        __syncthreads();
    }
    return 0;
}

}  // namespace apw
