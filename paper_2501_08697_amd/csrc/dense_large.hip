// Dense FP64 linear algebra of the Davidson subspace for orders too large for
// one compute unit (Rayleigh-Ritz over up to ndim * nb basis vectors, Sec. III.B
// Davidson; 2048 for 1024 bands at ndim = 2). The one-CU kernels of dense.hip
// stream the whole trailing matrix through a single CU for every column; here
// every column's matrix-vector product runs over the whole GPU and the O(n^3)
// updates run on the MFMA GEMMs.
//
// Tridiagonal reduction T = Q^H A Q (LAPACK's blocked scheme, restated): columns
// are reduced in panels of kTrdPanel. One launch per column k = k0 + c (k_trd_step): every
// work-group finishes the previous column's w vector (w = y - tau/2 (y^H v) v), forms
// column k as stored minus the panel's rank-2 updates so far (A - V W^H - W V^H), its
// Householder reflector H = I - tau v v^H (v[k+1] = 1, real off-diagonal beta) and the dot
// products W^H v, V^H v, all of which is O(n kTrdPanel) and done alike in each; then it computes
// its own rows of y = tau (A22 v - V (W^H v) - W (V^H v)), A22 the trailing matrix as it
// was when the panel started. After the panel the trailing matrix takes its updates at once
// (k_trd_update). What bounds it is the chain of launches and, in a launch, of waits: 5.0 us at
// n = 256 when each launch waits for memory once and sums by wave_sum, 7.8 with the panel read
// where it was used and shuffled sums. A column took 11.5 us at n = 256 in one work-group and
// 20.1 us at n = 1024 in two launches (one work-group for the vectors, then the product), 5.6
// and 9.3 us now.
//
// Back-transformation coef = Q Z (Z the real tridiagonal eigenvectors): the
// reflectors, kept as rows of Vr, are applied in blocks of kPL from the last to
// the first as I - V T V^H (compact WY; T upper triangular from the block's
// Gram matrix and the taus), each block two GEMMs.
//
// Cholesky G = L L^H in blocks of kCB columns: the diagonal block is factored
// and inverted in LDS by one work-group, the panel below it is L21 = A21 L11^-H
// (GEMM) and the trailing matrix takes A22 -= L21 L21^H (GEMM).
#include <algorithm>
#include <type_traits>

#include "chol_device.hpp"
#include "common.hpp"
#include "dense.hpp"
#include "gemm.hpp"

namespace apw {

namespace {

constexpr int kPL = 32;       // reflectors per WY block of the back-transformation
constexpr int kCB = 64;       // columns per block of the blocked Cholesky

__device__ __forceinline__ z64 zc(z64 a) { return z64{a.re, -a.im}; }
__device__ __forceinline__ double za2(z64 a) { return a.re * a.re + a.im * a.im; }

struct TrdArgs {
    int n, ld;
    z64 *A;
    double *d, *e;
    z64 *tau;
    z64 *Vr;      // [n][n] reflector rows (zero outside k+1 .. n-1)
    z64 *P;       // [2 PL][n] panel vectors by columns: V_0 .. V_{PL-1}, W_0 .. W_{PL-1}
    z64 *y;       // [2][n] y of the current column and of the one before (by parity of k)
};

// Sum over the work-group of one complex value per thread (fixed order); one barrier.
template <int NT> __device__ __forceinline__ z64 zsum(z64 v, z64 *red) {
    const double re = wave_sum(v.re), im = wave_sum(v.im);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = z64{re, im};
    __syncthreads();
    z64 s = z64{0.0, 0.0};
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) s = s + red[q];
    return s;
}

constexpr int kTrdPanel = 8;   // columns per panel
constexpr int kTrdRows = 2;    // rows of y per wavefront
constexpr int kTrdAhead = 4;   // 64-column pieces of a row fetched ahead

// Column k = k0 + C. ONE: a thread per row (m <= NT); its panel row comes in registers with the
// first loads of the launch and goes to LDS for the dot products, so the launch waits for memory
// once. Without it (the panel's 18 m values exceed LDS above m = 512) the panel is read from
// memory where it is used. C is a template argument so that no load of an absent column is made.
template <int NT, bool ONE, int C>
__global__ __launch_bounds__(NT) void k_trd_step(TrdArgs a, int k0) {
    constexpr int PL = kTrdPanel, NW = NT / 64, L = C > 0 ? C - 1 : 0;   // L: the last column so far
    extern __shared__ __align__(16) unsigned char smem_trd[];
    const int n = a.n, k = k0 + C, m = n - k;
    z64 *xs = reinterpret_cast<z64 *>(smem_trd);   // [m] column k, rows k ..
    z64 *wl = xs + m;                              // [m] w of panel column L, rows k ..
    z64 *pv = wl + m, *pw = pv + C * m;            // ONE: V [C][m] and W [C - 1][m], rows k ..
    __shared__ z64 pk[2 * PL];                     // row k of V and W
    __shared__ z64 dots[2 * PL];                   // W^H x, V^H x over rows k + 2 ..
    __shared__ z64 zred[NW];
    __shared__ double red[NW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const z64 *V = a.P + k, *W = V + (int64_t)PL * n;   // rows k ..
    const z64 *yp = a.y + (int64_t)((k - 1) & 1) * n + k;
    // everything that can be asked for at once: this thread's row of the panel and of column k,
    // row k of the panel, this wavefront's rows of A22
    const int ic = min(tid, m - 1);
    z64 vi[C > 0 ? C : 1], wi[C > 0 ? C : 1], x0, y0, yk, t0;
    if constexpr (ONE) {
        x0 = a.A[(int64_t)k * a.ld + k + ic];
#pragma unroll
        for (int q = 0; q < C; ++q) vi[q] = V[(int64_t)q * n + ic];
#pragma unroll
        for (int q = 0; q < L; ++q) wi[q] = W[(int64_t)q * n + ic];
    }
    if constexpr (C > 0) {
        y0 = yp[ic];
        yk = yp[0];
        t0 = a.tau[k - 1];
    }
    const z64 pk0 = a.P[(int64_t)(tid % (2 * PL)) * n + k];
    const int r0 = k + 1 + (blockIdx.x * NW + wv) * kTrdRows;
    z64 ar[kTrdRows][kTrdAhead], a0[kTrdRows];
#pragma unroll
    for (int r = 0; r < kTrdRows; ++r) {
        const z64 *row = a.A + (int64_t)min(r0 + r, n - 1) * a.ld;
#pragma unroll
        for (int u = 0; u < kTrdAhead; ++u) ar[r][u] = row[min(k + 2 + lane + 64 * u, n - 1)];
        a0[r] = row[k + 1];
    }
    if (tid < 2 * PL) pk[tid] = pk0;   // columns from C on are never read
    // w of column L over rows k .. (row k = its reflector's leading 1)
    z64 wk = z64{0.0, 0.0};   // w at row k
    z64 al = z64{0.0, 0.0};
    if constexpr (C > 0) {
        z64 s = z64{0.0, 0.0};
        if constexpr (ONE) {
            if (tid < m) s = cmulc(vi[L], y0);   // conj(y) v
        } else {
            for (int i = tid; i < m; i += NT) {
                const z64 yv = yp[i], v = V[(int64_t)L * n + i];
                wl[i] = yv;
                xs[i] = v;
                s = s + cmulc(v, yv);
            }
        }
        s = zsum<NT>(s, zred);
        al = cmul(z64{-0.5 * t0.re, -0.5 * t0.im}, s);
        wk = yk + al;
    } else {
        __syncthreads();
    }
    // column k, rows k ..: conj(row k of A) minus the panel's updates of columns q < C
    double p = 0.0;
    for (int i = tid; i < m; i += NT) {
        if constexpr (!ONE) {
            x0 = a.A[(int64_t)k * a.ld + k + i];
#pragma unroll
            for (int q = 0; q < C; ++q) vi[q] = V[(int64_t)q * n + i];
#pragma unroll
            for (int q = 0; q < L; ++q) wi[q] = W[(int64_t)q * n + i];
            if constexpr (C > 0) y0 = wl[i];
        }
        z64 x = zc(x0);
        if constexpr (C > 0) {
            wi[L] = y0 + cmul(al, vi[L]);
            wl[i] = wi[L];
            if (blockIdx.x == 0) a.P[(int64_t)(PL + L) * n + k + i] = wi[L];
        }
#pragma unroll
        for (int q = 0; q < C; ++q)   // v_i conj(w_k) + w_i conj(v_k)
            x = x - cmulc(vi[q], q == L ? wk : pk[PL + q]) - cmulc(wi[q], pk[q]);
        xs[i] = x;
        if constexpr (ONE) {
#pragma unroll
            for (int q = 0; q < C; ++q) pv[q * m + i] = vi[q];
#pragma unroll
            for (int q = 0; q < L; ++q) pw[q * m + i] = wi[q];
        }
        if (i >= 2) p += za2(x);
    }
    p = wave_sum(p);
    if (lane == 0) red[wv] = p;
    __syncthreads();
    auto vat = [&](int q, int i) { return ONE ? pv[q * m + i] : V[(int64_t)q * n + i]; };   // rows from k
    auto wat = [&](int q, int i) { return q == L ? wl[i] : ONE ? pw[q * m + i] : W[(int64_t)q * n + i]; };
    // W^H x and V^H x over rows k + 2 ..; a wavefront takes its products together
    if constexpr (C > 0) {
        constexpr int ND = (2 * C + NW - 1) / NW;
        z64 s[ND];
#pragma unroll
        for (int u = 0; u < ND; ++u) s[u] = z64{0.0, 0.0};
        for (int i = 2 + lane; i < m; i += 64) {
            const z64 x = xs[i];
#pragma unroll
            for (int u = 0; u < ND; ++u) {
                const int q = min(wv + NW * u, 2 * C - 1);
                s[u] = s[u] + cmulc(x, q < C ? wat(q, i) : vat(q - C, i));   // conj(u) x
            }
        }
#pragma unroll
        for (int u = 0; u < ND; ++u) {
            const int q = wv + NW * u;
            const double sr = wave_sum(s[u].re), si = wave_sum(s[u].im);
            if (lane == 0 && q < 2 * C) dots[q < C ? q : PL + q - C] = z64{sr, si};
        }
    }
    // W and V at row k + 1 and at this wavefront's rows, lane q < C the column q
    const int lq = min(lane, L);
    z64 w1 = z64{0.0, 0.0}, v1 = w1, vr[kTrdRows], wr[kTrdRows];
    if constexpr (C > 0) {
        w1 = wat(lq, 1);
        v1 = vat(lq, 1);
#pragma unroll
        for (int r = 0; r < kTrdRows; ++r) {
            const int i = min(r0 + r, n - 1) - k;
            vr[r] = vat(lq, i);
            wr[r] = wat(lq, i);
        }
    }
    __syncthreads();
    double xn2 = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) xn2 += red[q];
    const z64 alpha = xs[1];
    double beta = alpha.re;
    z64 t = z64{0.0, 0.0}, scale = z64{0.0, 0.0};
    if (!(xn2 == 0.0 && alpha.im == 0.0)) {
        beta = -copysign(sqrt(alpha.re * alpha.re + alpha.im * alpha.im + xn2), alpha.re);
        t = z64{(beta - alpha.re) / beta, -alpha.im / beta};
        const z64 den = z64{alpha.re - beta, alpha.im};   // scale = 1 / (alpha - beta)
        const double dd = za2(den);
        scale = z64{den.re / dd, -den.im / dd};
    }
    // y = tau (A22 v - V (W^H v) - W (V^H v)) for the wavefront's rows, v = [1, scale x];
    // lane q < C takes the panel column q of the correction
    z64 wd = z64{0.0, 0.0}, vd = wd;   // W_q^H v, V_q^H v
    if (C > 0 && lane < C) {
        wd = zc(w1) + cmul(scale, dots[lane]);
        vd = zc(v1) + cmul(scale, dots[PL + lane]);
    }
    z64 s[kTrdRows];
#pragma unroll
    for (int r = 0; r < kTrdRows; ++r) s[r] = z64{0.0, 0.0};
#pragma unroll
    for (int u = 0; u < kTrdAhead; ++u) {
        const int j = 2 + lane + 64 * u;
        const z64 x = j < m ? xs[j] : z64{0.0, 0.0};
#pragma unroll
        for (int r = 0; r < kTrdRows; ++r) s[r] = s[r] + (j < m ? cmul(ar[r][u], x) : z64{0.0, 0.0});
    }
    for (int j = 2 + lane + 64 * kTrdAhead; j < m; j += 256) {
        z64 v[kTrdRows][4];
#pragma unroll
        for (int r = 0; r < kTrdRows; ++r)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                v[r][u] = a.A[(int64_t)min(r0 + r, n - 1) * a.ld + k + min(j + 64 * u, m - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (j + 64 * u < m) {
                const z64 x = xs[j + 64 * u];
#pragma unroll
                for (int r = 0; r < kTrdRows; ++r) s[r] = s[r] + cmul(v[r][u], x);
            }
    }
#pragma unroll
    for (int r = 0; r < kTrdRows; ++r) {
        s[r] = cmul(scale, s[r]);
        if (C > 0 && lane < C) s[r] = s[r] - cmul(vr[r], wd) - cmul(wr[r], vd);
        const double sr = wave_sum(s[r].re), si = wave_sum(s[r].im);
        if (lane == 0 && r0 + r < n) a.y[(int64_t)(k & 1) * n + r0 + r] = cmul(t, a0[r] + z64{sr, si});
    }
    if (blockIdx.x == 0) {
        if (tid == 0) {
            a.d[k] = xs[0].re;
            a.e[k] = beta;
            a.tau[k] = t;
        }
        for (int i = tid; i < n; i += NT) {
            z64 v = z64{0.0, 0.0};
            if (i == k + 1) v = z64{1.0, 0.0};
            else if (i > k + 1) v = cmul(xs[i - k], scale);
            a.Vr[(int64_t)k * n + i] = v;
            if (i > k) a.P[(int64_t)C * n + i] = v;
        }
    }
}

// Trailing update after a panel of bw columns, A[i][j] -= sum_q V_iq conj(W_jq) + W_iq conj(V_jq)
// for i, j >= t0 = k0 + bw (full storage; entries (i, j) and (j, i) come out conjugate to rounding:
// which product of a pair is fused into its sum differs).
// The last w of the panel is finished here, by every work-group for its own rows and columns.
// A work-group takes 32 rows x 64 columns; a thread one column and eight rows.
__global__ __launch_bounds__(256) void k_trd_update(TrdArgs a, int k0, int bw) {
    constexpr int PL = kTrdPanel;
    __shared__ z64 rv[PL][32], rw[PL][32];
    __shared__ z64 zred[4];
    const int n = a.n, t0 = k0 + bw, kp = t0 - 1, tid = threadIdx.x;
    const int i0 = t0 + blockIdx.y * 32, j = t0 + blockIdx.x * 64 + (tid & 63);
    const z64 *V = a.P, *W = a.P + (int64_t)PL * n, *yp = a.y + (int64_t)(kp & 1) * n;
    const z64 *vl = V + (int64_t)(bw - 1) * n;
    z64 s = z64{0.0, 0.0};
    for (int i = t0 + tid; i < n; i += 256) s = s + cmulc(vl[i], yp[i]);   // conj(y) v
    const z64 t = a.tau[kp];
    s = zsum<256>(s, zred);
    const z64 al = cmul(z64{-0.5 * t.re, -0.5 * t.im}, s);
    for (int q = tid >> 5; q < PL; q += 8) {
        const int r = tid & 31, i = min(i0 + r, n - 1), qc = min(q, bw - 1);
        const z64 v = V[(int64_t)qc * n + i], w = q == bw - 1 ? yp[i] + cmul(al, v) : W[(int64_t)qc * n + i];
        rv[q][r] = q < bw ? v : z64{0.0, 0.0};
        rw[q][r] = q < bw ? w : z64{0.0, 0.0};
    }
    z64 vj[PL], wj[PL];
    const int jc = min(j, n - 1);
#pragma unroll
    for (int q = 0; q < PL; ++q) {
        const int qc = min(q, bw - 1);
        const z64 v = V[(int64_t)qc * n + jc], w = q == bw - 1 ? yp[jc] + cmul(al, v) : W[(int64_t)qc * n + jc];
        vj[q] = q < bw ? zc(v) : z64{0.0, 0.0};
        wj[q] = q < bw ? zc(w) : z64{0.0, 0.0};
    }
    __syncthreads();
    if (j >= n) return;
    z64 x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = a.A[(int64_t)min(i0 + (tid >> 6) + 4 * u, n - 1) * a.ld + j];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int r = (tid >> 6) + 4 * u;
        if (i0 + r >= n) break;
        z64 s0 = z64{0.0, 0.0}, s1 = z64{0.0, 0.0};   // two independent chains
#pragma unroll
        for (int q = 0; q < PL; ++q) {
            s0 = s0 + cmul(rv[q][r], wj[q]);
            s1 = s1 + cmul(rw[q][r], vj[q]);
        }
        a.A[(int64_t)(i0 + r) * a.ld + j] = x[u] - (s0 + s1);
    }
}

__global__ void k_trd_last(const z64 *A, int ld, int n, double *d) {
    if (threadIdx.x == 0 && blockIdx.x == 0) d[n - 1] = A[(int64_t)(n - 1) * ld + n - 1].re;
}

// coef[j][i] = Z[j][i] (real eigenvector rows to complex rows of ld ldc)
__global__ void k_real_rows(const double *Z, int ldz, int n, int nw, z64 *coef, int ldc) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * nw) return;
    const int j = (int)(t / n), i = (int)(t - (int64_t)j * n);
    coef[(int64_t)j * ldc + i] = z64{Z[(int64_t)j * ldz + i], 0.0};
}

// T (upper triangular, nbk x nbk, row-major) of the compact WY form of H_0 ... H_{nbk-1}:
// T[q][q] = tau_q, T[r][q] = -tau_q sum_{s = r}^{q-1} T[r][s] G[s][q] for r < q, where
// G[s][q] = v_s^H v_q is given transposed: Gt[q * nbk + s] = G[s][q]. One work-group per block of
// reflectors (kPL of the nref, the last one fewer): a block's serial recurrence takes 57 us, and
// launched one by one between the products of the blocks it was 4.3 ms of a Davidson run at 120^3.
__global__ void k_wy_t(int nref, const z64 *tau, const z64 *Gt, z64 *T) {
    __shared__ z64 Ts[kPL][kPL];
    const int r = threadIdx.x, b0 = blockIdx.x * kPL, nbk = min(kPL, nref - b0);
    tau += b0;
    Gt += (int64_t)b0 * kPL;
    T += (int64_t)b0 * kPL;
    for (int q = 0; q < nbk; ++q) {
        if (r < q) {
            z64 acc = z64{0.0, 0.0};
            for (int s2 = r; s2 < q; ++s2) acc = acc + cmul(Ts[r][s2], Gt[q * nbk + s2]);
            const z64 tq = tau[q];
            Ts[r][q] = z64{-(tq.re * acc.re - tq.im * acc.im), -(tq.re * acc.im + tq.im * acc.re)};
        } else if (r == q) {
            Ts[q][q] = tau[q];
        } else if (r < nbk) {
            Ts[r][q] = z64{0.0, 0.0};
        }
        __syncthreads();
    }
    for (int q = 0; q < nbk; ++q)
        if (r < nbk) T[r * nbk + q] = Ts[r][q];
}

// S'[j][q] = sum_r T[q][r] S[j][r]   (S, S' are [nw][nbk])
__global__ void k_wy_ts(int nbk, int nw, const z64 *T, const z64 *S, z64 *Sp) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)nw * nbk) return;
    const int j = (int)(t / nbk), q = (int)(t - (int64_t)j * nbk);
    z64 acc = z64{0.0, 0.0};
    for (int r = q; r < nbk; ++r) acc = acc + cmul(T[q * nbk + r], S[(int64_t)j * nbk + r]);
    Sp[t] = acc;
}

// Diagonal block of the blocked Cholesky: factor G[j0 .. j0+jb)^2 in LDS (lower, chol_device.hpp),
// write L11 back and Li = L11^{-1} (jb x jb, row-major). Skipped when an earlier block failed.
// The inverse: the 16 x 16 diagonal blocks by forward substitution, a column per lane, then
// twice X21 = -X22 (L21 X11) for neighbouring blocks of 16 and of 32 on the matrix cores.
// 39 us at jb = 64; column by column, with one thread per column of the inverse, 132 us.
__global__ __launch_bounds__(512) void k_chol_diag(z64 *G, int ld, int j0, int jb, z64 *Li, int *info) {
    __shared__ z64 L[kCB][kCB + 1];   // identity past jb
    __shared__ z64 X[kCB][kCB + 1];   // lower triangle; the products L21 X11 above it, cleared at the end
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (j0 == 0 && tid == 0) *info = 0;
    if (j0 > 0 && *info != 0) return;
    for (int t = tid; t < kCB * kCB; t += blockDim.x) {
        const int i = t / kCB, j = t - i * kCB;
        L[i][j] = j <= i && i < jb ? G[(int64_t)(j0 + i) * ld + j0 + j] : z64{i == j ? 1.0 : 0.0, 0.0};
    }
    __syncthreads();
    const int bad = chol_lds([&](int i, int j) -> z64 & { return L[i][j]; }, jb);
    if (bad) {
        if (tid == 0) *info = j0 + bad;
        return;
    }
    if (wv < kCB / 16 && lane < 16) {
        const int o = 16 * wv;
        z64 x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            z64 s = z64{i == lane ? 1.0 : 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < i; ++q) s = s - cmul(L[o + i][o + q], x[q]);
            const double r = 1.0 / L[o + i][o + i].re;
            x[i] = z64{s.re * r, s.im * r};
            X[o + i][o + lane] = x[i];
        }
    }
    __syncthreads();
    // blocks of 16: pair p = rows and columns [32 p, 32 p + 32), one wavefront each
    auto merge = [&](auto half, int o, int ti, int tj, bool second) {
        constexpr int H = decltype(half)::value;
        const int a = o, b = o + H;   // first rows of the upper and lower block
        if (!second)
            tile_product<H / 4>([&](int i, int k) { return L[b + 16 * ti + i][a + k]; },
                                [&](int k, int j) { return X[a + k][a + 16 * tj + j]; },
                                [&](int i, int j, z64 v) { X[a + 16 * ti + i][b + 16 * tj + j] = v; });
        else
            tile_product<H / 4>([&](int i, int k) { return X[b + 16 * ti + i][b + k]; },
                                [&](int k, int j) { return X[a + k][b + 16 * tj + j]; },
                                [&](int i, int j, z64 v) { X[b + 16 * ti + i][a + 16 * tj + j] = z64{-v.re, -v.im}; });
    };
    for (int second = 0; second < 2; ++second) {
        if (wv < 2) merge(std::integral_constant<int, 16>{}, 32 * wv, 0, 0, second);
        __syncthreads();
    }
    if (tid < 512) X[32 * (tid >> 8) + ((tid >> 4) & 15)][32 * (tid >> 8) + 16 + (tid & 15)] = z64{0.0, 0.0};
    __syncthreads();
    for (int second = 0; second < 2; ++second) {
        if (wv < 4) merge(std::integral_constant<int, 32>{}, 0, wv >> 1, wv & 1, second);
        __syncthreads();
    }
    for (int t = tid; t < jb * jb; t += blockDim.x) {
        const int i = t / jb, j = t - i * jb;
        if (j <= i) G[(int64_t)(j0 + i) * ld + j0 + j] = L[i][j];
        Li[t] = j <= i ? X[i][j] : z64{0.0, 0.0};
    }
}

}  // namespace

// ------------------------------------------------------------------ drivers --

template <int NT, bool ONE, int C> static int trd_step(const TrdArgs &a, int k0, hipStream_t st) {
    static bool once = false;
    if (!once) {
        APW_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_trd_step<NT, ONE, C>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024));
        once = true;
    }
    const int m = a.n - k0 - C;
    const size_t lds = sizeof(z64) * (size_t)m * (ONE ? 2 + std::max(0, 2 * C - 1) : 2);
    hipLaunchKernelGGL((k_trd_step<NT, ONE, C>), dim3((unsigned)ceil_div(m - 1, NT / 64 * kTrdRows)), dim3(NT), lds, st,
                       a, k0);
    return ABACUS_PW_OK;
}

// Columns k0 + C .. of a panel of bw
template <int C> static int trd_panel(const TrdArgs &a, int k0, int bw, hipStream_t st) {
    if constexpr (C < kTrdPanel) {
        if (C >= bw) return ABACUS_PW_OK;
        const int m = a.n - k0 - C;
        if (m <= 256) APW_TRY((trd_step<256, true, C>(a, k0, st)));
        else if (m <= 512) APW_TRY((trd_step<512, true, C>(a, k0, st)));
        else APW_TRY((trd_step<512, false, C>(a, k0, st)));   // 1024 threads leave 128 registers and spill
        return trd_panel<C + 1>(a, k0, bw, st);
    }
    return ABACUS_PW_OK;
}

static int trd_reduce(const TrdArgs &a, hipStream_t st) {
    for (int k0 = 0; k0 < a.n - 1; k0 += kTrdPanel) {
        const int bw = std::min(kTrdPanel, a.n - 1 - k0), mt = a.n - k0 - bw;
        APW_TRY(trd_panel<0>(a, k0, bw, st));
        hipLaunchKernelGGL(k_trd_update, dim3((unsigned)ceil_div(mt, 64), (unsigned)ceil_div(mt, 32)), dim3(256), 0, st,
                           a, k0, bw);
        APW_TRY(check_launch("hetrd panel"));
    }
    return ABACUS_PW_OK;
}

size_t trd_scratch_elems(int n) { return (size_t)(2 * kTrdPanel + 2) * n; }   // P and y

// A -> d[n], e[n - 1], tau[n], Vr [n][n]; work: trd_scratch_elems(n) complex128. A is destroyed.
int trd_multi(int n, z64 *A, int ld, double *d, double *e, z64 *tau, z64 *Vr, z64 *work, hipStream_t st) {
    TrdArgs a{n, ld, A, d, e, tau, Vr, work, work + (size_t)2 * kTrdPanel * n};
    APW_TRY(trd_reduce(a, st));
    hipLaunchKernelGGL(k_trd_last, dim3(1), dim3(64), 0, st, A, ld, n, d);
    return check_launch("hetrd last");
}

// Partial sums of the back-transformation's products: the Gram matrices of the reflector blocks
// (kPL x kPL, also where fewer vectors are wanted) and V^H coef (kPL x nw).
size_t heev_part_bytes(int n, int nw) {
    return std::max(gemm_cn_part_bytes(kPL, kPL, n, 16, 0), gemm_cn_part_bytes(kPL, nw, n, 16, 0));
}

// Scratch of the large-order routines (bytes), carved in the order below.
size_t heev_large_scratch_bytes(int n, int nw) {
    const size_t zn = sizeof(z64);
    return 12 * 256                                       // alignment of the regions
           + (size_t)n * (2 * sizeof(double) + zn)        // d, e, tau
           + (size_t)n * n * zn                           // Vr
           + trd_scratch_elems(n) * zn                    // panel vectors, y
           + (size_t)n * n * sizeof(double)               // Z
           + (size_t)2 * (n + kPL) * kPL * zn             // Gram, T of every block
           + (size_t)2 * nw * kPL * zn                    // S, S'
           + heev_part_bytes(n, nw) + 4096;
}

int stein_vectors(int n, const double *d, const double *e, int nw, const double *w, double *Z, int ldz, void *work,
                  size_t work_bytes, hipStream_t st);   // dense.hip
int stebz_values(int n, const double *d, const double *e, int nw, double *w, hipStream_t st);   // dense.hip
size_t stein_work_bytes(int n, int nw);   // dense.hip

int heev_lowest_large(int n, z64 *A, int ld, int nw, double *w, z64 *coef, int ldc, void *scratch,
                      hipStream_t st) {
    if (n > kMaxSub) return set_error(ABACUS_PW_EBAD_SHAPE, "subspace size above the device eigensolver limit");
    char *p = static_cast<char *>(scratch);
    auto take = [&](size_t bytes) {
        char *q = p;
        p += (bytes + 255) / 256 * 256;
        return q;
    };
    double *d = reinterpret_cast<double *>(take(sizeof(double) * n));
    double *e = reinterpret_cast<double *>(take(sizeof(double) * n));
    z64 *tau = reinterpret_cast<z64 *>(take(sizeof(z64) * n));
    z64 *Vr = reinterpret_cast<z64 *>(take(sizeof(z64) * (size_t)n * n));
    z64 *trd = reinterpret_cast<z64 *>(take(sizeof(z64) * trd_scratch_elems(n)));
    double *Z = reinterpret_cast<double *>(take(sizeof(double) * (size_t)n * n));
    const size_t tri_bytes = sizeof(z64) * (size_t)ceil_div(n, kPL) * kPL * kPL;
    z64 *Gt = reinterpret_cast<z64 *>(take(tri_bytes));
    z64 *T = reinterpret_cast<z64 *>(take(tri_bytes));
    z64 *S = reinterpret_cast<z64 *>(take(sizeof(z64) * (size_t)nw * kPL));
    z64 *Sp = reinterpret_cast<z64 *>(take(sizeof(z64) * (size_t)nw * kPL));
    void *part = take(heev_part_bytes(n, nw));
    {
        KernelTimer kt("hetrd_mc", st);
        APW_TRY(trd_multi(n, A, ld, d, e, tau, Vr, trd, st));
    }
    APW_TRY(stebz_values(n, d, e, nw, w, st));
    {
        // inverse-iteration work space: its own region after the GEMM partials
        void *work = take(stein_work_bytes(n, nw));
        APW_TRY(stein_vectors(n, d, e, nw, w, Z, n, work, stein_work_bytes(n, nw), st));
    }
    KernelTimer kt("unmtr_mc", st);
    {
        const int64_t tot = (int64_t)n * nw;
        hipLaunchKernelGGL(k_real_rows, dim3((unsigned)ceil_div64(tot, 256)), dim3(256), 0, st, Z, n, n, nw, coef, ldc);
        APW_TRY(check_launch("real rows"));
    }
    // coef = H_0 ... H_{n-2} Z, blocks of kPL reflectors from the last block to the first
    const int nref = n - 1;
    for (int b0 = 0; b0 < nref; b0 += kPL) {
        const int nbk = std::min(kPL, nref - b0);
        const z64 *Vb = Vr + (size_t)b0 * n;
        APW_TRY(gemm_cn(0, nbk, nbk, n, Vb, n, Vb, n, Gt + (size_t)b0 * kPL, nbk, 1.0, 0.0, part, 0, st));
    }
    hipLaunchKernelGGL(k_wy_t, dim3(ceil_div(nref, kPL)), dim3(kPL), 0, st, nref, tau, Gt, T);
    APW_TRY(check_launch("wy T"));
    for (int b0 = ((nref - 1) / kPL) * kPL; b0 >= 0; b0 -= kPL) {
        const int nbk = std::min(kPL, nref - b0);
        const z64 *Vb = Vr + (size_t)b0 * n, *Tb = T + (size_t)b0 * kPL;
        APW_TRY(gemm_cn(0, nbk, nw, n, Vb, n, coef, ldc, S, nbk, 1.0, 0.0, part, 0, st));
        const int64_t tot = (int64_t)nw * nbk;
        hipLaunchKernelGGL(k_wy_ts, dim3((unsigned)ceil_div64(tot, 256)), dim3(256), 0, st, nbk, nw, Tb, S, Sp);
        APW_TRY(check_launch("wy"));
        APW_TRY(gemm_nn(0, nw, n, nbk, Sp, nbk, Vb, n, coef, ldc, -1.0, 1.0, st));
    }
    return ABACUS_PW_OK;
}

size_t potrf_large_scratch_bytes(int n) {
    return (size_t)kCB * kCB * sizeof(z64) + (size_t)n * kCB * sizeof(z64) +
           gemm_cn_part_bytes(n, n, kCB, 16, 0) + gemm_cn_part_bytes(kCB, n, kCB, 16, 0) + 1024;
}

// Blocked Cholesky of G (lower triangle := L); *info_dev = 0 or (failed pivot + 1).
int potrf_large(int n, z64 *G, int ld, int *info_dev, void *scratch, hipStream_t st) {
    char *p = static_cast<char *>(scratch);
    z64 *Li = reinterpret_cast<z64 *>(p);
    z64 *tmp = Li + kCB * kCB;
    void *part = tmp + (size_t)n * kCB;
    KernelTimer kt("potrf_mc", st);
    for (int j0 = 0; j0 < n; j0 += kCB) {
        const int jb = std::min(kCB, n - j0), j1 = j0 + jb, m = n - j1;
        hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(512), 0, st, G, ld, j0, jb, Li, info_dev);
        APW_TRY(check_launch("chol diag"));
        if (m == 0) break;
        // L21 = A21 L11^{-H}: tmp[i][q] = sum_r conj(Li[q][r]) A21[i][r]
        APW_TRY(gemm_cn(0, jb, m, jb, Li, jb, G + (size_t)j1 * ld + j0, ld, tmp, jb, 1.0, 0.0, part, 0, st));
        APW_HIP(hipMemcpy2DAsync(G + (size_t)j1 * ld + j0, sizeof(z64) * ld, tmp, sizeof(z64) * jb, sizeof(z64) * jb, m,
                                 hipMemcpyDeviceToDevice, st));
        // A22 -= L21 L21^H
        APW_TRY(gemm_cn(0, m, m, jb, G + (size_t)j1 * ld + j0, ld, G + (size_t)j1 * ld + j0, ld,
                        G + (size_t)j1 * ld + j1, ld, -1.0, 1.0, part, 0, st));
    }
    return ABACUS_PW_OK;
}

}  // namespace apw
