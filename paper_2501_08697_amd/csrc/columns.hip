// Launchers of the column passes (columns.hpp).
#include <algorithm>

#include "columns.hpp"

namespace apw {

// The x transform runs one task per thread and phase (C max(A1, B1) <= threads), the y
// transform's tasks wrap around. C is the widest divisor of N2 that the threads and LDS allow:
// at 120^3 30 columns took 44.9 ms of plane passes per call of 4,096 bands, 24 took 48.1 and
// 20 took 55 (shorter chunks leave threads without a task in F). A plane alone on its CU takes 512
// threads: H psi of 128 bands and one atom at 90^3 with 49 slab rows took 1148 us with 256 (1122
// through the slab passes), 946 so.
PlaneShape plane_shape(const Plan &P, int fft_prec) {
    PlaneShape s{0, 0, P.N2 | 1, 0};
    int a1, b1, a2, b2;
    if (!lds_split_host(P.N1, &a1, &b1) || !lds_split_host(P.N2, &a2, &b2)) return s;
    if (P.N1 != P.N2 && !(P.zero_band[0] && P.zero_band[1])) return s;
    const int m1 = std::max(a1, b1), m2 = std::max(a2, b2);
    auto lds = [&](int C) {
        return ((size_t)P.nslab * s.ldr + (size_t)(P.N1 - P.nslab) * C + P.N1 + P.N2 + 1) *
               (fft_prec == 0 ? sizeof(z64) : sizeof(c32));
    };
    auto fit = [&](int nt) {
        s.C = std::min(P.N2, nt / m1);
        while (s.C > 0 && (P.N2 % s.C != 0 || lds(s.C) > 160 * 1024)) --s.C;
        s.lds = s.C > 0 ? lds(s.C) : 0;
        s.NT = std::min(nt, (std::max(s.C * m1, P.nslab * m2) + 63) / 64 * 64);
    };
    fit(plane_threads(P.N1, P.N2));
    // a plane with more slab rows than usual may be alone on its CU all the same: 256 threads would
    // then be half of what the CU holds
    if (s.lds > 80 * 1024) fit(512);
    return s;
}

// Whether the columns move and transform less than the slab passes would. Their share of the slab is
// pi / 2 times the sphere's radius over the grid length, 0.41 on the usual grid; small planes gain
// at any share, and so do planes that the slab passes cannot hold whole in LDS. H psi of 48 bands
// against the slab passes, FP64: share 0.68 72^3 440 / 480 us, 80^3 625 / 697, 96^3 1092 / 1223;
// 0.58 72^3 353 / 308, but where the plane is alone on its CU 81^3 491 / 503, 96^3 810 / 866; 0.51
// 81^3 405 / 347, 96^3 658 / 623. FP32: 0.51 64^3 234 / 222 (100 bands), 72^3 293 / 299, 80^3 429 / 477; 0.46
// 72^3 273 / 260, 80^3 371 / 346.
bool columns_pay(const Plan &P, int fft_prec) {
    const size_t eb = fft_prec == 0 ? sizeof(z64) : sizeof(c32);
    if (P.N1 * P.N2 < 72 * 72 || (size_t)P.N2 * P.N3 * eb > 160 * 1024) return true;
    const int most = fft_prec == 1 ? 48 : plane_shape(P, 0).lds > 80 * 1024 ? 55 : 62;   // per cent
    return 100 * (int64_t)P.max_ncol <= (int64_t)most * P.nslab * P.N2;
}

// Bands per z-pass work-group: up to 4 share the tables read once, while the launch keeps
// 2048 work-groups (eight a CU).
static int z_bands(const ColumnsCall &c, int ngrp) {
    if (g_yz_bands > 0) return std::min(g_yz_bands, c.ba.bbt);
    int bpw = 4;
    while (bpw > 1 && ngrp * c.nkb * ceil_div(c.ba.bbt, bpw) < 2048) bpw /= 2;
    return std::min(bpw, c.ba.bbt);
}

template <int N, typename T> static int launch_z_inv(const ColumnsCall &c, const void *psi, const double *v) {
    const Plan &P = *c.P;
    const int ngrp = ceil_div(P.max_ncol, ZTile<N>::C), bpw = z_bands(c, ngrp);
    const int nblk = ngrp * c.nkb * ceil_div(c.ba.bbt, bpw);
    const int nvt = v ? P.N1 * ceil_div(P.N2, kVtTile) * ceil_div(P.N3, kVtTile) : 0;
    auto kernel = P.zero_band[2] ? k_z_inv<N, T, T, true> : k_z_inv<N, T, T, false>;
    const void *tw = sizeof(T) == 8 ? P.tw64[2] : P.tw32[2];
    KernelTimer kt("z_inv", c.st);
    hipLaunchKernelGGL(kernel, dim3(nblk + nvt), dim3(ZTile<N>::NT), 0, c.st, static_cast<const cx<T> *>(psi),
                       P.kdesc + c.k0, c.ba, static_cast<const cx<T> *>(tw), static_cast<cx<T> *>(c.col), P.ldc,
                       ngrp, bpw, nblk, v, static_cast<T *>(c.vt), P.N1, P.N2);
    return check_launch("z_inv");
}

template <int N, typename T> static int launch_z_fwd(const ColumnsCall &c, const void *psi, void *hpsi) {
    const Plan &P = *c.P;
    const int ngrp = ceil_div(P.max_ncol, ZTile<N>::C), bpw = z_bands(c, ngrp);
    auto kernel = P.zero_band[2] ? k_z_fwd<N, T, T, true> : k_z_fwd<N, T, T, false>;
    const void *tw = sizeof(T) == 8 ? P.tw64[2] : P.tw32[2];
    KernelTimer kt("z_fwd", c.st);
    hipLaunchKernelGGL(kernel, dim3(ngrp * c.nkb * ceil_div(c.ba.bbt, bpw)), dim3(ZTile<N>::NT), 0, c.st,
                       static_cast<const cx<T> *>(c.col), P.ldc, P.kdesc + c.k0, c.ba,
                       static_cast<const cx<T> *>(tw), static_cast<const cx<T> *>(psi),
                       static_cast<cx<T> *>(hpsi), 1.0 / (double)P.N, ngrp, bpw);
    return check_launch("z_fwd");
}

// FP32 only below kColumnsF32: the FP64 kernel must never see FP32 data.
template <int N> static int z_inv(const ColumnsCall &c, const void *psi, const double *v) {
    if (c.prec == 0) return launch_z_inv<N, double>(c, psi, v);
    if constexpr (N < kColumnsF32) return launch_z_inv<N, float>(c, psi, v);
    return set_error(ABACUS_PW_EINTERNAL, "FP32 z pass without a kernel");
}
template <int N> static int z_fwd(const ColumnsCall &c, const void *psi, void *hpsi) {
    if (c.prec == 0) return launch_z_fwd<N, double>(c, psi, hpsi);
    if constexpr (N < kColumnsF32) return launch_z_fwd<N, float>(c, psi, hpsi);
    return set_error(ABACUS_PW_EINTERNAL, "FP32 z pass without a kernel");
}

int columns_inverse(const ColumnsCall &c, const void *psi, const double *v) {
    switch (c.P->N3) {
#define APW_CASE(n) case n: return z_inv<n>(c, psi, v);
        APW_LENGTHS(APW_CASE)
#undef APW_CASE
        default:
            return set_error(ABACUS_PW_EBAD_FFT_SIZE, "unsupported grid length");
    }
}

int columns_forward(const ColumnsCall &c, const void *psi, void *hpsi) {
    switch (c.P->N3) {
#define APW_CASE(n) case n: return z_fwd<n>(c, psi, hpsi);
        APW_LENGTHS(APW_CASE)
#undef APW_CASE
        default:
            return set_error(ABACUS_PW_EBAD_FFT_SIZE, "unsupported grid length");
    }
}

int columns_plane(const ColumnsCall &c) {
    if (c.prec == 1) return columns_plane_f32(c);
    switch (c.P->N1) {
#define APW_CASE(n) case n: return columns_plane_n1<n>(c);
        APW_LENGTHS(APW_CASE)
#undef APW_CASE
        default:
            return set_error(ABACUS_PW_EBAD_FFT_SIZE, "unsupported grid length");
    }
}

}  // namespace apw
