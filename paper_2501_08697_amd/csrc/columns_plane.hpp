// Launcher of the plane pass for one x length and every y length; the columns_plane_*.hip
// files instantiate it for a few x lengths each, so that they compile side by side.
#pragma once

#include <algorithm>

#include "columns.hpp"

namespace apw {

// Bands per plane work-group. A work-group's tables cost about as much as 0.6 bands (measured
// at 72^3: 250, 254 and 275 us with 4, 2 and 8), and the last round of work-groups may be
// part empty: the fewest rounds times bands, tables included.
inline int plane_bands(int n3, int nvb, int slots) {
    int best = 1;
    double cost = 1e30;
    for (int b = 8; b >= 1; b /= 2) {
        const double t = ceil_div(n3 * ceil_div(nvb, b), slots) * (std::min(b, nvb) + 0.6);
        if (t < cost) {
            cost = t;
            best = b;
        }
    }
    return std::min(best, nvb);
}

template <int N1, int N2, bool ZB, typename T = double> static int launch_plane(const ColumnsCall &c) {
    const Plan &P = *c.P;
    constexpr int prec = sizeof(T) == 8 ? 0 : 1;
    const PlaneShape sh = plane_shape(P, prec);
    auto kernel = k_plane<N1, N2, T, ZB>;
    static bool once = false;
    if (!once) {
        APW_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    160 * 1024));
        once = true;
    }
    const int nvb = c.nkb * c.ba.bbt;
    const int per_cu = std::max(1, std::min((int)(160 * 1024 / sh.lds), 512 / sh.NT));
    const int bpw = std::min(nvb, g_x_bands > 0 ? g_x_bands : plane_bands(P.N3, nvb, 256 * per_cu));
    const int ngrp = ceil_div(nvb, bpw);
    const void *const *tw = prec == 0 ? P.tw64 : P.tw32;
    PlaneArgs a{P.kdesc + c.k0, c.vt, tw[0], tw[1], P.xrow, P.nslab, P.ldc, sh.ldr, P.N3, nvb, c.ba.bbt, bpw,
                ngrp, sh.C};
    KernelTimer kt("plane", c.st);
    hipLaunchKernelGGL(kernel, dim3(P.N3 * ngrp), dim3(sh.NT), sh.lds, c.st, static_cast<cx<T> *>(c.col), a);
    return check_launch("plane");
}

template <int N1> int columns_plane_n1(const ColumnsCall &c) {
    if (c.P->N2 == N1 && !(c.P->zero_band[0] && c.P->zero_band[1])) return launch_plane<N1, N1, false>(c);
    switch (c.P->N2) {
#define APW_CASE(n) case n: return launch_plane<N1, n, true>(c);
        APW_LENGTHS(APW_CASE)
#undef APW_CASE
        default:
            return set_error(ABACUS_PW_EBAD_FFT_SIZE, "unsupported grid length");
    }
}

}  // namespace apw
