// Launcher of the plane pass for one x length and every y length; the columns_plane_*.hip
// files instantiate it for a few x lengths each, so that they compile side by side.
#pragma once

#include <algorithm>

#include "columns.hpp"

namespace apw {

// Bands per plane work-group, of which per_cu fit on a compute unit. A round of work-groups takes
// the longer the more of them share a unit, 1 + (q - 1) / 2 for q, and the last round may be part
// empty; a work-group's tables cost about as much as 0.2 bands. Fitted to 153 cases of length and
// bands, 1 to 8 bands a work-group each: within 0.6% of the best on average, 7.4% at most (2, 4 or 8
// bands by rounds alone, two work-groups of 256 to a unit whatever the registers allow: 7.3% and
// 47%). FP32 at 72^3 x 48 bands 89 -> 71 us, FP64 x 16 bands 65 -> 48.
inline int plane_bands(int n3, int nvb, int per_cu) {
    auto round = [](int q) { return 0.5 * (q + 1); };
    const int slots = 256 * per_cu;
    int best = 1;
    double cost = 1e30;
    for (int b = 1; b <= std::min(8, nvb); ++b) {
        const int wgs = n3 * ceil_div(nvb, b), last = wgs % slots;
        const double t = (b + 0.2) * (wgs / slots * round(per_cu) + (last > 0 ? round(ceil_div(last, 256)) : 0.0));
        if (t < 0.9999 * cost) {
            cost = t;
            best = b;
        }
    }
    return best;
}

// Wavefronts per SIMD that a kernel's registers allow.
template <typename K> int kernel_waves(K kernel) {
    int groups = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&groups, kernel, 64, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 2;
    }
    return std::max(2, groups / 4);
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
    static const int waves = kernel_waves(kernel);
    const int per_cu = std::max(1, std::min((int)(160 * 1024 / sh.lds), waves * 256 / sh.NT));
    const int bpw = std::min(nvb, g_x_bands > 0 ? g_x_bands : plane_bands(P.N3, nvb, per_cu));
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
