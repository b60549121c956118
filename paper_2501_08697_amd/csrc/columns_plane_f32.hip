// Plane pass in FP32, equal x and y lengths.
#include "columns_plane.hpp"

namespace apw {

template <int N> static int plane_f32(const ColumnsCall &c) {
    if constexpr (N < kColumnsF32)
        return c.P->zero_band[0] && c.P->zero_band[1] ? launch_plane<N, N, true, float>(c)
                                                      : launch_plane<N, N, false, float>(c);
    return set_error(ABACUS_PW_EINTERNAL, "FP32 plane pass without a kernel");
}

int columns_plane_f32(const ColumnsCall &c) {
    switch (c.P->N1) {
#define APW_CASE(n) case n: return plane_f32<n>(c);
        APW_LENGTHS(APW_CASE)
#undef APW_CASE
        default:
            return set_error(ABACUS_PW_EBAD_FFT_SIZE, "unsupported grid length");
    }
}

}  // namespace apw
