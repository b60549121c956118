// Band density through z columns, rho(r) = sum over bands of occ |psi(r)|^2 (columns.hpp has the
// column passes): k_z_inv, then one plane pass that transforms y and x in LDS and adds the
// weighted squares up in registers, so that a band's plane never leaves the compute unit. The
// work-groups of a plane share its bands; their sums are added in order at the end. 72^3 x 128
// bands with rho(G): 263 -> 219 us.
#include <algorithm>

#include "columns.hpp"
#include "local.hpp"

namespace apw {

// Chunk width: the widest divisor of N whose tasks fit the threads, one per thread and phase.
template <int N> struct DensTile {
    static constexpr int A = LdsSplit<N>::A, B = LdsSplit<N>::B, M = A > B ? A : B, NT = plane_threads(N, N);
    static constexpr int width(int c) { return N % c == 0 ? c : width(c - 1); }
    static constexpr int C = width(N < NT / M ? N : NT / M), NCH = N / C;
    // The sums of a thread, N A / C of them, have to stay in registers beside the transform: at 80,
    // 90, 120 and 128 (32 to 64) they spill, and those lengths keep the slab passes.
    static constexpr bool fits = NCH * A <= 27;
    // Columns of the next band are fetched behind this one where registers are left for them.
    static constexpr bool ahead = N < 80;
};

// LDS of a plane: slab rows, the chunk's values without a slab row, twiddles, one zero.
template <int N> static size_t dens_lds(int nslab) {
    return ((size_t)nslab * (N | 1) + (size_t)(N - nslab) * DensTile<N>::C + N + 1) * sizeof(z64);
}

// Work-group roles, LDS layout and the phases S, Y1, Y2, I and F are k_plane's (equal x and y
// lengths), without V and the way back. A thread of F owns the same grid points in every band: its
// A sums of each chunk stay in registers. part [group][z][x][y].
template <int N, bool ZB>
__global__ __launch_bounds__((DensTile<N>::NT)) __attribute__((amdgpu_waves_per_eu(2)))
void k_plane_density(const z64 *__restrict__ col, PlaneArgs p, const double *__restrict__ occ, int nb, int b0,
                     double *__restrict__ part, int first) {
    constexpr int A = DensTile<N>::A, B = DensTile<N>::B, NT = DensTile<N>::NT, C = DensTile<N>::C;
    constexpr int NCH = DensTile<N>::NCH, E = sizeof(z64), ldr = N | 1;
    constexpr int KC = DensTile<N>::ahead ? (N * N * 9 / 40 + NT - 1) / NT : 0;   // columns per thread fetched ahead
    constexpr int KY = (N * A * 53 / 100 + NT - 1) / NT;         // (s, ka) tasks per thread, roles in registers
    extern __shared__ __align__(16) unsigned char smem[];
    auto ld = [&](int a) -> z64 { return *reinterpret_cast<const z64 *>(smem + a); };
    auto st = [&](int a, z64 v) { *reinterpret_cast<z64 *>(smem + a) = v; };
    auto skip = [](int q) { return ZB && ZeroBand<B>::zero(q); };
    const int nslab = p.nslab, ebase = nslab * ldr * E, tw = ebase + (N - nslab) * C * E, zpos = tw + N * E;
    int tid = threadIdx.x;
    const int id = xcd_linear(blockIdx.x, gridDim.x), z = id / p.ngrp, grp = id - z * p.ngrp;
    const int vb0 = grp * p.bpw, vb1 = min(p.nvb, vb0 + p.bpw);
    const int c = tid % C, g = tid / C;
    const bool has_i = g < A, has_f = g < B;
    int io[B], fo[A];
    unsigned ip = 0, fp = 0;
#pragma unroll
    for (int q = 0; q < B; ++q) io[q] = p.xrow[B * min(g, A - 1) + q];
#pragma unroll
    for (int q = 0; q < A; ++q) fo[q] = p.xrow[min(g, B - 1) + B * q];
    for (int i = tid; i < N; i += NT) st(tw + i * E, static_cast<const z64 *>(p.tw1)[i]);
    if (tid == 0) st(zpos, czero<double>());
#pragma unroll
    for (int q = 0; q < B; ++q) {
        ip |= (io[q] >= 0 ? 1u : 0u) << q;
        io[q] = (io[q] >= 0 ? io[q] * ldr * E : ebase + (-1 - io[q]) * C * E) + c * E;
    }
#pragma unroll
    for (int q = 0; q < A; ++q) {
        fp |= (fo[q] >= 0 ? 1u : 0u) << q;
        fo[q] = (fo[q] >= 0 ? fo[q] * ldr * E : ebase + (-1 - fo[q]) * C * E) + c * E;
    }
    const int ny1 = nslab * A, ny2 = nslab * B;
    int ya[KY], yk[KY];
    unsigned ym[KY];
#pragma unroll
    for (int i = 0; i < KY; ++i) {
        const int t = min(tid + i * NT, ny1 - 1);
        yk[i] = t / nslab;
        ya[i] = ((t - yk[i] * nslab) * ldr + B * yk[i]) * E;
    }
    int kcur = -1, ncol = 0;
    const unsigned short *ymap = nullptr, *cpos = nullptr;
    int cp[KC > 0 ? KC : 1];
    z64 pre[KC > 0 ? KC : 1];
    auto column_mask = [&](int ka, int s) {
        unsigned m[B], r = 0;
#pragma unroll
        for (int q = 0; q < B; ++q) m[q] = ymap[(B * ka + q) * nslab + s];
#pragma unroll
        for (int q = 0; q < B; ++q) r |= (m[q] != 0xffffu ? 1u : 0u) << q;
        return r;
    };
    auto load_map = [&](int vb) {
        const int k = vb / p.bbt;
        if (k == kcur) return;
        kcur = k;
        ymap = p.kd[k].ymap;
        cpos = p.kd[k].cpos;
        ncol = p.kd[k].ncol;
#pragma unroll
        for (int i = 0; i < KC; ++i) cp[i] = cpos[min(tid + i * NT, ncol - 1)] * E;
#pragma unroll
        for (int i = 0; i < KY; ++i) ym[i] = column_mask(yk[i], min(tid + i * NT, ny1 - 1) - yk[i] * nslab);
    };
    auto source = [&](int vb) { return col + ((int64_t)vb * p.n3 + z) * p.ldc; };
    auto fetch = [&](int vb) {
        const z64 *src = source(vb);
#pragma unroll
        for (int i = 0; i < KC; ++i) pre[i] = at(src, (uint32_t)min(tid + i * NT, ncol - 1) * (uint32_t)E);
    };
    auto scatter = [&](int vb) {
#pragma unroll
        for (int i = 0; i < KC; ++i)
            if (tid + i * NT < ncol) st(cp[i], pre[i]);
        const z64 *src = source(vb);
        for (int i = tid + KC * NT; i < ncol; i += NT) st(cpos[i] * E, src[i]);
    };
    auto y1 = [&](int a, int ka, unsigned m) {
        z64 v[B];
#pragma unroll
        for (int q = 0; q < B; ++q)
            if (!skip(q)) v[q] = ld((m >> q) & 1u ? a + q * E : zpos);
        if constexpr (ZB) RegDftZ<B, double>::run(v);
        else RegDft<B, +1, double>::run(v);
#pragma unroll
        for (int q = 1; q < B; ++q) v[q] = cmul(v[q], ld(tw + (q * A + ka) * E));
#pragma unroll
        for (int q = 0; q < B; ++q) st(a + q * E, v[q]);
    };
    double acc[NCH][A];
#pragma unroll
    for (int h = 0; h < NCH; ++h)
#pragma unroll
        for (int q = 0; q < A; ++q) acc[h][q] = 0.0;
    load_map(vb0);
    fetch(vb0);
    scatter(vb0);
    for (int vb = vb0; vb < vb1; ++vb) {
        const double w = occ[(int64_t)kcur * nb + b0 + vb - kcur * p.bbt];
#pragma unroll
        for (int i = 0; i < KY; ++i) {
            opaque(ya[i]);
            opaque(yk[i]);
            opaque(ym[i]);
        }
        opaque(tid);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < KY; ++i)
            if (tid + i * NT < ny1) y1(ya[i], yk[i], ym[i]);
        for (int t = tid + KY * NT; t < ny1; t += NT) {
            const int ka = t / nslab, s = t - ka * nslab;
            y1((s * ldr + B * ka) * E, ka, column_mask(ka, s));
        }
        __syncthreads();
        for (int t = tid; t < ny2; t += NT) {
            const int jb = t / nslab, a = ((t - jb * nslab) * ldr + jb) * E;
            z64 v[A];
#pragma unroll
            for (int q = 0; q < A; ++q) v[q] = ld(a + q * B * E);
            RegDft<A, +1, double>::run(v);
#pragma unroll
            for (int q = 0; q < A; ++q) st(a + q * B * E, v[q]);
        }
        const int nxt = min(vb + 1, vb1 - 1);
        const bool same_k = nxt / p.bbt == kcur;
        if (same_k) fetch(nxt);
        __syncthreads();
#pragma unroll
        for (int h = 0; h < NCH; ++h) {
            // slots of chunk h: only slab rows move on from chunk to chunk
            if (has_i) {
                z64 v[B];
#pragma unroll
                for (int q = 0; q < B; ++q)
                    if (!skip(q)) v[q] = ld((ip >> q) & 1u ? io[q] + h * C * E : zpos);
                if constexpr (ZB) RegDftZ<B, double>::run(v);
                else RegDft<B, +1, double>::run(v);
#pragma unroll
                for (int q = 1; q < B; ++q) v[q] = cmul(v[q], ld(tw + (q * A + g) * E));
#pragma unroll
                for (int q = 0; q < B; ++q) st(io[q] + ((ip >> q) & 1u ? h * C * E : 0), v[q]);
            }
            __syncthreads();
            if (has_f) {
                z64 a[A];
#pragma unroll
                for (int q = 0; q < A; ++q) a[q] = ld(fo[q] + ((fp >> q) & 1u ? h * C * E : 0));
                RegDft<A, +1, double>::run(a);
#pragma unroll
                for (int q = 0; q < A; ++q) acc[h][q] += w * (a[q].re * a[q].re + a[q].im * a[q].im);
            }
            __syncthreads();
        }
        if (vb + 1 < vb1) {
            if (!same_k) {
                load_map(nxt);
                fetch(nxt);
            }
            scatter(nxt);
        }
    }
    if (!has_f) return;
    double *out = part + ((int64_t)grp * p.n3 + z) * N * N + g * N + c;
#pragma unroll
    for (int h = 0; h < NCH; ++h)
#pragma unroll
        for (int q = 0; q < A; ++q) {
            double *o = out + B * q * N + h * C;
            *o = first ? acc[h][q] : *o + acc[h][q];
        }
}

// rho [x][y][z] = sum over the groups, in order, of part [group][z][x][y]: 32 x 32 tiles of (y, z).
__global__ __launch_bounds__(256) void k_density_sum(const double *__restrict__ part, int G, int n1, int n2, int n3,
                                                     double *__restrict__ rho) {
    __shared__ double t[kVtTile][kVtTile + 1];
    const int x = blockIdx.z, y0 = blockIdx.x * kVtTile, z0 = blockIdx.y * kVtTile;
    const int64_t n = (int64_t)n1 * n2 * n3;
    const int u = threadIdx.x % kVtTile, w = threadIdx.x / kVtTile;
    constexpr int R = kVtTile * kVtTile / 256;
    double s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = 0.0;
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int z = min(z0 + w + 8 * r, n3 - 1), y = min(y0 + u, n2 - 1);
            s[r] += part[g * n + ((int64_t)z * n1 + x) * n2 + y];
        }
#pragma unroll
    for (int r = 0; r < R; ++r) t[w + 8 * r][u] = s[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = y0 + w + 8 * r, z = z0 + u;
        if (y < n2 && z < n3) rho[((int64_t)x * n2 + y) * n3 + z] = t[u][w + 8 * r];
    }
}

// Groups of bands per plane: the fewest rounds of work-groups times bands each (tables included, as
// plane_bands), up to kDensGroups partial grids.
constexpr int kDensGroups = 16;
static int dens_groups(int n3, int nvb, int slots) {
    int best = 1;
    double cost = 1e30;
    for (int g = 1; g <= std::min(kDensGroups, nvb); ++g) {
        const double t = ceil_div(n3 * g, slots) * (ceil_div(nvb, g) + 0.6);
        if (t < 0.999 * cost) {
            cost = t;
            best = g;
        }
    }
    return best;
}

template <int N> static bool dens_fits(const Plan &P) {
    return DensTile<N>::fits && dens_lds<N>(P.nslab) <= 160 * 1024;
}

template <int N, bool ZB>
static int launch_density_plane(const ColumnsCall &c, const double *occ, double *part, int G, int first) {
    const Plan &P = *c.P;
    if constexpr (!DensTile<N>::fits) {
        return set_error(ABACUS_PW_EINTERNAL, "density plane pass without a kernel");
    } else {
        auto kernel = k_plane_density<N, ZB>;
        static bool once = false;
        if (!once) {
            APW_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        160 * 1024));
            once = true;
        }
        const int nvb = c.nkb * c.ba.bbt, bpw = ceil_div(nvb, G), ngrp = ceil_div(nvb, bpw);
        PlaneArgs a{P.kdesc + c.k0, nullptr, P.tw64[0], P.tw64[1], P.xrow, P.nslab, P.ldc, N | 1, P.N3, nvb, c.ba.bbt, bpw,
                    ngrp, DensTile<N>::C};
        KernelTimer kt("density_plane", c.st);
        hipLaunchKernelGGL(kernel, dim3(P.N3 * ngrp), dim3(DensTile<N>::NT), dens_lds<N>(P.nslab), c.st,
                           static_cast<const z64 *>(c.col), a, occ, (int)c.ba.nb_total, c.ba.b0, part, first);
        return check_launch("density_plane");
    }
}

bool columns_density_fits(const Plan &P) {
    if (P.N1 != P.N2) return false;
    switch (P.N1) {
#define APW_CASE(n) case n: return dens_fits<n>(P);
        APW_LENGTHS(APW_CASE)
#undef APW_CASE
        default: return false;
    }
}

int columns_density_groups(const Plan &P, int nvb) {
    size_t lds = 1;
    int nt = 256;
    switch (P.N1) {
#define APW_CASE(n) case n: lds = dens_lds<n>(P.nslab); nt = DensTile<n>::NT; break;
        APW_LENGTHS(APW_CASE)
#undef APW_CASE
    }
    // as many as the bands of a group, rounded up, leave
    const int g = dens_groups(P.N3, nvb, 256 * std::max(1, std::min((int)(160 * 1024 / lds), 512 / nt)));
    return ceil_div(nvb, ceil_div(nvb, g));
}

int columns_density(const ColumnsCall &c, const double *occ, double *part, int G, int first) {
    const Plan &P = *c.P;
    const bool zb = P.zero_band[0] && P.zero_band[1];
    switch (P.N1) {
#define APW_CASE(n)                                                               \
    case n: return zb ? launch_density_plane<n, true>(c, occ, part, G, first) \
                      : launch_density_plane<n, false>(c, occ, part, G, first);
        APW_LENGTHS(APW_CASE)
#undef APW_CASE
        default:
            return set_error(ABACUS_PW_EBAD_FFT_SIZE, "unsupported grid length");
    }
}

int columns_density_sum(const Plan &P, const double *part, int G, double *rho, hipStream_t st) {
    KernelTimer kt("density_sum", st);
    hipLaunchKernelGGL(k_density_sum, dim3(ceil_div(P.N2, kVtTile), ceil_div(P.N3, kVtTile), P.N1), dim3(256), 0, st,
                       part, G, P.N1, P.N2, P.N3, rho);
    return check_launch("density_sum");
}

}  // namespace apw
