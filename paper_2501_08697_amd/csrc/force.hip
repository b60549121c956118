// Nonlocal (Kleinman-Bylander) force on the atoms (abacus_pw_force_nl).
//
// Sec. III.A gives the nonlocal force as the derivative of the projector
// energy with respect to the atomic positions. The projectors of atom a carry
// the structure factor exp(-i (k+G).tau_a), so d beta / d tau_alpha =
// -i (k+G)_alpha beta, and with E_NL = sum_k sum_n occ[k][n] sum_a P_a^H D_a P_a:
//   F[a][alpha] = -dE_NL/dtau_{a,alpha}
//               = -2 sum_k sum_n occ[k][n] sum_{i,j in a} D_ij Im(conj(P^alpha_in) P_jn),
//   P = B^H psi,  P^alpha = B^H ((k+G)_alpha psi).
// The sum over bands comes first: with Q = D P and W_in = occ_n conj(Q_in),
//   sum_n occ_n Im(conj(P^alpha_in) Q_in) = sum_G (k+G)_alpha Im(beta_i(G) conj(X_i(G))),
//   X_i(G) = sum_n W_in psi_n(G),
// so a k-point costs the projection P and one product of the same size whose epilogue contracts
// X with beta and k+G, instead of projecting psi, k_x psi, k_y psi and k_z psi. 72^3, 256
// projectors x 128 bands: 403 us with a stacked operator of 4 x 256 rows, 218 us now. The
// partial sums over tiles of G are added in a fixed order, k-points in order.
#include <algorithm>

#include "gemm.hpp"
#include "hamiltonian.hpp"

namespace apw {

namespace {

constexpr int kMaxAtomProj = 16;   // projectors per atom handled by the reduction

// W[n][i] = occ[n] conj(sum_j D_ij P[n][j]) (P, W [nb][nproj]); the D-block tables of the plan. Only for
// more projectors than proj_weights takes (it forms W as it sums the splits, one launch instead of two).
__global__ __launch_bounds__(256) void k_force_w(int nb, int nproj, const z64 *__restrict__ P,
                                                 const double *__restrict__ occ, const double *__restrict__ dmat,
                                                 const int *__restrict__ blo, const int *__restrict__ bn,
                                                 const int *__restrict__ bdoff, z64 *__restrict__ W) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)nb * nproj) return;
    const int n = (int)(t / nproj), i = (int)(t - (int64_t)n * nproj);
    const int lo = blo[i], na = bn[i];
    const double *d = dmat + bdoff[i] + (int64_t)(i - lo) * na;
    const z64 *row = P + (int64_t)n * nproj + lo;
    z64 q{0.0, 0.0};
    for (int j = 0; j < na; ++j) q = q + row[j] * d[j];
    const double w = occ[n];
    W[t] = z64{w * q.re, -w * q.im};
}

// One work-group per atom: force[a][al] (=, or += when accumulate) -2 sum over its projectors and
// the tiles of part [ntile][nproj][3].
__global__ __launch_bounds__(256) void k_force_reduce(int ntile, int nproj, const double *__restrict__ part,
                                                      const int *__restrict__ aoff, double *__restrict__ force,
                                                      int accumulate) {
    const int a = blockIdx.x, lo = aoff[a], m = 3 * (aoff[a + 1] - lo);
    // entry e = 3 (i - lo) + al of a tile is contiguous: thread t takes entry t % m, so its
    // direction stays the same, of the tiles t / m, t / m + step, ...
    __shared__ double red[256];
    const int step = 256 / m, e = threadIdx.x % m, t0 = threadIdx.x / m;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};   // four independent chains
    if (t0 < step) {
        const double *src = part + 3 * (int64_t)lo + e;
        int t = t0;
        for (; t + 3 * step < ntile; t += 4 * step)
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] += src[(int64_t)(t + u * step) * 3 * nproj];
        for (int u = 0; t < ntile; t += step, ++u) acc[u] += src[(int64_t)t * 3 * nproj];
    }
    red[threadIdx.x] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    __syncthreads();
    if (threadIdx.x < 3) {
        double s = 0.0;
        for (int q = threadIdx.x; q < step * m; q += 3) s += red[q];
        double *o = force + 3 * (int64_t)a + threadIdx.x;
        *o = accumulate ? *o - 2.0 * s : -2.0 * s;
    }
}

__global__ void k_force_zero(int n, double *__restrict__ f) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) f[i] = 0.0;
}

int force_tables(const abacus_pw_problem &p, Plan &P, hipStream_t st) {
    if (P.force_tab_ready) return ABACUS_PW_OK;
    std::vector<double> kg(3 * (size_t)P.npw_total);
    for (int k = 0; k < P.nk; ++k) {
        const int *mk = p.miller + 3 * P.pw_off[k];
        const double *kv = p.kpts + 3 * k;
        for (int g = 0; g < P.npw[k]; ++g) {
            const int *m = mk + 3 * g;
            double *o = kg.data() + 3 * (size_t)(P.pw_off[k] + g);
            for (int c = 0; c < 3; ++c) o[c] = kv[c] + m[0] * P.recip[c] + m[1] * P.recip[3 + c] + m[2] * P.recip[6 + c];
        }
    }
    const size_t kb = sizeof(double) * kg.size(), ab = sizeof(int) * P.proj_atom_offset.size();
    APW_TRY(P.force_tab.ensure(kb + ab));
    APW_HIP(hipMemcpyAsync(P.force_tab.ptr, kg.data(), kb, hipMemcpyHostToDevice, st));
    APW_HIP(hipMemcpyAsync(P.force_tab.as<char>() + kb, P.proj_atom_offset.data(), ab, hipMemcpyHostToDevice, st));
    APW_HIP(hipStreamSynchronize(st));   // the host vectors go out of scope
    P.force_tab_ready = true;
    return ABACUS_PW_OK;
}

}  // namespace

int force_nl_all(const abacus_pw_problem &p, Plan &P, int nb, const void *psi, const double *occ, double *force,
                 hipStream_t st) {
    if (P.natom == 0) return ABACUS_PW_OK;
    if (P.nproj == 0) {   // no projectors: no nonlocal force
        hipLaunchKernelGGL(k_force_zero, dim3(ceil_div(3 * P.natom, 256)), dim3(256), 0, st, 3 * P.natom, force);
        return check_launch("force_zero");
    }
    for (int a = 0; a < P.natom; ++a)
        if (P.proj_atom_offset[a + 1] - P.proj_atom_offset[a] > kMaxAtomProj)
            return set_error(ABACUS_PW_EBAD_SHAPE, "more than 16 projectors on one atom");
    APW_TRY(force_tables(p, P, st));
    const double *kg_all = P.force_tab.as<double>();
    const int *aoff = reinterpret_cast<const int *>(P.force_tab.as<char>() + sizeof(double) * 3 * (size_t)P.npw_total);
    const size_t pq = sizeof(z64) * (size_t)P.nproj * nb;
    if (!proj_weights_fit(P.nproj)) APW_TRY(P.proj.ensure(pq));
    APW_TRY(P.proj2.ensure(pq));
    APW_TRY(P.gemm_part.ensure(std::max(gemm_cn_part_bytes(P.nproj, nb, P.max_npw, 16, g_splitk_chunk),
                                        sizeof(double) * 3 * (size_t)P.nproj * force_contract_tiles(P.max_npw))));
    for (int k = 0; k < P.nk; ++k) {
        const KTables &K = P.k[k];
        const z64 *bk = static_cast<const z64 *>(p.beta) + (size_t)P.nproj * K.pw_off;
        const z64 *xk = static_cast<const z64 *>(psi) + (size_t)nb * K.pw_off;
        if (proj_weights_fit(P.nproj)) {
            APW_TRY(proj_weights(P.nproj, nb, K.npw, bk, xk, occ + (size_t)k * nb, static_cast<const double *>(p.dmat),
                                 P.proj_blk_lo, P.proj_blk_n, P.proj_blk_doff, P.proj2.ptr, P.gemm_part.ptr,
                                 g_splitk_chunk, st));
        } else {
            APW_TRY(gemm_cn(0, P.nproj, nb, K.npw, bk, K.npw, xk, K.npw, P.proj.ptr, P.nproj, 1.0, 0.0, P.gemm_part.ptr,
                            g_splitk_chunk, st));
            KernelTimer kt("force_w", st);
            hipLaunchKernelGGL(k_force_w, dim3((unsigned)ceil_div64((int64_t)nb * P.nproj, 256)), dim3(256), 0, st, nb,
                               P.nproj, P.proj.as<z64>(), occ + (size_t)k * nb, static_cast<const double *>(p.dmat),
                               P.proj_blk_lo, P.proj_blk_n, P.proj_blk_doff, P.proj2.as<z64>());
            APW_TRY(check_launch("force_w"));
        }
        APW_TRY(force_contract(P.nproj, K.npw, nb, P.proj2.ptr, xk, bk, kg_all + 3 * K.pw_off, P.gemm_part.as<double>(),
                               st));
        KernelTimer kt("force_reduce", st);
        hipLaunchKernelGGL(k_force_reduce, dim3(P.natom), dim3(256), 0, st, force_contract_tiles(K.npw), P.nproj,
                           P.gemm_part.as<double>(), aoff, force, k > 0 ? 1 : 0);
        APW_TRY(check_launch("force_reduce"));
    }
    return ABACUS_PW_OK;
}

}  // namespace apw
