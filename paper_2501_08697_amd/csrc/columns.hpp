// Local-potential term of H psi through z columns (plane-wave KS equation,
// Sec. III.A; V_local of the pseudopotential split, Sec. II.A):
//
//   (V psi)(G) = (1/N) sum_j e^{-iG.r_j} V(r_j) sum_{G'} psi(G') e^{+iG'.r_j}
//
// as three passes whose intermediate is only the z columns that hold sphere
// points (about 0.2 of the grid, where the slab of whole planes in local.hip is
// half of it):
//   k_z_inv  C columns of one band per step: gather each column's sphere points,
//            inverse z transform, store as [z][column] rows (a plane z of a band
//            is one contiguous run of ncol values).
//   k_plane  one plane z of one band per step, resident in LDS: inverse y on the
//            slab rows, then per chunk of C y-columns inverse x, x V, forward x,
//            then forward y; the columns are read and written in place.
//   k_z_fwd  C columns: forward z, times 1/N, plus |k+G|^2 psi, scattered to H psi.
// HBM traffic per band: psi twice, H psi once, four passes over the columns; the
// slab passes move four times the slab, 2.5 times as much.
#pragma once

#include "fft_device.hpp"
#include "plan.hpp"

namespace apw {

template <typename T> __device__ __forceinline__ cx<T> czero() { return cx<T>{T(0), T(0)}; }

// A band batch spread over the k-points [k0, k0 + nk) of a call: at every k the
// bands [b0, b0 + bbt) of that k's [nb_total][npw_k] block; off0 = pw_off[k0].
struct BatchArgs {
    int64_t nb_total;
    int64_t off0;
    int b0;
    int bbt;
};

// Columns of a z-pass work-group: one task per thread in both phases (C max(A, B) <= 256),
// a multiple of 8 so that a row segment of the column buffer is whole 128-byte lines.
template <int N> struct ZTile {
    static constexpr int A = LdsSplit<N>::A, B = LdsSplit<N>::B, M = A > B ? A : B;
    static constexpr int C = 256 / M / 8 * 8 > 32 ? 32 : 256 / M / 8 * 8;
    static constexpr int NT = (C * M + 63) / 64 * 64;
};

// Logical id of block w of the first W blocks, consecutive ids on one XCD (as xcd_block).
__device__ __forceinline__ int xcd_linear(int w, int W) {
    const int per = W / kNumXcd;
    return w < per * kNumXcd ? (w % kNumXcd) * per + w / kNumXcd : w;
}

// Element at a 32-bit byte offset from a wave-uniform base: the address is a scalar pair plus one
// vector register, where indexing a pointer would take two registers per element.
template <typename T> __device__ __forceinline__ T at(const T *base, uint32_t off) {
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + off);
}
template <typename T> __device__ __forceinline__ void put(T *base, uint32_t off, T v) {
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + off) = v;
}

// Hides where a value came from, so that what is computed from it in a loop is computed
// there: hoisted out of the band loop, the address arithmetic of a dozen LDS slots held
// more registers than the transform itself.
__device__ __forceinline__ void opaque(int &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void opaque(unsigned &x) { asm volatile("" : "+v"(x)); }
// A twiddled value as it would come out of LDS: its multiply-adds are not fused with the
// sums that follow, so the transforms round as lds_fft's do.
template <typename T> __device__ __forceinline__ cx<T> rounded(cx<T> a) {
    asm("" : "+v"(a.re));
    asm("" : "+v"(a.im));
    return a;
}

template <int S> struct Sign { static constexpr int value = S; };

constexpr int kVtTile = 32;   // V transposition tile

// One tile of V [N1][N2][N3] (float64) into vt [N3][N1][N2] (T), so that a plane z reads
// contiguous rows. Run by extra work-groups of the z pass before k_plane.
template <typename T>
__device__ __forceinline__ void transpose_v(const double *__restrict__ v, T *__restrict__ vt, int n1, int n2, int n3,
                                            int tile, T *lds) {
    const int ty = (n2 + kVtTile - 1) / kVtTile, tz = (n3 + kVtTile - 1) / kVtTile;
    const int x = tile / (ty * tz), r = tile - x * ty * tz;
    const int y0 = (r / tz) * kVtTile, z0 = (r % tz) * kVtTile;
    for (int i = threadIdx.x; i < kVtTile * kVtTile; i += blockDim.x) {
        const int y = y0 + i / kVtTile, z = z0 + i % kVtTile;
        if (y < n2 && z < n3) lds[(i / kVtTile) * (kVtTile + 1) + i % kVtTile] = static_cast<T>(v[((int64_t)x * n2 + y) * n3 + z]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kVtTile * kVtTile; i += blockDim.x) {
        const int z = z0 + i / kVtTile, y = y0 + i % kVtTile;
        if (y < n2 && z < n3) vt[((int64_t)z * n1 + x) * n2 + y] = lds[(i % kVtTile) * (kVtTile + 1) + i / kVtTile];
    }
}

// ------------------------------------------------------------- z passes ----
// Block id -> (column group, k-point, bands of the batch). The column groups of one band
// range are consecutive, so they share an L2 and with it the lines of that band's psi
// (sphere order scatters a column's points over the whole row).
__device__ __forceinline__ void z_block(const KDesc *kd, const BatchArgs &ba, int ngrp, int bpw, int id, KDesc &D,
                                        int &k, int &lb0, int &lb1, int &grp) {
    const int gpk = (ba.bbt + bpw - 1) / bpw;
    const int by = id / ngrp;
    grp = id - by * ngrp;
    k = by / gpk;
    const int g = by - k * gpk;
    D = kd[k];
    lb0 = g * bpw;
    lb1 = min(ba.bbt, lb0 + bpw);
}

// ZB: the slots of ZeroBand hold no sphere point for any column (nothing is loaded for them).
template <int N, typename T, typename TIN, bool ZB>
__global__ __launch_bounds__((ZTile<N>::NT)) void k_z_inv(const cx<TIN> *__restrict__ psi_all,
                                                          const KDesc *__restrict__ kd, BatchArgs ba,
                                                          const cx<T> *__restrict__ tw_g, cx<T> *__restrict__ col,
                                                          int ldc, int ngrp, int bpw, int nblk,
                                                          const double *__restrict__ v, T *__restrict__ vt, int n1,
                                                          int n2) {
    constexpr int A = ZTile<N>::A, B = ZTile<N>::B, C = ZTile<N>::C;
    constexpr size_t kBytes = sizeof(cx<T>) * N * C > sizeof(T) * kVtTile * (kVtTile + 1) ? sizeof(cx<T>) * N * C
                                                                                        : sizeof(T) * kVtTile * (kVtTile + 1);
    __shared__ __align__(16) unsigned char smem[kBytes];
    if ((int)blockIdx.x >= nblk) {
        transpose_v<T>(v, vt, n1, n2, N, blockIdx.x - nblk, reinterpret_cast<T *>(smem));
        return;
    }
    cx<T> *buf = reinterpret_cast<cx<T> *>(smem);   // [slot][C]
    KDesc D;
    int kk, b0, b1, grp;
    z_block(kd, ba, ngrp, bpw, xcd_linear(blockIdx.x, nblk), D, kk, b0, b1, grp);
    const int c0 = grp * C;
    if (c0 >= D.ncol) return;
    const cx<TIN> *psi = psi_all + ba.nb_total * (D.pw_off - ba.off0) + (int64_t)ba.b0 * D.npw;
    const int64_t ld = D.npw;
    const int tid = threadIdx.x, c = tid % C, g = tid / C;   // g: ka in phase 1, jb in phase 2
    const bool live = c0 + c < D.ncol, has_ka = live && g < A, has_jb = live && g < B;
    // psi index of the thread's B slots (-1: no sphere point there) and its twiddles, kept for every band
    // (every load of this kernel is unconditional, from a clamped address where the slot is empty:
    // a load in a branch of its own waits for the one before it)
    const int cc = live ? c0 + c : c0, gc = min(g, A - 1);
    int zs[B];
    uint32_t off[B];
    unsigned has = 0;
    cx<T> tw[B];
#pragma unroll
    for (int q = 0; q < B; ++q) {
        zs[q] = ZB && ZeroBand<B>::zero(q) ? -1 : D.zslot[(B * gc + q) * ldc + cc];
        tw[q] = tw_g[q * A + gc];
    }
#pragma unroll
    for (int q = 0; q < B; ++q) {
        has |= (zs[q] >= 0 ? 1u : 0u) << q;
        off[q] = (uint32_t)max(zs[q], 0) * (uint32_t)sizeof(cx<TIN>);
    }
    cx<TIN> pre[B];
#pragma unroll
    for (int q = 0; q < B; ++q)
        if (!(ZB && ZeroBand<B>::zero(q))) pre[q] = at(psi + b0 * ld, off[q]);
    const uint32_t oc = (uint32_t)(g * ldc + c0 + c) * (uint32_t)sizeof(cx<T>);
    const uint32_t ostep = (uint32_t)(B * ldc) * (uint32_t)sizeof(cx<T>);
    for (int b = b0; b < b1; ++b) {
        if (has_ka) {
            cx<T> z[B];
#pragma unroll
            for (int q = 0; q < B; ++q)
                if (!(ZB && ZeroBand<B>::zero(q))) z[q] = (has >> q) & 1u ? cvt<T>(pre[q]) : czero<T>();
#pragma unroll
            for (int q = 0; q < B; ++q)
                if (!(ZB && ZeroBand<B>::zero(q))) pre[q] = at(psi + min(b + 1, b1 - 1) * ld, off[q]);
            if constexpr (ZB) RegDftZ<B, T>::run(z);
            else RegDft<B, +1, T>::run(z);
            buf[(B * g) * C + c] = z[0];
#pragma unroll
            for (int q = 1; q < B; ++q) buf[(B * g + q) * C + c] = cmul(z[q], tw[q]);
        }
        __syncthreads();
        if (has_jb) {
            cx<T> a[A];
#pragma unroll
            for (int q = 0; q < A; ++q) a[q] = buf[(B * q + g) * C + c];
            RegDft<A, +1, T>::run(a);
            cx<T> *o = col + (int64_t)(kk * ba.bbt + b) * N * ldc;
#pragma unroll
            for (int q = 0; q < A; ++q) put(o, oc + q * ostep, a[q]);
        }
        __syncthreads();
    }
}

template <int N, typename T, typename TIO, bool ZB>
__global__ __launch_bounds__((ZTile<N>::NT)) void k_z_fwd(const cx<T> *__restrict__ col, int ldc,
                                                          const KDesc *__restrict__ kd, BatchArgs ba,
                                                          const cx<T> *__restrict__ tw_g,
                                                          const cx<TIO> *__restrict__ psi_all,
                                                          cx<TIO> *__restrict__ hpsi_all, double inv_n, int ngrp,
                                                          int bpw) {
    constexpr int A = ZTile<N>::A, B = ZTile<N>::B, C = ZTile<N>::C;
    __shared__ cx<T> buf[N * C];   // [slot][C]
    KDesc D;
    int kk, b0, b1, grp;
    z_block(kd, ba, ngrp, bpw, xcd_linear(blockIdx.x, gridDim.x), D, kk, b0, b1, grp);
    const int c0 = grp * C;
    if (c0 >= D.ncol) return;
    const int64_t koff = ba.nb_total * (D.pw_off - ba.off0) + (int64_t)ba.b0 * D.npw;
    const cx<TIO> *psi = psi_all + koff;
    cx<TIO> *hpsi = hpsi_all + koff;
    const int64_t ld = D.npw;
    const int tid = threadIdx.x, c = tid % C, g = tid / C;   // g: jb in phase 1, ka in phase 2
    const bool live = c0 + c < D.ncol, has_ka = live && g < A, has_jb = live && g < B;
    __shared__ cx<T> tw[N];
    for (int i = tid; i < N; i += ZTile<N>::NT) tw[i] = tw_g[i];
    const int cc = live ? c0 + c : c0, gc = min(g, A - 1);
    int zs[B];
    uint32_t off[B];
    unsigned has = 0;
    TIO kq[B];
#pragma unroll
    for (int q = 0; q < B; ++q) zs[q] = ZB && ZeroBand<B>::zero(q) ? -1 : D.zslot[(B * gc + q) * ldc + cc];
#pragma unroll
    for (int q = 0; q < B; ++q) {
        has |= (zs[q] >= 0 && has_ka ? 1u : 0u) << q;
        off[q] = (uint32_t)max(zs[q], 0) * (uint32_t)sizeof(cx<TIO>);
    }
#pragma unroll
    for (int q = 0; q < B; ++q)
        if (!(ZB && ZeroBand<B>::zero(q))) kq[q] = static_cast<TIO>(D.kin[off[q] / (uint32_t)sizeof(cx<TIO>)]);
    const TIO sc = static_cast<TIO>(inv_n);
    const uint32_t oc = (uint32_t)(g * ldc + c0 + c) * (uint32_t)sizeof(cx<T>);
    const uint32_t ostep = (uint32_t)(B * ldc) * (uint32_t)sizeof(cx<T>);
    for (int b = b0; b < b1; ++b) {
        if (has_jb) {
            const cx<T> *src = col + (int64_t)(kk * ba.bbt + b) * N * ldc;
            cx<T> a[A];
#pragma unroll
            for (int q = 0; q < A; ++q) a[q] = at(src, oc + q * ostep);
            RegDft<A, -1, T>::run(a);
#pragma unroll
            for (int q = 0; q < A; ++q) buf[(g + B * q) * C + c] = a[q];
        }
        cx<TIO> x[B];
#pragma unroll
        for (int q = 0; q < B; ++q)
            if (!(ZB && ZeroBand<B>::zero(q))) x[q] = at(psi + b * ld, off[q]);
        __syncthreads();
        if (has_ka) {
            cx<T> z[B];
            z[0] = buf[(B * g) * C + c];
#pragma unroll
            for (int q = 1; q < B; ++q) z[q] = rounded(cmulc(buf[(B * g + q) * C + c], tw[q * A + g]));
            RegDft<B, -1, T>::run(z);
#pragma unroll
            for (int q = 0; q < B; ++q)
                if (!(ZB && ZeroBand<B>::zero(q)) && ((has >> q) & 1u)) {
                    const cx<TIO> w = cvt<TIO>(z[q]);
                    put(hpsi + b * ld, off[q], cx<TIO>{kq[q] * x[q].re + sc * w.re, kq[q] * x[q].im + sc * w.im});
                }
        }
        __syncthreads();
    }
}

// ----------------------------------------------------------- plane pass ----
struct PlaneArgs {
    const KDesc *kd;        // first k-point of the batch
    const void *vt;         // V [N3][N1][N2]
    const void *tw1, *tw2;  // twiddles of the x and y transforms
    const int *xrow;        // [N1] slot of the x transform -> slab row, or -1 - (rank among the slots without one)
    int nslab, ldc, ldr;    // slab rows; column buffer row; LDS row (odd)
    int n3, nvb, bbt;       // planes, virtual bands (k-point, band) and bands per k-point of the batch
    int bpw, ngrp, C;       // bands per work-group, band groups, y-columns per chunk (divides N2)
};

// Threads of a plane work-group: 512 where a plane (at the usual n1 / 2 slab rows) takes more
// than half of a CU's LDS and is alone there, else 256, two or more to a CU.
constexpr int plane_threads(int n1, int n2) { return n1 * n2 >= 96 * 96 ? 512 : 256; }

// One work-group per (plane z, group of bands). LDS holds the plane's slab rows [nslab][ldr]
// (all N2 values of every x frequency that has sphere points; ldr odd, so that lanes on
// consecutive rows use different banks) and, for the chunk of y-columns that is in the x
// transform, the [N1 - nslab][C] values that have no slab row: the x transform runs in
// place over both. Phases of a band (N1 = A1 B1, N2 = A2 B2, tasks over all threads):
//   S   the plane's columns (fetched behind the band before) to their slots
//   Y1 (s, ka)  slots of row s (zero where it has no column), inverse DFT_B2, twiddle
//   Y2 (s, jb)  inverse DFT_A2: natural y
//   per chunk:  I (c, ka) inverse DFT_B1 of slots B1 ka + kb, twiddle
//               F (c, jb) inverse DFT_A1, times V, forward DFT_A1
//               O (c, ka) twiddle, forward DFT_B1, kept where the slot has a slab row
//   Y1' (s, jb) forward DFT_A2
//   Y2' (s, ka) twiddle, forward DFT_B2
//   G   the slots that are columns back to the column buffer
// Every phase writes the slots it read, O of a chunk and I of the next touch only the
// thread's own slots, and so do G and the next S: two barriers per chunk and six more a
// band. The forward twiddles are applied by the (c, ka) and (s, ka) tasks. LDS addresses
// are kept in bytes, so an access costs no arithmetic beyond its step. ZB: the slots of
// ZeroBand are empty in x and in y for every column, so the inverse codelets skip them and
// the forward ones do not compute them.
template <int N1, int N2, typename T, bool ZB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
void k_plane(cx<T> *__restrict__ col, PlaneArgs p) {
    constexpr int A1 = LdsSplit<N1>::A, B1 = LdsSplit<N1>::B, A2 = LdsSplit<N2>::A, B2 = LdsSplit<N2>::B;
    // columns per thread fetched ahead: those of a sphere of the grid's quarter radius (pi / 16 of a
    // plane), with some margin, over the work-group size plane_shape takes at this length
    constexpr int KC = (N1 * N2 * 9 / 40 + plane_threads(N1, N2) - 1) / plane_threads(N1, N2);
    // (s, ka) tasks per thread with their roles in registers (at about N1 / 2 slab rows)
    constexpr int KY = (N1 * A2 * 53 / 100 + plane_threads(N1, N2) - 1) / plane_threads(N1, N2);
    constexpr int KJ = 2;                        // (s, jb) tasks, likewise
    constexpr int E = sizeof(cx<T>);
    extern __shared__ __align__(16) unsigned char smem[];
    auto ld = [&](int a) -> cx<T> { return *reinterpret_cast<const cx<T> *>(smem + a); };
    auto st = [&](int a, cx<T> v) { *reinterpret_cast<cx<T> *>(smem + a) = v; };
    auto skip1 = [](int q) { return ZB && ZeroBand<B1>::zero(q); };
    auto skip2 = [](int q) { return ZB && ZeroBand<B2>::zero(q); };
    const int ldr = p.ldr, nslab = p.nslab, C = p.C;
    const int ebase = nslab * ldr * E, tw2 = ebase + (N1 - nslab) * C * E, tw1 = tw2 + N2 * E;
    const int zpos = tw1 + N1 * E;   // one zero, read for slots without a value
    int tid = threadIdx.x;
    const int NT = blockDim.x;
    const int id = xcd_linear(blockIdx.x, gridDim.x);   // the band groups of a plane share an L2, and V there
    const int z = id / p.ngrp, grp = id - z * p.ngrp;
    const int vb0 = grp * p.bpw, vb1 = min(p.nvb, vb0 + p.bpw);

    // x-transform role: LDS address of the thread's slots, which of them have a slab row
    // (loads first and unconditional, here and below: a load in a branch of its own waits
    // for the one before it)
    const int c = tid % C;
    int g = tid / C;
    const bool has_i = g < A1, has_f = g < B1;
    int io[B1], fo[A1];
    unsigned ip = 0, fp = 0;
#pragma unroll
    for (int q = 0; q < B1; ++q) io[q] = p.xrow[B1 * min(g, A1 - 1) + q];
#pragma unroll
    for (int q = 0; q < A1; ++q) fo[q] = p.xrow[min(g, B1 - 1) + B1 * q];
    // the task's twiddles, in registers where there is room for them
    constexpr bool kTwReg = N1 <= 120;
    cx<T> tx[kTwReg ? B1 : 1];
    if constexpr (kTwReg) {
#pragma unroll
        for (int q = 0; q < B1; ++q) tx[q] = static_cast<const cx<T> *>(p.tw1)[q * A1 + min(g, A1 - 1)];
    }
    for (int i = tid; i < N2; i += NT) st(tw2 + i * E, static_cast<const cx<T> *>(p.tw2)[i]);
    for (int i = tid; i < N1; i += NT) st(tw1 + i * E, static_cast<const cx<T> *>(p.tw1)[i]);
    if (tid == 0) st(zpos, czero<T>());
#pragma unroll
    for (int q = 0; q < B1; ++q) {
        ip |= (io[q] >= 0 ? 1u : 0u) << q;
        io[q] = (io[q] >= 0 ? io[q] * ldr * E : ebase + (-1 - io[q]) * C * E) + c * E;
    }
#pragma unroll
    for (int q = 0; q < A1; ++q) {
        fp |= (fo[q] >= 0 ? 1u : 0u) << q;
        fo[q] = (fo[q] >= 0 ? fo[q] * ldr * E : ebase + (-1 - fo[q]) * C * E) + c * E;
    }
    // step of a slot's address from chunk to chunk: only slab rows move on
    auto advance = [&](int d) {
#pragma unroll
        for (int q = 0; q < B1; ++q)
            if (!skip1(q)) io[q] += (ip >> q) & 1u ? d : 0;
#pragma unroll
        for (int q = 0; q < A1; ++q) fo[q] += (fp >> q) & 1u ? d : 0;
    };
    auto twx = [&](int q) -> cx<T> {
        if constexpr (kTwReg) return tx[q];
        else return ld(tw1 + (q * A1 + g) * E);
    };
    const T *vt = static_cast<const T *>(p.vt) + (int64_t)z * (N1 * N2);
    const int gv = min(g, B1 - 1) * N2 + c;

    // y-transform roles: (s, ka) tasks tid + i NT, their first slot, their ka and (per k-point)
    // which slots hold a column; (s, jb) tasks
    const int ny1 = nslab * A2, ny2 = nslab * B2;
    int ya[KY], yk[KY], yb[KJ];
    unsigned ym[KY];
#pragma unroll
    for (int i = 0; i < KY; ++i) {
        const int t = min(tid + i * NT, ny1 - 1);
        yk[i] = t / nslab;
        ya[i] = ((t - yk[i] * nslab) * ldr + B2 * yk[i]) * E;
    }
#pragma unroll
    for (int i = 0; i < KJ; ++i) {
        const int t = min(tid + i * NT, ny2 - 1), jb = t / nslab;
        yb[i] = ((t - jb * nslab) * ldr + jb) * E;
    }
    int kcur = -1, ncol = 0;
    const unsigned short *ymap = nullptr, *cpos = nullptr;
    int cp[KC];
    cx<T> pre[KC];
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
        for (int i = 0; i < KY; ++i) {
            const int t = min(tid + i * NT, ny1 - 1), s = t - yk[i] * nslab;
            unsigned m[B2];
#pragma unroll
            for (int q = 0; q < B2; ++q) m[q] = ymap[(B2 * yk[i] + q) * nslab + s];
            ym[i] = 0;
#pragma unroll
            for (int q = 0; q < B2; ++q) ym[i] |= (m[q] != 0xffffu ? 1u : 0u) << q;
        }
    };
    auto fetch = [&](int vb) {
        const cx<T> *src = col + ((int64_t)vb * p.n3 + z) * p.ldc;
#pragma unroll
        for (int i = 0; i < KC; ++i) pre[i] = at(src, (uint32_t)min(tid + i * NT, ncol - 1) * (uint32_t)E);
    };
    // inverse DFT_B2 of the B2 slots from a (mask m: those with a column), twiddle, in place
    auto y1 = [&](int a, int ka, unsigned m) {
        cx<T> v[B2];
#pragma unroll
        for (int q = 0; q < B2; ++q)
            if (!skip2(q)) v[q] = ld((m >> q) & 1u ? a + q * E : zpos);
        if constexpr (ZB) RegDftZ<B2, T>::run(v);
        else RegDft<B2, +1, T>::run(v);
        // (all twiddles are read before the first store: LDS reads are not moved over stores)
#pragma unroll
        for (int q = 1; q < B2; ++q) v[q] = cmul(v[q], ld(tw2 + (q * A2 + ka) * E));
#pragma unroll
        for (int q = 0; q < B2; ++q) st(a + q * E, v[q]);
    };
    auto y1f = [&](int a, int ka) {   // forward counterpart
        cx<T> v[B2];
        v[0] = ld(a);
#pragma unroll
        for (int q = 1; q < B2; ++q) v[q] = rounded(cmulc(ld(a + q * E), ld(tw2 + (q * A2 + ka) * E)));
        RegDft<B2, -1, T>::run(v);
#pragma unroll
        for (int q = 0; q < B2; ++q)
            if (!skip2(q)) st(a + q * E, v[q]);
    };
    // DFT_A2 of the slots a, a + B2, ..., in place
    auto y2 = [&](int a, auto sign) {
        cx<T> v[A2];
#pragma unroll
        for (int q = 0; q < A2; ++q) v[q] = ld(a + q * B2 * E);
        RegDft<A2, decltype(sign)::value, T>::run(v);
#pragma unroll
        for (int q = 0; q < A2; ++q) st(a + q * B2 * E, v[q]);
    };
    auto y2_all = [&](auto sign) {
#pragma unroll
        for (int i = 0; i < KJ; ++i)
            if (tid + i * NT < ny2) y2(yb[i], sign);
        for (int t = tid + KJ * NT; t < ny2; t += NT) {
            const int jb = t / nslab;
            y2(((t - jb * nslab) * ldr + jb) * E, sign);
        }
    };
    // S: the fetched columns of band vb to their slots
    auto scatter = [&](int vb) {
#pragma unroll
        for (int i = 0; i < KC; ++i)
            if (tid + i * NT < ncol) st(cp[i], pre[i]);
        const cx<T> *src = col + ((int64_t)vb * p.n3 + z) * p.ldc;
        for (int i = tid + KC * NT; i < ncol; i += NT) st(cpos[i] * E, src[i]);
    };
    load_map(vb0);
    fetch(vb0);
    scatter(vb0);
    for (int vb = vb0; vb < vb1; ++vb) {
        cx<T> *pl = col + ((int64_t)vb * p.n3 + z) * p.ldc;
#pragma unroll
        for (int i = 0; i < KY; ++i) {
            opaque(ya[i]);
            opaque(yk[i]);
            opaque(ym[i]);
        }
        opaque(tid);
        opaque(g);
        __syncthreads();
        // Y1
#pragma unroll
        for (int i = 0; i < KY; ++i)
            if (tid + i * NT < ny1) y1(ya[i], yk[i], ym[i]);
        for (int t = tid + KY * NT; t < ny1; t += NT) {
            const int ka = t / nslab, s = t - ka * nslab;
            unsigned m = 0;
#pragma unroll
            for (int q = 0; q < B2; ++q) m |= (ymap[(B2 * ka + q) * nslab + s] != 0xffff ? 1u : 0u) << q;
            y1((s * ldr + B2 * ka) * E, ka, m);
        }
        __syncthreads();
        y2_all(Sign<+1>{});
        __syncthreads();
        // x transform, chunk by chunk; off: first y-column of the chunk
        for (int off = 0; off <= N2; off += C) {
            if (has_i && off > 0) {   // O of the chunk before
                cx<T> v[B1];
                v[0] = ld(io[0]);
#pragma unroll
                for (int q = 1; q < B1; ++q) v[q] = rounded(cmulc(ld(io[q]), twx(q)));
                RegDft<B1, -1, T>::run(v);
#pragma unroll
                for (int q = 0; q < B1; ++q)
                    if (!skip1(q) && ((ip >> q) & 1u)) st(io[q], v[q]);
            }
            if (off == N2) break;
            if (off > 0) advance(C * E);
            if (has_i) {   // I
                cx<T> v[B1];
#pragma unroll
                for (int q = 0; q < B1; ++q)
                    if (!skip1(q)) v[q] = ld((ip >> q) & 1u ? io[q] : zpos);
                if constexpr (ZB) RegDftZ<B1, T>::run(v);
                else RegDft<B1, +1, T>::run(v);
                // (all twiddles are read before the first store: LDS reads are not moved over stores)
#pragma unroll
                for (int q = 1; q < B1; ++q) v[q] = cmul(v[q], twx(q));
#pragma unroll
                for (int q = 0; q < B1; ++q) st(io[q], v[q]);
            }
            T vr[A1];
            const uint32_t vo = (uint32_t)(gv + off) * (uint32_t)sizeof(T);
#pragma unroll
            for (int q = 0; q < A1; ++q) vr[q] = at(vt + B1 * q * N2, vo);
            __syncthreads();
            if (has_f) {   // F
                cx<T> a[A1];
#pragma unroll
                for (int q = 0; q < A1; ++q) a[q] = ld(fo[q]);
                RegDft<A1, +1, T>::run(a);
#pragma unroll
                for (int q = 0; q < A1; ++q) a[q] = a[q] * vr[q];
                RegDft<A1, -1, T>::run(a);
#pragma unroll
                for (int q = 0; q < A1; ++q) st(fo[q], a[q]);
            }
            __syncthreads();
        }
        advance(-(N2 - C) * E);
        __syncthreads();
        const int nxt = min(vb + 1, vb1 - 1);
        const bool same_k = nxt / p.bbt == kcur;
        fetch(same_k ? nxt : vb);
        y2_all(Sign<-1>{});
        __syncthreads();
        // Y2'
#pragma unroll
        for (int i = 0; i < KY; ++i)
            if (tid + i * NT < ny1) y1f(ya[i], yk[i]);
        for (int t = tid + KY * NT; t < ny1; t += NT) {
            const int ka = t / nslab;
            y1f(((t - ka * nslab) * ldr + B2 * ka) * E, ka);
        }
        __syncthreads();
        // G, and S of the next band between its reads and its stores to memory: a thread's slots
        // are its own, and S must not wait behind the stores for its columns
        cx<T> out[KC];
        const int n = ncol;
#pragma unroll
        for (int i = 0; i < KC; ++i) out[i] = ld(cp[i]);
        for (int i = tid + KC * NT; i < ncol; i += NT) pl[i] = ld(cpos[i] * E);
        if (!same_k) {
            load_map(nxt);
            fetch(nxt);
            __syncthreads();   // another sphere's slots: not the thread's own any more
        }
        if (vb + 1 < vb1) scatter(nxt);
#pragma unroll
        for (int i = 0; i < KC; ++i)
            if (tid + i * NT < n) put(pl, (uint32_t)(tid + i * NT) * (uint32_t)E, out[i]);
    }
}

// ------------------------------------------------------------ launchers ----
// One call's view of the column passes: the k-points [k0, k0 + nkb) of the batch ba.
struct ColumnsCall {
    const Plan *P;
    int k0, nkb;
    BatchArgs ba;
    void *col;          // [nkb bbt][N3][ldc] complex128 (complex64 in FP32)
    void *vt;           // V transposed
    hipStream_t st;
    int prec = 0;       // transforms, psi and H psi: 0 FP64, 1 FP32
};

// Chunk width and threads of k_plane, and its LDS bytes; C = 0 when the plane does not fit
// or its pair of lengths has no kernel.
struct PlaneShape {
    int C, NT, ldr;
    size_t lds;
};
PlaneShape plane_shape(const Plan &P, int fft_prec);
bool columns_pay(const Plan &P, int fft_prec);

int columns_inverse(const ColumnsCall &c, const void *psi, const double *v);
int columns_plane(const ColumnsCall &c);
int columns_forward(const ColumnsCall &c, const void *psi, void *hpsi);
// Band density of the batch's columns (columns_density.hip): whether the grid has a kernel, the
// partial grids for nvb bands, the plane pass (adding w |psi|^2 of its bands to part [G][N3][N1][N2];
// first: overwriting), and their sum. occ [nk][nb_total] from the call's first k-point.
bool columns_density_fits(const Plan &P);
int columns_density_groups(const Plan &P, int nvb);
int columns_density(const ColumnsCall &c, const double *occ, double *part, int G, int first);
int columns_density_sum(const Plan &P, const double *part, int G, double *rho, hipStream_t st);
// columns_plane in FP32: equal x and y lengths below kColumnsF32 (local_uses_columns has the reason)
constexpr int kColumnsF32 = 90;
int columns_plane_f32(const ColumnsCall &c);
// columns_plane for the grids with x length N1 (instantiated in columns_plane_*.hip)
template <int N1> int columns_plane_n1(const ColumnsCall &c);

}  // namespace apw
