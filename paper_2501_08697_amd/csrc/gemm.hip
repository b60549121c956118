// Complex GEMMs on the matrix cores (MFMA) for the Kleinman-Bylander term
// sum_ij |beta_i> D_ij <beta_j| psi (Sec. II.A) and for the Davidson subspace
// products. Two shapes cover every use, both with K-contiguous row vectors:
//
//   CN  C[j][i] = alpha * sum_k conj(A[i][k]) B[j][k] + beta * C[j][i]
//       (projections <a_i|b_j>; K = npw is long, so K is split across
//        work-groups and the partial tiles are summed in a fixed order)
//   NN  C[j][g] = alpha * sum_i A[j][i] B[i][g] + beta * C[j][g]
//       (combinations of basis vectors: Y += B Q, Psi = V Y)
//
// Tiles: a 256-thread work-group owns a 64 x 64 output tile; each of its four
// waves a 32 x 32 quarter as 2 x 2 blocks of 16 x 16 MFMA results. A complex
// product takes three real products (3M: ar br, ai bi and the product of the
// sums, from which the real and imaginary parts follow), so each block keeps
// three accumulators. Operands are staged in LDS (16 k per stage). FP64 uses v_mfma_f64_16x16x4f64, FP32 v_mfma_f32_16x16x4f32;
// both take one value of A and of B per lane (A[i][k] at lane i + 16 k, B[k][j]
// at lane j + 16 k) and return four values per lane in column j = lane % 16.
// The row of element e differs: the FP64 instruction interleaves rows
// (i = lane / 16 + 4 e), the FP32 one blocks them (i = 4 (lane / 16) + e);
// Acc<T>::row encodes this (measured on gfx950).
#include <algorithm>

#include "common.hpp"
#include "gemm.hpp"

namespace apw {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T> struct Acc;
template <> struct Acc<double> {
    using V = d4;
    __device__ static V zero() { return V{0.0, 0.0, 0.0, 0.0}; }
    __device__ static V mma(double a, double b, V c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    __device__ static int row(int lane, int e) { return (lane >> 4) + 4 * e; }
};
template <> struct Acc<float> {
    using V = f4;
    __device__ static V zero() { return V{0.f, 0.f, 0.f, 0.f}; }
    __device__ static V mma(float a, float b, V c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    __device__ static int row(int lane, int e) { return 4 * (lane >> 4) + e; }
};

constexpr int TM = 64, TN = 64, KT = 16, KP = KT + 1;
constexpr int kMaxBatch = kGemmMaxBatch;   // products of one launch
// Asking for at least two waves per SIMD makes the compiler keep the twelve
// accumulator blocks in ordinary VGPRs (166 in FP64, three waves per SIMD)
// instead of spreading them over VGPRs and AGPRs (278, one wave per SIMD).
constexpr int kGemmWaves = 2;

// ----------------------------------------------------------------- CN ------
// part[s][j][i] = sum over k in split s of conj(A[i][k]) B[j][k]
// TS is the type operands are stored in; they are rounded to T while staged
// (FP32 products of FP64 vectors for the reduced-precision subspace projection).
// Tile order: the blocks of one K chunk are logically consecutive (and so share an XCD's
// L2); inside a chunk they run in groups of gm row tiles by every column tile, so the
// tiles that run at the same time read few distinct A and B tiles while they move
// through K together (with the row tiles fastest, a chunk of a 2304 x 1024 product
// kept all 36 A tiles in flight and read 15.7x the operands).
// One launch covers up to kMaxBatch products of one shape M x N (the k-points of a call, whose
// K = npw differ): grid z counts their splits one after the other. A batch has room for NB, 1 or
// kMaxBatch, and keeps a product's fields together: what a launch looks up in its arguments it waits
// for before its first load. MIXED_FP32 H psi of 32 projectors x 16 bands at 32^3 (one product a launch)
// took 60.9 us with eight arrays of fields and a search in every launch, 59.0 so.
// herm: A and B are the same rows, so the result is Hermitian; tiles with i0 > j0 are left out
// and k_reduce fills them in from their mirror images (36 of 64 tiles at 512 x 512: the Gram
// matrix of 512 bands of 115k plane waves takes 2.05 ms, whole it took 2.95).
template <int NB> struct CnBatch {
    int n, z0[NB];                 // z0: first splits in grid z
    struct {
        int K, kchunk;
        int64_t lda, ldb, a, b;    // rows and element offsets of A and B
    } p[NB];
};
template <typename T, typename TS, int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kGemmWaves))) void k_gemm_cn_part(int M, int N, CnBatch<NB> bt, const cx<TS> *__restrict__ A,
                                                      const cx<TS> *__restrict__ B, cx<T> *__restrict__ part, int gm, int herm) {
    __shared__ cx<T> As[TM][KP];
    __shared__ cx<T> Bs[TN][KP];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int bx, by, bz;
    xcd_block(bx, by, bz);   // the tiles of one K chunk share an L2
    const int nm = gridDim.x, nn = gridDim.y;
    const int t = bx + nm * by;                        // tile of the chunk, in logical order
    const int grp = t / (gm * nn), first = grp * gm, rows = min(gm, nm - first);
    const int r = t - grp * gm * nn;
    const int i0 = (first + r % rows) * TM, j0 = (r / rows) * TN;
    if (herm && i0 > j0) return;
    int pb = 0;
    if constexpr (NB > 1)
        while (pb + 1 < bt.n && bz >= bt.z0[pb + 1]) ++pb;
    const int s = bz;   // the partial sums of the products follow each other
    const auto &pr = bt.p[pb];
    const int kb = (bz - bt.z0[pb]) * pr.kchunk, ke = min(pr.K, kb + pr.kchunk);
    const int64_t lda = pr.lda, ldb = pr.ldb;
    A += pr.a;
    B += pr.b;
    using AV = typename Acc<T>::V;
    AV c1[2][2], c2[2][2], c3[2][2];   // sums of ar br, ai bi, (ar - ai)(br + bi)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) c1[a][b] = c2[a][b] = c3[a][b] = Acc<T>::zero();
    const int lr = tid >> 2, lk = (tid & 3) * 4;   // loader: row, first k of 4
    const int wi = (w & 1) * 32, wj = (w >> 1) * 32;
    // loader rows past M (N) read the last row instead: they only feed outputs that are
    // never stored, and a whole stage then loads with no per-load branch (only the k tail
    // of a chunk is bounded, and zero-filled, since it enters every sum)
    const cx<TS> *ga = A + (int64_t)min(i0 + lr, M - 1) * lda + lk;
    const cx<TS> *gb = B + (int64_t)min(j0 + lr, N - 1) * ldb + lk;
    cx<T> ra[4], rb[4];
    auto load = [&](int k0) {
        if (k0 + KT <= ke) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ra[q] = cvt<T>(ga[k0 + q]);
                rb[q] = cvt<T>(gb[k0 + q]);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool in = k0 + lk + q < ke;
                ra[q] = in ? cvt<T>(ga[k0 + q]) : cx<T>{T(0), T(0)};
                rb[q] = in ? cvt<T>(gb[k0 + q]) : cx<T>{T(0), T(0)};
            }
        }
    };
    load(kb);
    for (int k0 = kb; k0 < ke; k0 += KT) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            As[lr][lk + q] = ra[q];
            Bs[lr][lk + q] = rb[q];
        }
        __syncthreads();
        if (k0 + KT < ke) load(k0 + KT);   // next stage in flight while this one multiplies
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int kk = 4 * q + (lane >> 4);
            cx<T> a[2], b[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) a[r] = As[wi + 16 * r + (lane & 15)][kk];
#pragma unroll
            for (int c = 0; c < 2; ++c) b[c] = Bs[wj + 16 * c + (lane & 15)][kk];
            T as[2], bs[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) as[r] = a[r].re - a[r].im;
#pragma unroll
            for (int c = 0; c < 2; ++c) bs[c] = b[c].re + b[c].im;
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    // conj(a) b with three real products:
                    //   re = ar br + ai bi,  im = (ar - ai)(br + bi) - ar br + ai bi
                    c1[r][c] = Acc<T>::mma(a[r].re, b[c].re, c1[r][c]);
                    c2[r][c] = Acc<T>::mma(a[r].im, b[c].im, c2[r][c]);
                    c3[r][c] = Acc<T>::mma(as[r], bs[c], c3[r][c]);
                }
        }
        __syncthreads();
    }
    cx<T> *out = part + (int64_t)s * N * M;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int gj = j0 + wj + 16 * c + (lane & 15);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int gi = i0 + wi + 16 * r + Acc<T>::row(lane, e);
                if (gi < M && gj < N)
                    out[(int64_t)gj * M + gi] = cx<T>{c1[r][c][e] + c2[r][c][e], c3[r][c][e] - c1[r][c][e] + c2[r][c][e]};
            }
        }
}

// C[j][i] = alpha * sum_s part[s][j][i] + beta * C[j][i]   (fixed summation order)
// A work-group takes kReduceThreads / groups elements; the splits are divided among its `groups`
// thread groups, each thread summing its own in four independent chains, and the group sums are
// added in order. Bound by the latency of the loads of a chain: 32 projectors x 16 bands in 425
// splits took 38 us (timed by events) with one thread per element, 8.4 with sixteen.
// herm (beta = 0): the tiles i0 > j0 hold nothing and become the conjugates of their mirror images.
constexpr int kReduceThreads = 256;
template <typename T, typename TC = T>
__global__ __launch_bounds__(kReduceThreads) void k_reduce(int M, int N, int nsplit, const cx<T> *__restrict__ part,
                                                           cx<TC> *__restrict__ C, int64_t ldc, double alpha,
                                                           double beta, int herm, int groups) {
    __shared__ z64 sums[kReduceThreads];
    const int per = kReduceThreads / groups, e = threadIdx.x % per, g = threadIdx.x / per;
    const int64_t idx = (int64_t)blockIdx.x * per + e;
    const int j = (int)(idx / M), i = (int)(idx - (int64_t)j * M);
    const bool live = idx < (int64_t)M * N && !(herm && i / TM > j / TN);
    const int64_t ss = (int64_t)M * N;
    double r4[4] = {0.0, 0.0, 0.0, 0.0}, i4[4] = {0.0, 0.0, 0.0, 0.0};   // four independent chains
    if (live) {
        int s = g;
        for (; s + 3 * groups < nsplit; s += 4 * groups) {
            cx<T> v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = part[(int64_t)(s + u * groups) * ss + idx];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                r4[u] += (double)v[u].re;
                i4[u] += (double)v[u].im;
            }
        }
        for (int u = 0; s < nsplit; s += groups, ++u) {
            const cx<T> v = part[(int64_t)s * ss + idx];
            r4[u] += (double)v.re;
            i4[u] += (double)v.im;
        }
    }
    double re = (r4[0] + r4[1]) + (r4[2] + r4[3]), im = (i4[0] + i4[1]) + (i4[2] + i4[3]);
    if (groups > 1) {
        sums[threadIdx.x] = z64{re, im};
        __syncthreads();
        if (g > 0) return;
        for (int q = 1; q < groups; ++q) {
            re += sums[q * per + e].re;
            im += sums[q * per + e].im;
        }
    }
    if (!live) return;
    cx<TC> *c = C + (int64_t)j * ldc + i;
    if (beta != 0.0) {
        re = alpha * re + beta * (double)c->re;
        im = alpha * im + beta * (double)c->im;
    } else {
        re *= alpha;
        im *= alpha;
    }
    *c = cx<TC>{(TC)re, (TC)im};
    if (herm && i / TM < j / TN) C[(int64_t)i * ldc + j] = cx<TC>{(TC)re, (TC)-im};
}

// Thread groups per element of k_reduce: a chain is at most four rounds of loads up to 256 splits
// (the default chunks make up to 512), and an element's partial sums stay runs of 256 bytes.
static int reduce_split_groups(int nsplit) { return nsplit <= 16 ? 1 : nsplit <= 64 ? 4 : 16; }

template <typename T, typename TC>
static int launch_reduce(int M, int N, int nsplit, const void *part, void *C, int64_t ldc, double alpha, double beta,
                         int herm, hipStream_t st) {
    const int groups = reduce_split_groups(nsplit);
    KernelTimer kt("gemm_reduce", st);
    hipLaunchKernelGGL((k_reduce<T, TC>), dim3((unsigned)ceil_div64((int64_t)M * N, kReduceThreads / groups)),
                       dim3(kReduceThreads), 0, st, M, N, nsplit, static_cast<const cx<T> *>(part),
                       static_cast<cx<TC> *>(C), ldc, alpha, beta, herm, groups);
    return check_launch("gemm_reduce");
}

// P[j][i] = sum_s part[s][j][i]; Q[j][i] = sum_t D_blk(i)[i - lo][t] P[j][lo + t], with occ (one product
// only) occ[j] times its conjugate instead.
// One work-group per band j. The splits are divided among G thread groups
// (G M <= blockDim.x), each thread summing its splits in four independent
// chains; the group sums are added in a fixed order, so the result does not
// depend on timing. P of the band is then in LDS for the D blocks.
constexpr int kRedThreads = 1024, kRedMaxGroups = 8;
__host__ __device__ inline int reduce_groups(int M) {
    return M <= 0 ? 1 : std::max(1, std::min(kRedMaxGroups, std::min(kRedThreads / M, 4096 / M)));
}

struct RedBatch {
    int z0[kMaxBatch + 1];   // splits [z0[p], z0[p + 1]) belong to product p
};
template <typename T>
__global__ __launch_bounds__(kRedThreads) void k_reduce_dapply(int M, RedBatch rb, const cx<T> *__restrict__ part,
                                                               int N, const double *__restrict__ dmat,
                                                               const int *__restrict__ blo, const int *__restrict__ bn,
                                                               const int *__restrict__ bdoff, cx<T> *__restrict__ P,
                                                               cx<T> *__restrict__ Q, const double *__restrict__ occ) {
    extern __shared__ __align__(16) unsigned char smem[];
    cx<double> *pl = reinterpret_cast<cx<double> *>(smem);   // [G][M] group sums, then the total in [0][M]
    const int j = blockIdx.x, pb = blockIdx.y, nsplit = rb.z0[pb + 1] - rb.z0[pb];
    const int G = reduce_groups(M);
    const int64_t sstride = (int64_t)N * M;
    part += rb.z0[pb] * sstride;
    Q += pb * sstride;
    if (P) P += pb * sstride;
    for (int idx = threadIdx.x; idx < G * M; idx += blockDim.x) {
        const int g = idx / M, i = idx - g * M;
        const cx<T> *src = part + (int64_t)j * M + i;
        double re[4] = {0.0, 0.0, 0.0, 0.0}, im[4] = {0.0, 0.0, 0.0, 0.0};
        int s = g;
        for (; s + 3 * G < nsplit; s += 4 * G) {
            cx<T> v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = src[(int64_t)(s + u * G) * sstride];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                re[u] += (double)v[u].re;
                im[u] += (double)v[u].im;
            }
        }
        for (int u = 0; s < nsplit; s += G, ++u) {
            const cx<T> v = src[(int64_t)s * sstride];
            re[u] += (double)v.re;
            im[u] += (double)v.im;
        }
        pl[idx] = cx<double>{(re[0] + re[1]) + (re[2] + re[3]), (im[0] + im[1]) + (im[2] + im[3])};
    }
    __syncthreads();
    for (int i = threadIdx.x; i < M; i += blockDim.x) {
        cx<double> t = pl[i];
        for (int g = 1; g < G; ++g) t = t + pl[g * M + i];
        pl[i] = t;
        if (P) P[(int64_t)j * M + i] = cx<T>{(T)t.re, (T)t.im};
    }
    __syncthreads();
    for (int i = threadIdx.x; i < M; i += blockDim.x) {
        const int lo = blo[i], n = bn[i];
        const double *d = dmat + bdoff[i] + (int64_t)(i - lo) * n;
        double re = 0.0, im = 0.0;
        for (int t = 0; t < n; ++t) {
            re += d[t] * pl[lo + t].re;
            im += d[t] * pl[lo + t].im;
        }
        if (occ) {
            re *= occ[j];
            im *= -occ[j];
        }
        Q[(int64_t)j * M + i] = cx<T>{(T)re, (T)im};
    }
}

// ----------------------------------------------------------------- NN ------
// C[j][g] = alpha * sum_i A[j][i] B[i][g] + beta * C[j][g]
// TS is the type A and B are stored in; they are rounded to T while staged.
// One launch covers up to kMaxBatch products of one M and K (the k-points of a call, whose G =
// npw differ): grid y counts their column tiles one after the other.
// tri: A is lower triangular (zeros stored above its diagonal), so a row tile stops at its own
// last column (a 512 x 512 inverse factor on 512 bands of 115k plane waves: 2.2 ms, whole 3.0).
template <int NB> struct NnBatch {
    int n, y0[NB];                    // y0: first column tiles in grid y
    struct {
        int G;
        int64_t ldb, ldc, a, b, c;    // rows, element offsets
    } p[NB];
};
template <typename T, typename TC, typename TS, int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kGemmWaves))) void k_gemm_nn(int M, int Kall, NnBatch<NB> bt, const cx<TS> *__restrict__ A, int64_t lda,
                                                 const cx<TS> *__restrict__ B, cx<TC> *__restrict__ C, double alpha, double beta, int tri) {
    __shared__ cx<T> As[TM][KP];
    __shared__ cx<T> Bs[KT][TN + 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int bx, by, bz;
    xcd_block(bx, by, bz);   // the row tiles of one column block share an L2
    int pb = 0;
    if constexpr (NB > 1)
        while (pb + 1 < bt.n && by >= bt.y0[pb + 1]) ++pb;
    const auto &pr = bt.p[pb];
    const int j0 = bx * TM, g0 = (by - bt.y0[pb]) * TN, G = pr.G;
    const int K = tri ? min(Kall, j0 + TM) : Kall;
    const int64_t ldb = pr.ldb, ldc = pr.ldc;
    A += pr.a;
    B += pr.b;
    C += pr.c;
    using AV = typename Acc<T>::V;
    AV c1[2][2], c2[2][2], c3[2][2];   // sums of ar br, ai bi, (ar + ai)(br + bi)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) c1[a][b] = c2[a][b] = c3[a][b] = Acc<T>::zero();
    const int wj = (w & 1) * 32, wg = (w >> 1) * 32;
    const int ar = tid >> 2, ak = (tid & 3) * 4;       // A loader: row j, 4 consecutive i
    const int bk = tid >> 4, bg = (tid & 15) * 4;      // B loader: row i, 4 consecutive g
    cx<T> ra[4], rb[4];
    // Whole stages of whole column tiles load with no per-load branch: rows past M read the last one
    // (their outputs are never stored), and an address is a uniform base plus a 32-bit byte offset
    // (lda, ldb below 2^22, 2^24): 168 registers, three waves per SIMD, where 64-bit addresses took
    // 178 and two. 120^3 x 4,096 bands: H psi 138.9 -> 136.5 ms against a branch for each load.
    const bool whole = g0 + TN <= G;
    const unsigned ao = (unsigned)(min(ar, M - 1 - j0) * (int)lda + ak) * (unsigned)sizeof(cx<TS>);
    const unsigned bo = ((unsigned)bk * (unsigned)ldb + bg) * (unsigned)sizeof(cx<TS>);
    auto load = [&](int k0) {
        const char *pa = reinterpret_cast<const char *>(A + (int64_t)j0 * lda + k0);
        const char *pb = reinterpret_cast<const char *>(B + (int64_t)k0 * ldb + g0);
        if (whole && k0 + KT <= K) {
#pragma unroll
            for (int q = 0; q < 4; ++q) ra[q] = cvt<T>(reinterpret_cast<const cx<TS> *>(pa + ao)[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) rb[q] = cvt<T>(reinterpret_cast<const cx<TS> *>(pb + bo)[q]);
        } else {
            const int nk = K - k0 - ak, ng = k0 + bk < K ? G - g0 - bg : 0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                ra[q] = q < nk ? cvt<T>(reinterpret_cast<const cx<TS> *>(pa + ao)[q]) : cx<T>{T(0), T(0)};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                rb[q] = q < ng ? cvt<T>(reinterpret_cast<const cx<TS> *>(pb + bo)[q]) : cx<T>{T(0), T(0)};
        }
    };
    load(0);
    for (int k0 = 0; k0 < K; k0 += KT) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            As[ar][ak + q] = ra[q];
            Bs[bk][bg + q] = rb[q];
        }
        __syncthreads();
        if (k0 + KT < K) load(k0 + KT);   // next stage in flight while this one multiplies
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int kk = 4 * q + (lane >> 4);
            cx<T> a[2], b[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) a[r] = As[wj + 16 * r + (lane & 15)][kk];
#pragma unroll
            for (int c = 0; c < 2; ++c) b[c] = Bs[kk][wg + 16 * c + (lane & 15)];
            T as[2], bs[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) as[r] = a[r].re + a[r].im;
#pragma unroll
            for (int c = 0; c < 2; ++c) bs[c] = b[c].re + b[c].im;
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    // a b with three real products:
                    //   re = ar br - ai bi,  im = (ar + ai)(br + bi) - ar br - ai bi
                    c1[r][c] = Acc<T>::mma(a[r].re, b[c].re, c1[r][c]);
                    c2[r][c] = Acc<T>::mma(a[r].im, b[c].im, c2[r][c]);
                    c3[r][c] = Acc<T>::mma(as[r], bs[c], c3[r][c]);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int gg = g0 + wg + 16 * c + (lane & 15);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int gj = j0 + wj + 16 * r + Acc<T>::row(lane, e);
                if (gj < M && gg < G) {
                    cx<TC> *p = C + (int64_t)gj * ldc + gg;
                    const double p1 = c1[r][c][e], p2 = c2[r][c][e], p3 = c3[r][c][e];
                    double re = alpha * (p1 - p2), im = alpha * (p3 - p1 - p2);
                    if (beta != 0.0) {
                        const cx<TC> o = *p;
                        re += beta * (double)o.re;
                        im += beta * (double)o.im;
                    }
                    *p = cx<TC>{(TC)re, (TC)im};
                }
            }
        }
}

// --------------------------------------------------------------- force -----
// X[i][g] = sum_n W[n][i] psi[n][g] (the NN product with a transposed A), contracted in the
// epilogue: part[tile][i][al] = sum over the tile's g of kg[g][al] Im(beta[i][g] conj(X[i][g])).
// X is never stored: the product and one read of beta, where projecting (k+G)_al psi as well
// took four projections' worth of products and a stacked copy of beta.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kGemmWaves))) void k_force_contract(
    int M, int G, int nb, const z64 *__restrict__ W, const z64 *__restrict__ psi, const z64 *__restrict__ beta,
    const double *__restrict__ kg, double *__restrict__ part) {
    using A = Acc<double>;
    __shared__ z64 As[TM][KP];
    __shared__ z64 Bs[KT][TN + 1];
    __shared__ double red[2][TM][3];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int bx, by, bz;
    xcd_block(bx, by, bz);   // the row tiles of one column block share an L2
    const int i0 = bx * TM, g0 = by * TN;
    d4 c1[2][2], c2[2][2], c3[2][2];   // sums of ar br, ai bi, (ar + ai)(br + bi)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) c1[a][b] = c2[a][b] = c3[a][b] = A::zero();
    const int wi = (w & 1) * 32, wg = (w >> 1) * 32;
    const int lk = tid >> 4, lc = (tid & 15) * 4;   // loader of both: row n, 4 consecutive i or g
    z64 ra[4], rb[4];
    auto load = [&](int k0) {
        const int n = k0 + lk;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            ra[q] = n < nb && i0 + lc + q < M ? W[(int64_t)n * M + i0 + lc + q] : z64{0.0, 0.0};
            rb[q] = n < nb && g0 + lc + q < G ? psi[(int64_t)n * G + g0 + lc + q] : z64{0.0, 0.0};
        }
    };
    load(0);
    for (int k0 = 0; k0 < nb; k0 += KT) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            As[lc + q][lk] = ra[q];
            Bs[lk][lc + q] = rb[q];
        }
        __syncthreads();
        if (k0 + KT < nb) load(k0 + KT);   // next stage in flight while this one multiplies
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int kk = 4 * q + (lane >> 4);
            z64 a[2], b[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) a[r] = As[wi + 16 * r + (lane & 15)][kk];
#pragma unroll
            for (int c = 0; c < 2; ++c) b[c] = Bs[kk][wg + 16 * c + (lane & 15)];
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    c1[r][c] = A::mma(a[r].re, b[c].re, c1[r][c]);
                    c2[r][c] = A::mma(a[r].im, b[c].im, c2[r][c]);
                    c3[r][c] = A::mma(a[r].re + a[r].im, b[c].re + b[c].im, c3[r][c]);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int li = wi + 16 * r + A::row(lane, e), gi = i0 + li;
            double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int gg = g0 + wg + 16 * c + (lane & 15);
                if (gi < M && gg < G) {
                    const z64 b = beta[(int64_t)gi * G + gg];
                    const double p1 = c1[r][c][e], p2 = c2[r][c][e], p3 = c3[r][c][e];
                    const double t = b.im * (p1 - p2) - b.re * (p3 - p1 - p2);
#pragma unroll
                    for (int al = 0; al < 3; ++al) s[al] += kg[3 * (int64_t)gg + al] * t;
                }
            }
#pragma unroll
            for (int al = 0; al < 3; ++al) {
#pragma unroll
                for (int o = 8; o > 0; o >>= 1) s[al] += __shfl_xor(s[al], o, 16);
                if ((lane & 15) == 0) red[w >> 1][li][al] = s[al];
            }
        }
    __syncthreads();
    for (int t = tid; t < TM * 3; t += 256) {
        const int li = t / 3, al = t - 3 * li;
        if (i0 + li < M) part[((int64_t)by * M + i0 + li) * 3 + al] = red[0][li][al] + red[1][li][al];
    }
}

int force_contract_tiles(int G) { return ceil_div(G, TN); }

int force_contract(int M, int G, int nb, const void *W, const void *psi, const void *beta, const double *kg,
                   double *part, hipStream_t st) {
    KernelTimer kt("force_contract", st);
    hipLaunchKernelGGL(k_force_contract, dim3(ceil_div(M, TM), ceil_div(G, TN)), dim3(256), 0, st, M, G, nb,
                       static_cast<const z64 *>(W), static_cast<const z64 *>(psi), static_cast<const z64 *>(beta), kg,
                       part);
    return check_launch("force_contract");
}

// grad_d[blk(i)][i - lo][t] (+)= sum_n Re(Q[n][i] conj(P[n][lo + t])): 64 projectors i by
// kGradDGroups groups of bands (n = g mod kGradDGroups), group sums added in order. Bound by the
// latency of its loads: 512 projectors x 256 bands took 207 us with one thread per projector in
// one chain over the bands, now 25.
constexpr int kGradDGroups = 16;
template <typename T>
__global__ __launch_bounds__(64 * kGradDGroups) void k_grad_d(int nb, int M, const cx<T> *__restrict__ P,
                                                              const cx<T> *__restrict__ Q, const int *__restrict__ blo,
                                                              const int *__restrict__ bn, const int *__restrict__ bdoff,
                                                              double *__restrict__ gd, int first) {
    __shared__ double red[kGradDGroups][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6, i = blockIdx.x * 64 + lane, ic = min(i, M - 1);
    const int lo = blo[ic], n = bn[ic];
    double *out = gd + bdoff[ic] + (int64_t)(ic - lo) * n;
    for (int t = 0; __syncthreads_or(t < n); ++t) {
        const int tc = lo + min(t, n - 1);
        double s = 0.0;
#pragma unroll 4
        for (int b = g; b < nb; b += kGradDGroups) {
            const cx<T> q = Q[(int64_t)b * M + ic], p = P[(int64_t)b * M + tc];
            s += (double)q.re * (double)p.re + (double)q.im * (double)p.im;
        }
        red[g][lane] = s;
        __syncthreads();
        if (g == 0 && i < M && t < n) {
            double r = red[0][lane];
            for (int u = 1; u < kGradDGroups; ++u) r += red[u][lane];
            out[t] = first ? r : out[t] + r;
        }
    }
}

// ------------------------------------------------------------ launchers ----
// Default K chunk of `batch` products in one launch: at least 512 work-groups, chunks of at
// most 1024 (a K chunk of A and B read by every tile of the chunk stays in the caches, where
// one long K range per tile streams A once per column of tiles from HBM: at 2304 x 1024 x
// 161,235 the projection read 13.7x its operands with one split, measured with FETCH_SIZE),
// but no more splits than keep the partial sums under kPartCap bytes. A work-group spends about
// 2 us on a stage of 16 k when few others run, so small products are split down to chunks of
// 32: 32 x 16 x 1503 took 33.5 us in chunks of 256 (6 work-groups of 16 stages), 13.0 in chunks
// of 64 and 9.3 in chunks of 32. 768 work-groups (three a CU) gained nothing at 256 x 128 x
// 23,847: 87.4 us and 12.8 us of reduction against 84.9 and 11.0.
// `wide` is the rule of the reduced-precision products whose sums feed complex128 results
// (chunks of at least 256): the chunk groups their FP32 sums, so it stays.
constexpr size_t kPartCap = size_t(1) << 30;
static int splits_wanted(int M, int N, int batch) {
    const int tiles = ceil_div(M, TM) * ceil_div(N, TN) * batch;
    return std::max(1, 512 / std::max(1, tiles));
}
static int splits_for(int M, int N, int K, int chunk_hint, int batch, bool wide, int *chunk) {
    int c = chunk_hint > 0 ? chunk_hint : 0;
    if (c <= 0) {
        c = std::min(1024, std::max(wide ? 256 : 32, ceil_div(K, splits_wanted(M, N, batch))));
        const int64_t max_splits = std::max<int64_t>(1, (int64_t)(kPartCap / ((size_t)M * N * 16)));
        c = std::max<int64_t>(c, ceil_div64(K, max_splits));
    }
    c = ceil_div(c, KT) * KT;
    *chunk = c;
    return std::max(1, ceil_div(K, c));
}

// Upper bound over every M' <= M, N' <= N, K' <= K and either rule. A product has either chunks
// of 1024 (or the capped or hinted length), or at most 512 / tiles splits of at least 32 k, and
// tiles * 64 * 64 >= M' N'.
size_t gemm_cn_part_bytes(int M, int N, int K, int elem_bytes, int chunk_hint) {
    const size_t mn = (size_t)M * N;
    if (chunk_hint > 0) return (size_t)ceil_div(K, ceil_div(chunk_hint, KT) * KT) * mn * elem_bytes;
    const size_t few = std::max(mn, std::min((size_t)ceil_div(K, 1024) * mn, kPartCap / 16));
    const size_t many = std::min<size_t>((size_t)512 * TM * TN, (size_t)ceil_div(K, 32) * mn);
    return std::max(few, many) * elem_bytes;
}

// A launch takes at most 65,536 work-groups in y and in z (hipDeviceAttributeMaxGridDimY, Z), and the
// products of a launch add up there: the splits of the projection in z, the column tiles in y.
constexpr int kMaxGridYZ = 65535;
int gemm_batch_limit(int M, int N, int K, int elem_bytes, int chunk_hint) {
    const size_t part = gemm_cn_part_bytes(M, N, K, elem_bytes, chunk_hint);
    const int splits = chunk_hint > 0 ? ceil_div(K, ceil_div(chunk_hint, KT) * KT) : std::max(512, ceil_div(K, 1024));
    return (int)std::max<size_t>(1, std::min<size_t>({kMaxBatch, kPartCap / part, (size_t)(kMaxGridYZ / splits)}));
}
int gemm_nn_batch_limit(int G) { return std::max(1, std::min(kMaxBatch, kMaxGridYZ / ceil_div(G, TN))); }

template <typename T, typename TS, int NB>
static int cn_part_nb(int M, int N, const CnProduct *pr, int np, const void *A, const void *B, void *part,
                      int chunk_hint, bool wide, RedBatch *rb, hipStream_t st, int herm) {
    CnBatch<NB> bt;
    bt.n = np;
    rb->z0[0] = 0;
    for (int i = 0; i < np; ++i) {
        auto &p = bt.p[i];
        p = {pr[i].K, 0, pr[i].lda, pr[i].ldb, pr[i].a, pr[i].b};
        bt.z0[i] = rb->z0[i];
        rb->z0[i + 1] = rb->z0[i] + splits_for(M, N, p.K, chunk_hint, np, wide, &p.kchunk);
    }
    dim3 grid(ceil_div(M, TM), ceil_div(N, TN), rb->z0[np]);
    // group of row tiles: about one XCD's resident work-groups (32 CUs x 3) per group;
    // a chunk of at most two such groups keeps the row tiles fastest (one group): at
    // 864 x 512 per k-point that order measured 1-2% faster than groups of 12 rows
    const int tiles = (int)(grid.x * grid.y);
    const int gm = tiles <= 192 ? (int)grid.x : std::max(1, std::min((int)grid.x, 96 / (int)grid.y));
    KernelTimer kt("gemm_cn", st);
    hipLaunchKernelGGL((k_gemm_cn_part<T, TS, NB>), grid, dim3(256), 0, st, M, N, bt, static_cast<const cx<TS> *>(A),
                       static_cast<const cx<TS> *>(B), static_cast<cx<T> *>(part), gm, herm);
    return check_launch("gemm_cn");
}

template <typename T, typename TS = T>
static int cn_part(int M, int N, const CnProduct *pr, int np, const void *A, const void *B, void *part,
                   int chunk_hint, bool wide, RedBatch *rb, hipStream_t st, int herm = 0) {
    return np > 1 ? cn_part_nb<T, TS, kMaxBatch>(M, N, pr, np, A, B, part, chunk_hint, wide, rb, st, herm)
                  : cn_part_nb<T, TS, 1>(M, N, pr, np, A, B, part, chunk_hint, wide, rb, st, herm);
}

// T: arithmetic and partial sums; TS: storage of A, B and C.
template <typename T, typename TS = T>
static int gemm_cn_t(int M, int N, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
                     int64_t ldc, double alpha, double beta, void *part, int chunk_hint, hipStream_t st, int herm = 0) {
    if (M <= 0 || N <= 0) return ABACUS_PW_OK;
    RedBatch rb;
    const CnProduct pr{K, lda, ldb, 0, 0};
    APW_TRY((cn_part<T, TS>(M, N, &pr, 1, A, B, part, chunk_hint, sizeof(T) < sizeof(TS), &rb, st, herm)));
    return launch_reduce<T, TS>(M, N, rb.z0[1], part, C, ldc, alpha, beta, herm, st);
}

int reduce_parts_f32_to_f64(int M, int N, int nsplit, const void *part, void *C, int64_t ldc, double alpha,
                            double beta, hipStream_t st) {
    if (M <= 0 || N <= 0) return ABACUS_PW_OK;
    return launch_reduce<float, double>(M, N, nsplit, part, C, ldc, alpha, beta, 0, st);
}

int gemm_cn_f32_of_f64(int M, int N, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
                       int64_t ldc, double alpha, double beta, void *part, int chunk_hint, hipStream_t st) {
    return gemm_cn_t<float, double>(M, N, K, A, lda, B, ldb, C, ldc, alpha, beta, part, chunk_hint, st);
}

int gemm_cn(int prec, int M, int N, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
            int64_t ldc, double alpha, double beta, void *part, int chunk_hint, hipStream_t st) {
    return prec == 0 ? gemm_cn_t<double>(M, N, K, A, lda, B, ldb, C, ldc, alpha, beta, part, chunk_hint, st)
                     : gemm_cn_t<float>(M, N, K, A, lda, B, ldb, C, ldc, alpha, beta, part, chunk_hint, st);
}

int gemm_cn_herm(int M, int K, const void *A, int64_t lda, void *C, int64_t ldc, void *part, hipStream_t st) {
    return gemm_cn_t<double>(M, M, K, A, lda, A, lda, C, ldc, 1.0, 0.0, part, 0, st, 1);
}

// LDS of k_reduce_dapply: the group sums of a band. M above 4096 exceeds the limit.
constexpr size_t kDapplyLds = 64 * 1024;
static size_t dapply_lds(int M) { return (size_t)reduce_groups(M) * M * sizeof(z64); }

template <typename T>
static int proj_dapply_t(int M, int N, const CnProduct *pr, int np, const void *Bm, const void *psi,
                         const double *dmat, const int *blo, const int *bn, const int *bdoff, void *P, void *Q,
                         void *part, int chunk_hint, bool wide, hipStream_t st, const double *occ = nullptr) {
    if (M <= 0 || N <= 0) return ABACUS_PW_OK;
    RedBatch rb;
    APW_TRY(cn_part<T>(M, N, pr, np, Bm, psi, part, chunk_hint, wide, &rb, st));
    const size_t lds = dapply_lds(M);
    if (lds > kDapplyLds) return set_error(ABACUS_PW_EBAD_SHAPE, "too many projectors for the D-apply stage");
    KernelTimer kt("reduce_dapply", st);
    hipLaunchKernelGGL(k_reduce_dapply<T>, dim3(N, np), dim3(kRedThreads), lds, st, M, rb, static_cast<const cx<T> *>(part), N,
                       dmat, blo, bn, bdoff, static_cast<cx<T> *>(P), static_cast<cx<T> *>(Q), occ);
    return check_launch("reduce_dapply");
}

bool proj_weights_fit(int M) { return dapply_lds(M) <= kDapplyLds; }

int proj_weights(int M, int N, int K, const void *Bm, const void *psi, const double *occ, const double *dmat,
                 const int *blo, const int *bn, const int *bdoff, void *W, void *part, int chunk_hint, hipStream_t st) {
    const CnProduct pr{K, K, K, 0, 0};
    return proj_dapply_t<double>(M, N, &pr, 1, Bm, psi, dmat, blo, bn, bdoff, nullptr, W, part, chunk_hint, false, st,
                                 occ);
}

int proj_dapply(int prec, int M, int N, const CnProduct *pr, int np, const void *Bm, const void *psi,
                const double *dmat, const int *blo, const int *bn, const int *bdoff, void *P, void *Q, void *part,
                int chunk_hint, bool wide, hipStream_t st) {
    return prec == 0 ? proj_dapply_t<double>(M, N, pr, np, Bm, psi, dmat, blo, bn, bdoff, P, Q, part, chunk_hint, wide,
                                             st)
                     : proj_dapply_t<float>(M, N, pr, np, Bm, psi, dmat, blo, bn, bdoff, P, Q, part, chunk_hint, wide,
                                            st);
}

template <typename T, typename TC, typename TS, int NB>
static int gemm_nn_nb(int M, int K, const NnProduct *pr, int np, const void *A, int64_t lda, const void *B, void *C,
                      double alpha, double beta, hipStream_t st, int tri) {
    if (M <= 0) return ABACUS_PW_OK;
    NnBatch<NB> bt;
    bt.n = np;
    int tiles = 0;
    for (int i = 0; i < np; ++i) {
        bt.y0[i] = tiles;
        bt.p[i] = {pr[i].G, pr[i].ldb, pr[i].ldc, pr[i].a, pr[i].b, pr[i].c};
        tiles += ceil_div(pr[i].G, TN);
    }
    if (tiles == 0) return ABACUS_PW_OK;
    dim3 grid(ceil_div(M, TM), tiles);
    KernelTimer kt("gemm_nn", st);
    hipLaunchKernelGGL((k_gemm_nn<T, TC, TS, NB>), grid, dim3(256), 0, st, M, K, bt, static_cast<const cx<TS> *>(A), lda,
                       static_cast<const cx<TS> *>(B), static_cast<cx<TC> *>(C), alpha, beta, tri);
    return check_launch("gemm_nn");
}

template <typename T, typename TC, typename TS = T>
static int gemm_nn_batch_t(int M, int K, const NnProduct *pr, int np, const void *A, int64_t lda, const void *B,
                           void *C, double alpha, double beta, hipStream_t st, int tri = 0) {
    return np > 1 ? gemm_nn_nb<T, TC, TS, kMaxBatch>(M, K, pr, np, A, lda, B, C, alpha, beta, st, tri)
                  : gemm_nn_nb<T, TC, TS, 1>(M, K, pr, np, A, lda, B, C, alpha, beta, st, tri);
}

int gemm_nn_batch(int prec, int M, int K, const NnProduct *pr, int np, const void *A, int64_t lda, const void *B,
                  void *C, double alpha, double beta, hipStream_t st) {
    return prec == 0 ? gemm_nn_batch_t<double, double>(M, K, pr, np, A, lda, B, C, alpha, beta, st)
                     : gemm_nn_batch_t<float, float>(M, K, pr, np, A, lda, B, C, alpha, beta, st);
}

template <typename T, typename TC, typename TS = T>
static int gemm_nn_t(int M, int G, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
                     int64_t ldc, double alpha, double beta, hipStream_t st) {
    if (M <= 0 || G <= 0) return ABACUS_PW_OK;
    const NnProduct pr{G, ldb, ldc, 0, 0, 0};
    return gemm_nn_batch_t<T, TC, TS>(M, K, &pr, 1, A, lda, B, C, alpha, beta, st);
}

int gemm_nn_f32_of_f64(int M, int G, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
                       int64_t ldc, double alpha, double beta, hipStream_t st) {
    return gemm_nn_t<float, double, double>(M, G, K, A, lda, B, ldb, C, ldc, alpha, beta, st);
}

int gemm_nn(int prec, int M, int G, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
            int64_t ldc, double alpha, double beta, hipStream_t st) {
    return prec == 0 ? gemm_nn_t<double, double>(M, G, K, A, lda, B, ldb, C, ldc, alpha, beta, st)
                     : gemm_nn_t<float, float>(M, G, K, A, lda, B, ldb, C, ldc, alpha, beta, st);
}

int gemm_nn_tri(int M, int G, const void *A, int64_t lda, const void *B, int64_t ldb, void *C, int64_t ldc,
                hipStream_t st) {
    if (M <= 0 || G <= 0) return ABACUS_PW_OK;
    const NnProduct pr{G, ldb, ldc, 0, 0, 0};
    return gemm_nn_batch_t<double, double>(M, M, &pr, 1, A, lda, B, C, 1.0, 0.0, st, 1);
}

int gemm_nn_f32_into_f64(int M, int K, const NnProduct *pr, int np, const void *A, int64_t lda, const void *B, void *C,
                         double alpha, double beta, hipStream_t st) {
    return gemm_nn_batch_t<float, double>(M, K, pr, np, A, lda, B, C, alpha, beta, st);
}

int reduce_dapply_f32(int M, int N, int nsplit, const void *part, const double *dmat, const int *blo, const int *bn,
                      const int *bdoff, void *Q, hipStream_t st) {
    const size_t lds = dapply_lds(M);
    if (lds > kDapplyLds) return set_error(ABACUS_PW_EBAD_SHAPE, "too many projectors for the D-apply stage");
    KernelTimer kt("reduce_dapply", st);
    RedBatch rb;
    rb.z0[0] = 0;
    rb.z0[1] = nsplit;
    hipLaunchKernelGGL(k_reduce_dapply<float>, dim3(N), dim3(kRedThreads), lds, st, M, rb, static_cast<const c32 *>(part),
                       N, dmat, blo, bn, bdoff, static_cast<c32 *>(nullptr), static_cast<c32 *>(Q),
                       static_cast<const double *>(nullptr));
    return check_launch("reduce_dapply");
}

int grad_d_accumulate(int prec, int nb, int M, const void *P, const void *Q, const int *blo, const int *bn,
                      const int *bdoff, double *gd, int first, hipStream_t st) {
    KernelTimer kt("grad_d", st);
    if (prec == 0)
        hipLaunchKernelGGL(k_grad_d<double>, dim3(ceil_div(M, 64)), dim3(64 * kGradDGroups), 0, st, nb, M,
                           static_cast<const z64 *>(P), static_cast<const z64 *>(Q), blo, bn, bdoff, gd, first);
    else
        hipLaunchKernelGGL(k_grad_d<float>, dim3(ceil_div(M, 64)), dim3(64 * kGradDGroups), 0, st, nb, M,
                           static_cast<const c32 *>(P), static_cast<const c32 *>(Q), blo, bn, bdoff, gd, first);
    return check_launch("grad_d");
}

}  // namespace apw
