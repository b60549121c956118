// Complex GEMMs on MFMA; see gemm.hip. prec: 0 complex128, 1 complex64.
#pragma once

#include "common.hpp"

namespace apw {

// Bytes of split-K partial sums gemm_cn / proj_dapply need.
size_t gemm_cn_part_bytes(int M, int N, int K, int elem_bytes, int chunk_hint);

// C[j*ldc + i] = alpha * sum_k conj(A[i*lda + k]) B[j*ldb + k] + beta * C[...],  i < M, j < N.
int gemm_cn(int prec, int M, int N, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
            int64_t ldc, double alpha, double beta, void *part, int chunk_hint, hipStream_t st);

// C = A^H A (M x M, FP64): half of gemm_cn's products, the other triangle as conjugates. part:
// gemm_cn_part_bytes(M, M, K, 16, 0).
int gemm_cn_herm(int M, int K, const void *A, int64_t lda, void *C, int64_t ldc, void *part, hipStream_t st);

// Products of one launch, one per k-point of a call: their inner (or outer) length and rows,
// and where their operands start (elements from the launch's base pointers).
constexpr int kGemmMaxBatch = 8;
struct CnProduct {
    int K;
    int64_t lda, ldb, a, b;
};
struct NnProduct {
    int G;
    int64_t ldb, ldc, a, b, c;
};
// Products of that shape (K at most) one launch may take: kGemmMaxBatch, partial sums of at most
// 1 GiB (gemm_cn_part_bytes each), and the splits that a grid holds.
int gemm_batch_limit(int M, int N, int K, int elem_bytes, int chunk_hint);
// Products with G columns at most that one gemm_nn_batch may take.
int gemm_nn_batch_limit(int G);

// For every product p: P[j][i] = <beta_i | psi_j> (M = nproj, N = bands, K = npw);
// Q[j][i] = sum_t D_blk(i) P[j][.], P and Q [np][N][M]. P may be NULL. D-block tables as in the
// plan. wide: the K chunks of the mixed modes.
int proj_dapply(int prec, int M, int N, const CnProduct *pr, int np, const void *Bm, const void *psi,
                const double *dmat, const int *blo, const int *bn, const int *bdoff, void *P, void *Q, void *part,
                int chunk_hint, bool wide, hipStream_t st);

// W[j][i] = occ[j] conj(Q[j][i]) of one FP64 product (the band weights of the nonlocal force), for M that
// proj_weights_fit allows.
bool proj_weights_fit(int M);
int proj_weights(int M, int N, int K, const void *Bm, const void *psi, const double *occ, const double *dmat,
                 const int *blo, const int *bn, const int *bdoff, void *W, void *part, int chunk_hint, hipStream_t st);

// gemm_cn on complex128 A, B, C with FP32 products: the operands are rounded to
// complex64 as they are staged, partial sums are FP32, the split-K sum and C are FP64
// (the subspace projection of the reduced-precision Davidson phase).
int gemm_cn_f32_of_f64(int M, int N, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
                       int64_t ldc, double alpha, double beta, void *part, int chunk_hint, hipStream_t st);

// C[j*ldc + g] = alpha * sum_i A[j*lda + i] B[i*ldb + g] + beta * C[...],  j < M, g < G, for np
// products: A [M][lda], B rows of ldb, C rows of ldc, from their offsets.
int gemm_nn_batch(int prec, int M, int K, const NnProduct *pr, int np, const void *A, int64_t lda, const void *B,
                  void *C, double alpha, double beta, hipStream_t st);

int gemm_nn(int prec, int M, int G, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
            int64_t ldc, double alpha, double beta, hipStream_t st);

// C = A B with A [M][lda] lower triangular (zeros stored above the diagonal), FP64.
int gemm_nn_tri(int M, int G, const void *A, int64_t lda, const void *B, int64_t ldb, void *C, int64_t ldc,
                hipStream_t st);

// As gemm_nn on complex128 A, B and C with FP32 products: the operands are rounded to
// complex64 as they are staged, C accumulates in FP64 (basis updates of the
// reduced-precision Davidson phase).
int gemm_nn_f32_of_f64(int M, int G, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
                       int64_t ldc, double alpha, double beta, hipStream_t st);

// As gemm_nn_batch with complex64 A and B accumulated into a complex128 C.
int gemm_nn_f32_into_f64(int M, int K, const NnProduct *pr, int np, const void *A, int64_t lda, const void *B, void *C,
                         double alpha, double beta, hipStream_t st);

// part[tile][i][al] = sum over the tile's g of kg[g][al] Im(beta[i][g] conj(X[i][g])) with
// X[i][g] = sum_n W[n][i] psi[n][g]: W [nb][M], psi [nb][G], beta [M][G], kg [G][3]; tiles of
// g = force_contract_tiles(G).
int force_contract_tiles(int G);
int force_contract(int M, int G, int nb, const void *W, const void *psi, const void *beta, const double *kg,
                   double *part, hipStream_t st);

// grad_d entry (i, lo+t) of each atom block (+)= sum_n Re(Q[n][i] conj(P[n][lo+t])); P, Q are [nb][M].
int grad_d_accumulate(int prec, int nb, int M, const void *P, const void *Q, const int *blo, const int *bn,
                      const int *bdoff, double *gd, int first, hipStream_t st);

// Split-K sum of complex64 partials [nsplit][N][M] followed by the D blocks: Q[j][i] (complex64).
int reduce_dapply_f32(int M, int N, int nsplit, const void *part, const double *dmat, const int *blo, const int *bn,
                      const int *bdoff, void *Q, hipStream_t st);

// ---- BF16 operands, FP32 accumulation (gemm_bf16.hip) ----
// Leading dimension of packed bf16 rows of K values: K rounded up to a multiple of 32.
inline int bf16_ld(int K) { return (K + 31) / 32 * 32; }
// out[r][c] = in[r][c] (complex128 when in_is_f64, else complex64) rounded to a packed bf16 pair
// (re low, im high) for c < K, 0 for K <= c < ldo.
int pack_bf16_rows(int rows, int K, const void *in, int in_is_f64, int64_t ldi, void *out, int64_t ldo,
                   hipStream_t st);
size_t gemm_cn_bf16_part_bytes(int M, int N, int K, int chunk_hint);
// Q[j][i] = sum_t D_blk(i) P[j][.], P[j][i] = <beta_i|psi_j> with bf16 operands: Bpk packed bf16 beta
// [M][ldb], psi_pk packed bf16 psi [N][ldp], both with zero-padded rows (ldb, ldp = bf16_ld(K)).
int proj_dapply_bf16(int M, int N, int K, const void *Bpk, int64_t ldb, const void *psi_pk, int64_t ldp,
                     const double *dmat, const int *blo, const int *bn, const int *bdoff, void *Q, void *part,
                     int chunk_hint, hipStream_t st);
// C = alpha sum_s part[s] + beta C: complex64 split-K partials [nsplit][N][M] into complex128 C (ldc).
int reduce_parts_f32_to_f64(int M, int N, int nsplit, const void *part, void *C, int64_t ldc, double alpha,
                            double beta, hipStream_t st);
// C = A^H B (M x N, ldc) for complex128 rows A [M][lda], B [N][ldb] of length K, computed with both
// operands rounded to bf16 and FP32 accumulation; scratch of gemm_cn_bf16_of_f64_bytes(M, N, K) bytes.
size_t gemm_cn_bf16_of_f64_bytes(int M, int N, int K);
int gemm_cn_bf16_of_f64(int M, int N, int K, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
                        int64_t ldc, void *scratch, hipStream_t st);
// out[i][g] and outT[g][i] = in[i][g] (complex128 [rows][ldi], g < cols) as packed bf16, zero for
// cols <= g < ldo and rows <= i < ldt; ldo = bf16_ld(cols), ldt = bf16_ld(rows).
int pack_bf16_both(int rows, int cols, const void *in, int64_t ldi, void *out, int64_t ldo, void *outT, int64_t ldt,
                   hipStream_t st);
// C[j][g] += sum_i A[j][i] B[i][g] for j < N, g < G, i < K: Apk packed bf16 A [N][lda], BTpk packed bf16
// transposed B [G][ldbt], lda and ldbt = bf16_ld(K) with zero padding; C complex128 [N][ldc].
int gemm_nn_bf16_into_f64(int N, int G, int K, const void *Apk, int64_t lda, const void *BTpk, int64_t ldbt, void *C,
                          int64_t ldc, hipStream_t st);

}  // namespace apw
