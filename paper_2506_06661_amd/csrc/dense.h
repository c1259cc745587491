// Dense helpers (dense.hip, eigen.hip): matrix products and the symmetric
// eigensolver.
#pragma once

#include "internal.h"

namespace dfjk {

constexpr int kMaxEighN = 4096;

// Largest edge of a result that 16 x 16 tiles take (gemm_tile.h).  Square products, us:
// 256: 5 with them, 41 with the wide tiles (A B^T: 6, 11 with 64 x 64 tiles);
// 448: 18, 80 (6, 20); 640: 41, 98 (15, 24).  Each operand is read from L2 once
// per 16 rows or columns, not 64 or 128, so their lead shrinks with size; not
// measured beyond 640.
constexpr int64_t kSmallN = 640;

// C = alpha op(A) op(B) + beta C (row-major; op = transpose when ta / tb).
int dgemm(hipStream_t st, bool ta, bool tb, int64_t M, int64_t N, int64_t K, double alpha,
          const double* A, int64_t lda, const double* B, int64_t ldb, double beta, double* C,
          int64_t ldc);

// What a product of the network does with its sums before they are stored.
enum { EPI_NONE = 0, EPI_BIAS = 1, EPI_DSILU = 2 };  // C = s, s + bias[n], s * silu'(Z[m][n])
struct GemmEpi {
    const float* bias = nullptr;  // EPI_BIAS: N values
    const float* Z = nullptr;     // EPI_DSILU: M x N, rows ldc apart
};

// C = op(A) op(B) in FP32 (row-major, contraction in 4-deep matrix-core
// steps), or, with bf16, the FP32 operands rounded once to bfloat16 and the
// products on the 16-bit matrix cores (FP32 sums).  With kslab > 0 the
// contraction is cut into slabs of kslab terms and slab s writes its own
// product to C + s * M * ldc (epi must be EPI_NONE then).
int net_gemm(hipStream_t st, bool bf16, bool ta, bool tb, int64_t M, int64_t N, int64_t K, const float* A,
             int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc, int64_t kslab = 0,
             int epi = EPI_NONE, GemmEpi e = GemmEpi());

// Workspace of the eigensolver for n x n matrices, carved from one buffer.
constexpr int kEigLdsN = 198;       // largest n solved in LDS (eigen.hip)
constexpr int kEigMaxSweeps = 40;   // the log of rotations holds them all
struct EigWork {
    double* A;    // n x n (larger n only)
    double* work; // n + 2 (larger n only)
    double* log;  // log_elems(n): rotations to apply to the eigenvectors
    int* iwork;   // iwork_elems(n): sweeps, index of each rank (larger n only), rank of each index, ...
    double* w;    // n eigenvalues in ascending order
    __host__ __device__ static int rank_at(int n) { return n + 2; }
    __host__ __device__ static int rounds_at(int n) { return 2 * n + 2; }
    static size_t iwork_elems(int64_t n) { return 2 * (size_t)n + 3; }
    static size_t log_elems(int64_t n) {
        const int64_t h = (n + 1) / 2;
        return n <= kEigLdsN ? (size_t)(2 * kEigMaxSweeps * (2 * h - 1) * h) : 0;
    }
};

// Eigendecomposition of F = (X + X^T) / 2 by cyclic Jacobi.  V (n x n) holds a
// basis as ROWS: on entry X must be expressed in that basis (X = V F V^T; with
// v_identity V is taken as the identity and need not be set), on exit row k of
// V is an eigenvector of F.  out (n x ncol) = eigenvector columns of the ncol
// smallest eigenvalues; mode 1 scales column c by sqrt|w_c| and writes
// sign(w_c) to sign.  A non-finite entry in X: w and out are NaN, V is as on entry.
int eigh_cols(hipStream_t st, const double* X, double* V, int n, bool v_identity, const EigWork& ws, int ncol,
              int mode, double* out, double* sign);

// The form for n <= kEigLdsN (eigen.hip).
int eig_lds(hipStream_t st, const double* X, double* V, int n, bool v_identity, const EigWork& ws, int ncol,
            int mode, double* out, double* sign);

// ---- one molecule's SCF step (scf.hip): what its kernels read from the device
struct ScfRecord {  // mirrors dfjk_scf_info
    double e_tot, e_1e, e_j, e_k, err_norm, d_e;
    int iter, converged;
};
struct ScfMol {
    int n, nocc;
    const double *J, *K;
    double *D, *C;
    double *V, *F, *G, *Fx;        // eigenbasis (rows), Fock matrix, scratch, extrapolated Fock matrix
    double *Fh, *Eh;               // DIIS history
    double *gram, *coef, *part, *e_prev, *first;
    ScfRecord* rec;
    EigWork eig;
};
// A launch over molecules takes the pointers that a call brings for up to
// kMolChunk of them by value.
constexpr int kMolChunk = 64;
struct MolPtrs {
    const double* p[kMolChunk];
};

// Eigenvectors of up to kMolChunk molecules with n <= kEigLdsN in one launch
// each for rotations and vectors: of X.p[i], V then starting as the identity,
// or, without X, of each one's Fx in the basis V.
// max_n: the largest n, lds_n: the one that takes the most LDS.
int eig_lds_many(hipStream_t st, const ScfMol* mols, const MolPtrs* X, bool v_identity, int nmol, int max_n,
                 int lds_n);
size_t eig_lds_bytes(int n);

// The SCF step after J and K, and the aufbau of a given F, of up to kMolChunk
// molecules (scf.hip): mols on the device, h their handles, all at the same
// iteration.  scf_describe fills one entry; its record goes to rec, its eigensolver's
// log of rotations (EigWork::log_elems values) to log.
int scf_describe(dfjk_ctx* h, double* D, double* C, int64_t nocc, const double* J, const double* K, void* rec,
                 double* log, ScfMol* out);
int scf_tail_many(hipStream_t st, const ScfMol* mols, dfjk_ctx* const* h, const double* const* H, int nmol);
int aufbau_many(hipStream_t st, const ScfMol* mols, dfjk_ctx* const* h, const double* const* F, int nmol);

}  // namespace dfjk
