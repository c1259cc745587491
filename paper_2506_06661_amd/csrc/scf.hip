// One restricted closed-shell SCF iteration on the GPU (FP64), and the
// exchange matrix of a general symmetric density.
//
// Iteration k with density D_k (paper Sec. IV.A: a mean-field run takes a
// guess density dm0, which need not be idempotent; Sec. IV.B: DIIS is the
// default accelerator):
//   J, K from D_k (K through C when D_k = 2 C C^T, else from D_k itself or its
//   signed eigen-factors); F = H + J - K/2;
//   E_k = tr(D H) + tr(D J)/2 - tr(D K)/4 = tr(D (H + F))/2;
//   e = F D - D F = G - G^T with G = F D (F, D symmetric);
//   Pulay DIIS over the last `diis_space` (F, e): minimise |sum c_i e_i| with
//   sum c_i = 1 through the bordered Gram system, solved by Gaussian
//   elimination with partial pivoting, after dropping the oldest pairs while
//   the Gram matrix's condition number exceeds 1e12; F' = sum c_i F_i;
//   aufbau on F' (Jacobi eigensolver): C = the nocc lowest eigenvectors,
//   D_{k+1} = 2 C C^T.
// Everything stays on the device; the host reads the iteration record only
// when the caller asks for it.
//
// At the sizes an SCF is run at, the step after J and K is bound by the number of
// its dependent launches (3 to 5 us each) and by the eigensolver's chain of
// rounds, not by arithmetic.  So it is a few fused kernels, each over all
// molecules of a batch at once (grid z: molecule): Fock matrix, its history slot
// and the energies' partial sums; F D; commutator and its products with the
// history; one wavefront for energies, Gram matrix, convergence and DIIS;
// combination; products and eigensolver.  MI355X: six
// iterations at nao=128 4.5 ms (5.0 with twenty launches for one), a guess and three
// iterations of 16 molecules 6.5 ms (15.2 with every molecule's launches on one
// of eight streams).
#include "dense.h"
#include "gemm_tile.h"
#include "numerics.h"

#include <algorithm>

namespace dfjk {

namespace {

__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

__global__ void symmetrize_kernel(const double* __restrict__ X, int64_t n, double* __restrict__ Y) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * n) return;
    const int64_t r = i / n, c = i % n;
    Y[i] = 0.5 * (X[r * n + c] + X[c * n + r]);
}

struct Slots {
    int s[16];
};

// What a step does, the same for every molecule of a launch
struct ScfStep {
    int space, snew, m, iter;  // DIIS vectors: capacity, newest slot, stored; iteration
    Slots order;               // stored slots in chronological order
    double conv_tol, conv_tol_grad;
};

// Where a kernel finds molecule blockIdx.z: by value, or in a list on the device
struct One {
    ScfMol d;
    const double* H;
    __device__ const ScfMol& mol(int) const { return d; }
    __device__ const double* h(int) const { return H; }
};
struct Many {
    const ScfMol* list;
    MolPtrs H;
    __device__ const ScfMol& mol(int i) const { return list[i]; }
    __device__ const double* h(int i) const { return as_global(H.p[i]); }
};

// Sums over n^2 entries run in kSlices slices, one workgroup each, and the slices
// in a fixed order: bitwise reproducible.
constexpr int kSlices = 128, kEnergies = 3, kMaxSums = kEnergies + 16, kStepT = 256;

// Sums v[0 .. nd) of this workgroup's threads to part[(t0 + t) kSlices + slice]
template <int N>
__device__ inline void slice_sums(double (&v)[N], int nd, double* __restrict__ part) {
    __shared__ double red[N][kStepT / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t < N; ++t) {
        if (t < nd) {
            const double s = wave_sum(v[t]);
            if (lane == 0) red[t][wave] = s;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < nd) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kStepT / 64; ++w) s += red[threadIdx.x][w];
        part[threadIdx.x * kSlices + blockIdx.x] = s;
    }
}

// F = H + J - K/2, also to its history slot, and the slices of tr(DH), tr(DJ), tr(DK)
template <typename S>
__global__ __launch_bounds__(kStepT) void scf_fock(S src, ScfStep a) {
    const ScfMol& d = src.mol(blockIdx.z);
    const double *H = src.h(blockIdx.z), *J = as_global(d.J), *K = as_global(d.K), *D = as_global(d.D);
    const int64_t n2 = (int64_t)d.n * d.n, per = cdiv(n2, kSlices), beg = blockIdx.x * per;
    const int64_t end = beg + per < n2 ? beg + per : n2;
    double *F = as_global(d.F), *Fnew = as_global(d.Fh) + a.snew * n2;
    double s[kEnergies] = {};
    for (int64_t i = beg + threadIdx.x; i < end; i += kStepT) {
        const double h = H[i], j = J[i], k = K[i], dm = D[i];
        const double f = h + j - 0.5 * k;
        F[i] = f;
        Fnew[i] = f;
        s[0] = fma(dm, h, s[0]);
        s[1] = fma(dm, j, s[1]);
        s[2] = fma(dm, k, s[2]);
    }
    slice_sums(s, kEnergies, as_global(d.part));
}

// e = G - G^T to its history slot and the slices of its products with the stored ones
template <typename S>
__global__ __launch_bounds__(kStepT) void scf_error(S src, ScfStep a) {
    const ScfMol& d = src.mol(blockIdx.z);
    const int n = d.n;
    const int64_t n2 = (int64_t)n * n, per = cdiv(n2, kSlices), beg = blockIdx.x * per;
    const int64_t end = beg + per < n2 ? beg + per : n2;
    const double* G = as_global(d.G);
    double* Eh = as_global(d.Eh);
    double s[16] = {};
    for (int64_t i = beg + threadIdx.x; i < end; i += kStepT) {
        const int64_t r = i / n, c = i - r * n;
        const double e = G[i] - G[c * n + r];
        Eh[a.snew * n2 + i] = e;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            if (j < a.m) s[j] = fma(e, a.order.s[j] == a.snew ? e : Eh[a.order.s[j] * n2 + i], s[j]);
        }
    }
    slice_sums(s, a.m, as_global(d.part) + kEnergies * kSlices);
}

constexpr double kDiisMaxCond = 1e12;

// Extreme eigenvalues of the symmetric k x k matrix (k <= 15) in a by cyclic Jacobi
// rotations (Golub & Van Loan, Sec. 8.5), on one wavefront: lane r holds index r of
// the rotated rows and columns.
__device__ inline void small_eig_range(double (*a)[19], int k, double* lo, double* hi) {
    const int r = threadIdx.x;
    for (int sweep = 0; sweep < 30; ++sweep) {
        double off = 0.0, tot = 0.0;
        if (r < k)
            for (int j = 0; j < k; ++j) {
                const double x = a[r][j];
                tot += x * x;
                if (r != j) off += x * x;
            }
        off = wave_sum(off);
        tot = wave_sum(tot);
        if (off <= 1e-30 * tot) break;
        for (int p = 0; p < k - 1; ++p)
            for (int q = p + 1; q < k; ++q) {
                const double apq = a[p][q];
                if (apq == 0.0) continue;
                const double theta = (a[q][q] - a[p][p]) / (2.0 * apq);
                const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                const double c = 1.0 / sqrt(t * t + 1.0), sn = t * c;
                __syncthreads();
                if (r < k) {  // columns p, q
                    const double ap = a[r][p], aq = a[r][q];
                    a[r][p] = c * ap - sn * aq;
                    a[r][q] = sn * ap + c * aq;
                }
                __syncthreads();
                if (r < k) {  // rows p, q
                    const double ap = a[p][r], aq = a[q][r];
                    a[p][r] = c * ap - sn * aq;
                    a[q][r] = sn * ap + c * aq;
                }
                __syncthreads();
            }
    }
    double l = a[0][0], h = a[0][0];
    for (int i = 1; i < k; ++i) {
        l = fmin(l, a[i][i]);
        h = fmax(h, a[i][i]);
    }
    *lo = l;
    *hi = h;
}

// Energies, the newest error vector's row of the Gram matrix, the iteration's
// record, and the bordered DIIS system for the stored vectors in chronological
// order, solved by Gaussian elimination with partial pivoting (m <= 15).  The
// oldest vectors are dropped, for this and every later iteration, while the
// Gram matrix of the remaining error vectors has a 2-norm condition number
// above kDiisMaxCond (or is singular); at least the newest stays.  first[0]
// holds the oldest iteration still in use (reset on iteration 1).  coef gets
// m entries in the order of `order`, zero for dropped vectors.
// One wavefront per molecule; its chain of divisions and roots bounds it: lanes hold
// the rows.
template <typename S>
__global__ __launch_bounds__(64) void scf_solve(S src, ScfStep st) {
    __shared__ double sum[kMaxSums], g[16][17], a[17][19], x[16];
    const ScfMol& d = src.mol(blockIdx.z);
    const int lane = threadIdx.x, m = st.m, space = st.space, iter = st.iter;
    const double* part = as_global(d.part);
    double *gram = as_global(d.gram), *first = as_global(d.first), *coef = as_global(d.coef);
    for (int t = 0; t < kEnergies + m; ++t) {
        const double s = wave_sum(part[t * kSlices + lane] + part[t * kSlices + 64 + lane]);
        if (lane == 0) sum[t] = s;
    }
    __syncthreads();
    // Gram matrix in chronological order, the newest last
    for (int e = lane; e < m * m; e += 64) {
        const int i = e / m, j = e % m, si = st.order.s[i], sj = st.order.s[j];
        const double v = si == st.snew ? sum[kEnergies + j] : sj == st.snew ? sum[kEnergies + i] : gram[si * space + sj];
        g[i][j] = v;
        if (si == st.snew || sj == st.snew) gram[si * space + sj] = v;
    }
    __syncthreads();
    if (lane == 0) {
        ScfRecord r;
        r.e_1e = sum[0];
        r.e_j = 0.5 * sum[1];
        r.e_k = -0.25 * sum[2];
        r.e_tot = r.e_1e + r.e_j + r.e_k;
        r.err_norm = sqrt(g[m - 1][m - 1]);
        r.d_e = iter > 1 ? r.e_tot - *d.e_prev : r.e_tot;
        r.iter = iter;
        r.converged = (iter > 1 && fabs(r.d_e) < st.conv_tol && r.err_norm < st.conv_tol_grad) ? 1 : 0;
        *d.e_prev = r.e_tot;
        *d.rec = r;
    }
    const int it0 = iter - m + 1;  // iteration of order.s[0]
    int k0 = 0;                     // first index of order still kept
    if (iter > 1) {
        const int f = (int)first[0];
        k0 = f > it0 ? f - it0 : 0;
    }
    if (k0 > m - 1) k0 = m - 1;
    while (k0 < m - 1) {
        const int k = m - k0;
        __syncthreads();
        for (int e = lane; e < k * k; e += 64) a[e / k][e % k] = g[k0 + e / k][k0 + e % k];
        __syncthreads();
        double lo, hi;
        small_eig_range(a, k, &lo, &hi);
        if (lo > 0.0 && hi / lo <= kDiisMaxCond) break;
        ++k0;
    }
    __syncthreads();
    if (lane == 0) first[0] = (double)(it0 + k0);
    if (lane < k0) coef[lane] = 0.0;
    const int mk = m - k0;  // vectors kept: order.s[k0 .. m-1]
    const int n = mk + 1;
    for (int e = lane; e < n * (n + 1); e += 64) {
        const int i = e / (n + 1), j = e % (n + 1);
        a[i][j] = i < mk && j < mk ? g[k0 + i][k0 + j] : j == n ? (i == mk ? -1.0 : 0.0) : i == mk && j == mk ? 0.0 : -1.0;
    }
    __syncthreads();
    bool singular = false;
    for (int col = 0; col < n; ++col) {
        int piv = col;
        for (int r = col + 1; r < n; ++r)
            if (fabs(a[r][col]) > fabs(a[piv][col])) piv = r;
        if (a[piv][col] == 0.0) {
            singular = true;
            break;
        }
        __syncthreads();
        if (piv != col && lane <= n) {
            const double t = a[col][lane];
            a[col][lane] = a[piv][lane];
            a[piv][lane] = t;
        }
        __syncthreads();
        if (lane > col && lane < n) {
            const double f = a[lane][col] / a[col][col];
            for (int c = col; c <= n; ++c) a[lane][c] -= f * a[col][c];
        }
        __syncthreads();
    }
    if (!singular && lane == 0)
        for (int r = n - 1; r >= 0; --r) {
            double t = a[r][n];
            for (int c = r + 1; c < n; ++c) t -= a[r][c] * x[c];
            x[r] = t / a[r][r];
        }
    __syncthreads();
    if (lane < mk) coef[k0 + lane] = singular ? (lane == mk - 1 ? 1.0 : 0.0) : x[lane];
}

// F' = sum_j coef_j F_j
template <typename S>
__global__ __launch_bounds__(kStepT) void scf_combine(S src, ScfStep a) {
    const ScfMol& d = src.mol(blockIdx.z);
    const int64_t n2 = (int64_t)d.n * d.n, i = (int64_t)blockIdx.x * kStepT + threadIdx.x;
    if (i >= n2) return;
    const double *Fh = as_global(d.Fh), *coef = as_global(d.coef);
    double s = 0.0;
    for (int j = 0; j < a.m; ++j) s += coef[j] * Fh[a.order.s[j] * n2 + i];
    as_global(d.Fx)[i] = s;
}

// The step's products in 16 x 16 tiles
enum { PR_FD = 0, PR_FV, PR_VG, PR_CC };  // G = F D; G = F' V^T; F' = V G; D = 2 C C^T
template <typename S, int PR>
__global__ __launch_bounds__(256) void scf_product(S src) {
    const ScfMol& d = src.mol(blockIdx.z);
    const int n = d.n;
    if ((int)blockIdx.x * 16 >= n || (int)blockIdx.y * 16 >= n) return;
    const double *F = as_global(d.F), *V = as_global(d.V);
    double *G = as_global(d.G), *Fx = as_global(d.Fx), *D = as_global(d.D);
    if (PR == PR_FD) gemm_tile16<false, false>(n, n, n, 1.0, F, n, D, n, 0.0, G, n);
    if (PR == PR_FV) gemm_tile16<false, true>(n, n, n, 1.0, Fx, n, V, n, 0.0, G, n);
    if (PR == PR_VG) gemm_tile16<false, false>(n, n, n, 1.0, V, n, G, n, 0.0, Fx, n);
    if (PR == PR_CC) {
        const double* C = as_global(d.C);
        gemm_tile16<false, true>(n, n, d.nocc, 2.0, C, d.nocc, C, d.nocc, 0.0, D, n);
    }
}

}  // namespace

// Workspace carved from h->eig: see scf_ws().
struct ScfWs {
    EigWork eig;                           // eigen-work (also used by the D path of K)
    double *V, *Cf, *sign;
    double *J, *K, *F, *G, *Fx;            // SCF matrices
    double *Fh, *Eh;                       // DIIS history: space x n^2 each
    double *gram, *coef, *part, *e_prev, *diis_first;
    ScfRecord* rec;
};

// log: with the eigensolver's log of rotations, the last part (a batch lends its own)
static int scf_ws(dfjk_ctx* h, bool scf, ScfWs& ws, bool log = true) {
    const int64_t n = h->nao, n2 = n * n;
    const int space = h->opts.diis_space;
    size_t need = 0;
    auto take = [&](size_t elems) {
        const size_t off = need;
        need += (elems + 31) / 32 * 32;
        return off;
    };
    const size_t oA = take(n2), oV = take(n2), ow = take(n), owork = take(n + 2), oCf = take(n2),
                 osign = take(n), oiw = take((EigWork::iwork_elems(n) + 1) / 2);
    size_t oJ = 0, oK = 0, oF = 0, oG = 0, oFx = 0, oFh = 0, oEh = 0, ogr = 0, oco = 0, opart = 0, oep = 0,
           orec = 0, ofirst = 0;
    if (scf) {
        oJ = take(n2), oK = take(n2), oF = take(n2), oG = take(n2), oFx = take(n2);
        oFh = take((size_t)space * n2), oEh = take((size_t)space * n2);
        ogr = take((size_t)space * space), oco = take(16), opart = take(kMaxSums * kSlices), oep = take(1),
        orec = take(sizeof(ScfRecord) / sizeof(double) + 1), ofirst = take(1);
    }
    const size_t olog = take(log ? EigWork::log_elems(n) : 0);
    if (need * sizeof(double) > h->eig.bytes) h->scf_v_warm = false;  // fresh buffer
    int rc = h->eig.ensure(need * sizeof(double));
    if (rc) return rc;
    double* base = static_cast<double*>(h->eig.ptr);
    ws.eig = EigWork{base + oA, base + owork, log ? base + olog : nullptr, reinterpret_cast<int*>(base + oiw), base + ow};
    ws.V = base + oV;
    ws.Cf = base + oCf;
    ws.sign = base + osign;
    if (scf) {
        ws.J = base + oJ;
        ws.K = base + oK;
        ws.F = base + oF;
        ws.G = base + oG;
        ws.Fx = base + oFx;
        ws.Fh = base + oFh;
        ws.Eh = base + oEh;
        ws.gram = base + ogr;
        ws.coef = base + oco;
        ws.part = base + opart;
        ws.e_prev = base + oep;
        ws.rec = reinterpret_cast<ScfRecord*>(base + orec);
        ws.diis_first = base + ofirst;
    }
    return DFJK_OK;
}

// K of a density from D itself instead of D's eigen-factors: always with FP64 B (the
// eigensolver alone takes 1 ms at nao=128), from this nao on with FP32 compute,
// where the two differ by the FP32 sums (nao=200, naux=800: 61 ms through the
// factors, almost all of it the eigensolver; nao=300, naux=900 1.4 ms without them).
constexpr int64_t kDensityF32 = 256;

int k_build_from_D(dfjk_ctx* h, const double* D, double* K) {
    const int64_t n = h->nao;
    h->scf_v_warm = false;  // the eigensolver's buffers are used below
    if (n > kMaxEighN) {
        set_error("K from a density needs nao <= %d (got %lld); pass Cocc", kMaxEighN, (long long)n);
        return DFJK_E_INVALID;
    }
    // the SCF workspace also holds the eigen-work; keep it if it exists
    ScfWs ws;
    int rc = scf_ws(h, h->scf_ready, ws);
    if (rc) return rc;
    const hipStream_t st = h->stream;
    if (h->opts.max_ncol == 0 && (h->dtype == DFJK_F64 || n >= kDensityF32)) {
        // K = sum_P B_P D B_P; a reserved workspace (at most nao columns) keeps the
        // eigen-factor path, which fits it
        symmetrize_kernel<<<dim3((unsigned)cdiv(n * n, 256)), 256, 0, st>>>(D, n, ws.eig.A);
        DFJK_LAUNCH_CHECK("symmetrize_kernel");
        rc = k_build_density(h, ws.eig.A, K);
        // its rows of B_P D and of B_P may not fit where the factors' rows, half as many,
        // do; from kDensityF32 on an eigensolution would take far longer than the build
        if (rc != DFJK_E_OOM || n >= kDensityF32) return rc;
        clear_error();
    }
    // D = sum_c w_c v_c v_c^T = sum_c sign_c (sqrt|w_c| v_c)(sqrt|w_c| v_c)^T
    if ((rc = eigh_cols(st, D, ws.V, (int)n, true, ws.eig, (int)n, 1, ws.Cf, ws.sign))) return rc;
    return k_build_factored(h, ws.Cf, n, ws.sign, 1.0, K);
}

int aufbau(dfjk_ctx* h, const double* F, int64_t nocc, double* C, double* D) {
    const int64_t n = h->nao;
    h->scf_v_warm = false;
    if (n > kMaxEighN) {
        set_error("dfjk_aufbau: nao=%lld above %d", (long long)n, kMaxEighN);
        return DFJK_E_INVALID;
    }
    ScfWs ws;
    int rc = scf_ws(h, h->scf_ready, ws);
    if (rc) return rc;
    const hipStream_t st = h->stream;
    if ((rc = eigh_cols(st, F, ws.V, (int)n, true, ws.eig, (int)nocc, 0, C, nullptr))) return rc;
    if (D) return dgemm(st, false, true, n, n, nocc, 2.0, C, nocc, C, nocc, 0.0, D, n);
    return DFJK_OK;
}

int scf_reserve(dfjk_ctx* h) {
    ScfWs ws;
    return scf_ws(h, true, ws);
}

int scf_reset(dfjk_ctx* h) {
    h->scf_v_warm = false;
    h->scf_iter = 0;
    h->scf_count = 0;
    return DFJK_OK;
}

int scf_step(dfjk_ctx* h, const double* H, double* D, double* C, int64_t nocc, int flags,
             dfjk_scf_info* info) {
    const int64_t n = h->nao;
    if (n > kMaxEighN) {
        set_error("dfjk_scf_step: nao=%lld above %d", (long long)n, kMaxEighN);
        return DFJK_E_INVALID;
    }
    ScfWs ws;
    int rc = scf_ws(h, true, ws);
    if (rc) return rc;
    h->scf_ready = true;
    // J and K of the current density
    if ((rc = j_build(h, D, ws.J, nullptr, nullptr))) return rc;
    if (flags & DFJK_SCF_C_VALID)
        rc = k_build_factored(h, C, nocc, nullptr, 2.0, ws.K);
    else
        rc = k_build_from_D(h, D, ws.K);
    if (rc) return rc;
    const void* rec = nullptr;
    if ((rc = scf_tail(h, H, D, C, nocc, ws.J, ws.K, &rec))) return rc;
    if (info) return scf_read_info(h, rec, info);
    return DFJK_OK;
}

int scf_read_info(dfjk_ctx* h, const void* rec, dfjk_scf_info* info) {
    DFJK_HIP_TRY(hipMemcpyAsync(info, rec, sizeof(ScfRecord), hipMemcpyDeviceToHost, h->stream));
    DFJK_HIP_TRY(hipStreamSynchronize(h->stream));
    if (!(info->e_tot == info->e_tot)) {
        set_error("dfjk_scf_step: non-finite energy at iteration %d", info->iter);
        return DFJK_E_NONFINITE;
    }
    return info->converged ? DFJK_OK : DFJK_W_NOT_CONVERGED;
}

// The next iteration's step of a handle
static ScfStep next_step(const dfjk_ctx* h) {
    ScfStep a{};
    a.space = h->opts.diis_space;
    a.iter = h->scf_iter + 1;
    a.snew = (a.iter - 1) % a.space;
    a.m = h->scf_count + 1 < a.space ? h->scf_count + 1 : a.space;
    for (int j = 0; j < a.m; ++j) a.order.s[j] = (a.iter - a.m + j) % a.space;
    a.conv_tol = h->opts.conv_tol;
    a.conv_tol_grad = h->opts.conv_tol_grad;
    return a;
}

static ScfMol describe(const dfjk_ctx* h, const ScfWs& ws, double* D, double* C, int64_t nocc, const double* J,
                       const double* K) {
    return ScfMol{(int)h->nao, (int)nocc, J,     K,       D,       C,        ws.V,      ws.F,
                  ws.G,        ws.Fx,     ws.Fh, ws.Eh,   ws.gram, ws.coef,  ws.part,   ws.e_prev,
                  ws.diis_first, ws.rec,  ws.eig};
}

// The kernels from the Fock matrix to F' over nmol molecules of up to n functions
// (F D by the caller where the tiles of scf_product are not the right ones)
template <typename S, typename FD>
static int fock_to_diis(hipStream_t st, const S& src, const ScfStep& a, int64_t n, unsigned nmol, FD product_fd) {
    scf_fock<S><<<dim3(kSlices, 1, nmol), kStepT, 0, st>>>(src, a);
    DFJK_LAUNCH_CHECK("scf_fock");
    if (int rc = product_fd()) return rc;
    scf_error<S><<<dim3(kSlices, 1, nmol), kStepT, 0, st>>>(src, a);
    DFJK_LAUNCH_CHECK("scf_error");
    scf_solve<S><<<dim3(1, 1, nmol), 64, 0, st>>>(src, a);
    DFJK_LAUNCH_CHECK("scf_solve");
    scf_combine<S><<<dim3((unsigned)cdiv(n * n, kStepT), 1, nmol), kStepT, 0, st>>>(src, a);
    DFJK_LAUNCH_CHECK("scf_combine");
    return DFJK_OK;
}

// Everything of an SCF iteration after J and K: Fock matrix, energies,
// commutator, DIIS, aufbau, next D and C, on the handle's stream.  *rec gets
// the device address of the iteration record.
int scf_tail(dfjk_ctx* h, const double* H, double* D, double* C, int64_t nocc, const double* J,
             const double* K, const void** rec) {
    const int64_t n = h->nao;
    ScfWs ws;
    int rc = scf_ws(h, true, ws);
    if (rc) return rc;
    h->scf_ready = true;
    const hipStream_t st = h->stream;
    const ScfStep a = next_step(h);
    const One src{describe(h, ws, D, C, nocc, J, K), H};
    rc = fock_to_diis(st, src, a, n, 1,
                      [&] { return dgemm(st, false, false, n, n, n, 1.0, ws.F, n, D, n, 0.0, ws.G, n); });
    if (rc) return rc;
    // aufbau on the extrapolated Fock matrix; from the second iteration on the
    // Jacobi sweeps start in the previous eigenbasis (rows of V): V F V^T is
    // then nearly diagonal and needs few sweeps; V accumulates the rotations
    const bool warm = h->scf_v_warm;
    if (warm) {
        if ((rc = dgemm(st, false, true, n, n, n, 1.0, ws.Fx, n, ws.V, n, 0.0, ws.G, n))) return rc;
        if ((rc = dgemm(st, false, false, n, n, n, 1.0, ws.V, n, ws.G, n, 0.0, ws.Fx, n))) return rc;
    }
    if ((rc = eigh_cols(st, ws.Fx, ws.V, (int)n, !warm, ws.eig, (int)nocc, 0, C, nullptr))) return rc;
    h->scf_v_warm = true;
    if ((rc = dgemm(st, false, true, n, n, nocc, 2.0, C, nocc, C, nocc, 0.0, D, n))) return rc;

    h->scf_iter = a.iter;
    h->scf_count = a.m;
    *rec = ws.rec;
    return DFJK_OK;
}

// ---- all molecules of a batch at once (n <= kEigLdsN)

int scf_describe(dfjk_ctx* h, double* D, double* C, int64_t nocc, const double* J, const double* K, void* rec,
                 double* log, ScfMol* out) {
    ScfWs ws;
    if (int rc = scf_ws(h, true, ws, false)) return rc;
    h->scf_ready = true;
    *out = describe(h, ws, D, C, nocc, J, K);
    out->eig.log = log;
    out->rec = static_cast<ScfRecord*>(rec);
    return DFJK_OK;
}

template <int PR>
static int product_many(hipStream_t st, const Many& src, int max_n, unsigned nmol) {
    const unsigned nt = (unsigned)cdiv(max_n, 16);
    scf_product<Many, PR><<<dim3(nt, nt, nmol), 256, 0, st>>>(src);
    DFJK_LAUNCH_CHECK("scf_product");
    return DFJK_OK;
}

int scf_tail_many(hipStream_t st, const ScfMol* mols, dfjk_ctx* const* h, const double* const* H, int nmol) {
    int max_n = 0, lds_n = 1;
    for (int i = 0; i < nmol; ++i) {
        const int n = (int)h[i]->nao;
        max_n = std::max(max_n, n);
        if (eig_lds_bytes(n) > eig_lds_bytes(lds_n)) lds_n = n;
    }
    Many src{mols, {}};
    for (int i = 0; i < nmol; ++i) src.H.p[i] = H[i];
    const ScfStep a = next_step(h[0]);
    const bool warm = h[0]->scf_v_warm;
    int rc = fock_to_diis(st, src, a, max_n, (unsigned)nmol,
                          [&] { return product_many<PR_FD>(st, src, max_n, (unsigned)nmol); });
    if (rc) return rc;
    if (warm) {
        if ((rc = product_many<PR_FV>(st, src, max_n, (unsigned)nmol))) return rc;
        if ((rc = product_many<PR_VG>(st, src, max_n, (unsigned)nmol))) return rc;
    }
    if ((rc = eig_lds_many(st, mols, nullptr, !warm, nmol, max_n, lds_n))) return rc;
    if ((rc = product_many<PR_CC>(st, src, max_n, (unsigned)nmol))) return rc;
    for (int i = 0; i < nmol; ++i) {
        h[i]->scf_v_warm = true;
        h[i]->scf_iter = a.iter;
        h[i]->scf_count = a.m;
    }
    return DFJK_OK;
}

int aufbau_many(hipStream_t st, const ScfMol* mols, dfjk_ctx* const* h, const double* const* F, int nmol) {
    int max_n = 0, lds_n = 1;
    for (int i = 0; i < nmol; ++i) {
        const int n = (int)h[i]->nao;
        h[i]->scf_v_warm = false;
        max_n = std::max(max_n, n);
        if (eig_lds_bytes(n) > eig_lds_bytes(lds_n)) lds_n = n;
    }
    Many src{mols, {}};
    for (int i = 0; i < nmol; ++i) src.H.p[i] = F[i];
    if (int rc = eig_lds_many(st, mols, &src.H, true, nmol, max_n, lds_n)) return rc;
    return product_many<PR_CC>(st, src, max_n, (unsigned)nmol);
}

}  // namespace dfjk
