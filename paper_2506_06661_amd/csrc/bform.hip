// The 3-index factor of the density-fitted integrals (Sec. IV.C.2, the T of
// Eq. eq:df:eri): M = L L^T (Cholesky of the auxiliary metric, lower L) and
// T = L^-1 Q for the 3-index integrals Q = (P|mu nu), one column per packed
// pair.  Both factorisation and substitution are blocked by 64 rows:
//   Cholesky, for each diagonal block k: factor L_kk and invert it; panel L_ik = M_ik L_kk^-T in place and trailing
//     update M_ij -= L_ik L_jk^T of the lower block triangle, 64 x 64 tiles on
//     the FP64 matrix cores.
//   Substitution, for each panel of 128 rows: the product with all rows above,
//     then Q_k <- L_kk^-1 Q_k and Q_i -= L_ik Q_k inside the panel.
// The 64 x 64 diagonal blocks are applied through their explicit inverses
// (forward substitution on the identity), which keeps every large step on
// the matrix cores; the accuracy is that of the diagonal blocks' condition.
// All sums run in a fixed order: the result is bitwise reproducible.
#include "internal.h"
#include "mma.h"

namespace dfjk {
namespace {

constexpr int NB = 64;    // block size (diagonal blocks, Cholesky panels)
constexpr int NB2 = 128;  // row panel of the substitution (2 diagonal blocks)
constexpr int kT = 256;
constexpr int TP = NB + 16;  // LDS pitch of a 64 x 64 block: 16 modulo 32 doubles

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// A 64 x 64 block whose rows are contiguous along the contraction index k is
// kept as LDS rows of k (operand reads: 16 consecutive rows of the block at 4
// k); row k keeps column m at m ^ swz(k), so the transposed stores of a pair of
// k fall on different banks.
__device__ inline int swz(int k) { return 2 * ((k >> 1) & 7); }

__device__ inline double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Factor the kb x kb diagonal block at (k0, k0) of A (row-major, lda) in
// place (lower triangle <- L_kk, strict upper <- 0) and write its inverse,
// padded to 64 x 64 with the identity, to Linv.  A non-positive (or
// non-finite) pivot sets *flag.  The chain of 64 columns is what bounds it (the
// rest of the factorisation waits), so it is cut into panels of 16 columns: one
// wavefront factors a panel without barriers (lane i holds row i's 16 entries, a
// column's entries reach the other lanes through scalar registers), the matrix
// cores update the rest.  The inverse: each wavefront a 16 x 16 diagonal block,
// then the blocks below by distance from the diagonal.  On MI355X 23 us a
// block; all 64 columns in one wavefront's registers 45 us (19000 instructions,
// each run once), 256 threads with three barriers a column 226 us.
__global__ __launch_bounds__(kT) void chol_diag(double* __restrict__ A, int64_t lda, int64_t k0, int kb,
                                                double* __restrict__ Linv, int* __restrict__ flag) {
    __shared__ double T[NB][NB + 1], X[NB][NB + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 15, lq = lane >> 4;
#pragma unroll
    for (int q = 0; q < NB * NB / kT; ++q) {
        const int e = tid + q * kT, i = e / NB, j = e % NB;
        T[i][j] = (i < kb && j <= i) ? A[(k0 + i) * lda + k0 + j] : (i == j ? 1.0 : 0.0);
    }
    __syncthreads();
#pragma unroll 1
    for (int p = 0; p < 4; ++p) {
        if (wave == 0) {
            double a[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) a[j] = T[lane][16 * p + j];
            bool bad = false;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const double d = lane_value(a[j], 16 * p + j);
                bad |= !(d > 0.0) || !(d < 1e300);
                const double s = sqrt(d);  // NaN for a non-positive pivot; reported through flag
                const double l = a[j] / s;
#pragma unroll
                for (int k = j + 1; k < 16; ++k) a[k] = fma(-l, lane_value(l, 16 * p + k), a[k]);
                a[j] = lane == 16 * p + j ? s : lane > 16 * p + j ? l : 0.0;
            }
            if (bad && lane == 0) flag[0] = 1;
#pragma unroll
            for (int j = 0; j < 16; ++j) T[lane][16 * p + j] = a[j];
        }
        __syncthreads();
        int t = 0;
        for (int I = p + 1; I < 4; ++I)
            for (int J = p + 1; J <= I; ++J, ++t) {
                if ((t & 3) != wave) continue;
                v4d acc;
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] = T[16 * I + Mma<double>::row(lane, r)][16 * J + lc];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    acc = Mma<double>::step(-T[16 * I + lc][16 * p + 4 * kk + lq], T[16 * J + lc][16 * p + 4 * kk + lq],
                                            acc);
#pragma unroll
                for (int r = 0; r < 4; ++r) T[16 * I + Mma<double>::row(lane, r)][16 * J + lc] = acc[r];
            }
        __syncthreads();
    }
    // column lc of the inverse of diagonal block `wave`: L x = e_lc, rows in order
    {
        const int b = 16 * wave;
        double x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            double sum = j == lc ? 1.0 : 0.0;
#pragma unroll
            for (int l = 0; l < j; ++l) sum = fma(-T[b + j][b + l], x[l], sum);
            x[j] = j < lc ? 0.0 : sum / T[b + j][b + j];
        }
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if (lq == 0) X[b + j][b + lc] = x[j];
    }
    __syncthreads();
    // X_ij = -X_ii sum_{j <= k < i} L_ik X_kj
#pragma unroll 1
    for (int d = 1; d < 4; ++d) {
        const int i = wave, j = wave - d;
        if (j >= 0) {
            v4d sum = Mma<double>::zero(), acc = Mma<double>::zero();
            for (int k = j; k < i; ++k)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    sum = Mma<double>::step(T[16 * i + lc][16 * k + 4 * kk + lq], X[16 * k + 4 * kk + lq][16 * j + lc],
                                            sum);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)  // a result row block is the operand of step kk
                acc = Mma<double>::step(-X[16 * i + lc][16 * i + 4 * kk + lq], sum[kk], acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) X[16 * i + Mma<double>::row(lane, r)][16 * j + lc] = acc[r];
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < NB * NB / kT; ++q) {
        const int e = tid + q * kT, i = e / NB, j = e % NB;
        Linv[e] = j <= i ? X[i][j] : 0.0;
        if (i < kb && j < kb) A[(k0 + i) * lda + k0 + j] = j <= i ? T[i][j] : 0.0;
    }
}

// One 64 x 64 block (rows ld apart, nrow valid ones: the others zero) into LDS
// as rows of k
template <int NT>
struct Block64 {
    static constexpr int N = NB * NB / 2 / NT;  // pairs per thread
    double v[N][2];
    __device__ inline void load(const double* __restrict__ src, int64_t ld, int nrow, int tid) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int e = tid + j * NT, r = e / 32, k = 2 * (e % 32);
            __builtin_memcpy(v[j], src + (r < nrow ? r : 0) * ld + k, 16);
        }
    }
    __device__ inline void store(double (*S)[TP], int nrow, bool neg, int tid) const {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int e = tid + j * NT, r = e / 32, k = 2 * (e % 32);
#pragma unroll
            for (int d = 0; d < 2; ++d) S[k + d][r ^ swz(k)] = r < nrow ? (neg ? -v[j][d] : v[j][d]) : 0.0;
        }
    }
};

// operand of a 64-deep product: element (row 16 q + lane % 16, k = 4 kk + lane / 16) of the block
__device__ inline double oper(const double (*S)[TP], int q, int kk, int lane) {
    const int k = 4 * kk + (lane >> 4);
    return S[k][q * 16 + ((lane & 15) ^ swz(k))];
}

// Panel below the diagonal block: rows [r0, r0 + 64) of P (64 columns wide)
// <- P Linv^T, in place: a workgroup owns its rows.
__global__ __launch_bounds__(kT) void chol_panel(double* __restrict__ P, int64_t lda, int64_t n,
                                                 const double* __restrict__ Linv) {
    __shared__ __attribute__((aligned(16))) double sA[NB][TP], sB[NB][TP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int64_t r0 = (int64_t)blockIdx.x * NB;
    const int nrow = n - r0 < NB ? (int)(n - r0) : NB;
    Block64<kT> ba, bb;
    ba.load(P + r0 * lda, lda, nrow, tid);
    bb.load(Linv, NB, NB, tid);
    ba.store(sA, nrow, false, tid);
    bb.store(sB, NB, false, tid);
    __syncthreads();
    v4d acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x) acc[x][0] = acc[x][1] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < NB / 4; ++kk) {
        const double a0 = oper(sA, 2 * wm, kk, lane), a1 = oper(sA, 2 * wm + 1, kk, lane);
        const double b0 = oper(sB, 2 * wn, kk, lane), b1 = oper(sB, 2 * wn + 1, kk, lane);
        acc[0][0] = Mma<double>::step(a0, b0, acc[0][0]);
        acc[0][1] = Mma<double>::step(a0, b1, acc[0][1]);
        acc[1][0] = Mma<double>::step(a1, b0, acc[1][0]);
        acc[1][1] = Mma<double>::step(a1, b1, acc[1][1]);
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = wm * 32 + x * 16 + Mma<double>::row(lane, r), col = wn * 32 + y * 16 + (lane & 15);
                if (row < nrow) P[(r0 + row) * lda + col] = acc[x][y][r];
            }
}

// Trailing update C_ij -= P_i P_j^T of the lower block triangle (64 x 64 tiles,
// P: n rows of 64).  The 64 terms are summed by themselves and then subtracted once:
// each has a fraction of C's size, and rounding the running result at every one of them
// made L's error four times as large (naux=1024: 3.6e-16 -> 1.4e-15).
__global__ __launch_bounds__(kT) void chol_update(const double* __restrict__ P, double* __restrict__ C, int64_t lda,
                                                  int64_t n) {
    __shared__ __attribute__((aligned(16))) double sA[NB][TP], sB[NB][TP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int64_t t = blockIdx.x;
    int64_t I = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (I * (I + 1) / 2 > t) --I;
    while ((I + 1) * (I + 2) / 2 <= t) ++I;
    const int64_t J = t - I * (I + 1) / 2, m0 = I * NB, n0 = J * NB;
    const int nr = n - m0 < NB ? (int)(n - m0) : NB, nc = n - n0 < NB ? (int)(n - n0) : NB;
    Block64<kT> ba, bb;
    ba.load(P + m0 * lda, lda, nr, tid);
    bb.load(P + n0 * lda, lda, nc, tid);
    v4d acc[2][2], old[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = wm * 32 + x * 16 + Mma<double>::row(lane, r), col = wn * 32 + y * 16 + (lane & 15);
                old[x][y][r] = row < nr && col < nc ? C[(m0 + row) * lda + n0 + col] : 0.0;
                acc[x][y][r] = 0.0;
            }
    ba.store(sA, nr, true, tid);
    bb.store(sB, nc, false, tid);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < NB / 4; ++kk) {
        const double a0 = oper(sA, 2 * wm, kk, lane), a1 = oper(sA, 2 * wm + 1, kk, lane);
        const double b0 = oper(sB, 2 * wn, kk, lane), b1 = oper(sB, 2 * wn + 1, kk, lane);
        acc[0][0] = Mma<double>::step(a0, b0, acc[0][0]);
        acc[0][1] = Mma<double>::step(a0, b1, acc[0][1]);
        acc[1][0] = Mma<double>::step(a1, b0, acc[1][0]);
        acc[1][1] = Mma<double>::step(a1, b1, acc[1][1]);
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = wm * 32 + x * 16 + Mma<double>::row(lane, r), col = wn * 32 + y * 16 + (lane & 15);
                if (row < nr && col < nc) C[(m0 + row) * lda + n0 + col] = old[x][y][r] + acc[x][y][r];
            }
}

// strict upper triangle of M <- 0
__global__ void zero_upper(double* __restrict__ M, int64_t n, int64_t i0) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, i = i0 + blockIdx.y;
    if (j < n && j > i) M[i * n + j] = 0.0;
}

// Q <- L^-1 Q, one launch: a workgroup owns 64 columns and takes the rows in
// panels of 128, so nothing crosses workgroups.  A wavefront holds 16 columns of
// all the panel's rows in registers, as accumulators: first
// -L[panel, above] Q[above], in 32-deep chunks (L staged in LDS one
// chunk ahead for the four wavefronts, each one's columns of Q straight from
// global memory into operand registers), then the triangle inside the panel, 64
// rows at a time: the FP64 result layout (row 4 r + lane / 16 of a 16 x 16 block)
// is the operand layout of the 4-deep step r, so Q_k <- Linv_k Q_k feeds
// Q_i -= L_ik Q_k without leaving the registers.  Sums start at zero and are added to
// Q per 256 rows above and per 64 inside the panel: a running result that starts as Q
// rounds all of it at every term (error of B at naux=1536 1.2e-15, 5.1e-15 together with
// the same in chol_update).  Q and the sums of the panel are in registers side by side;
// panels of 256 rows have no room for that and went through memory at every
// addition (4.28 ms).  The matrix cores bound it.
// naux=1536, 73920 columns: 4.17 ms, 42 TFLOP/s (1155 workgroups in 512 slots: the third
// round is a quarter full; 4.06 with running results in panels of 256); with an update
// of all rows below after each panel (Q rewritten 5 times) 5.0 ms, with one
// product, one copy and one update per 64 rows 7.6 ms.
constexpr int SK = 32, SP = NB2 + 16;  // chunk depth; LDS pitch (16 modulo 32)
constexpr int SFOLD = 256;             // rows above per sum
__global__ __launch_bounds__(kT, 2) void solve(const double* __restrict__ L, int64_t naux,
                                               const double* __restrict__ Linv, double* __restrict__ Q, int64_t ldQ,
                                               int64_t ncol) {
    __shared__ __attribute__((aligned(16))) double smem[2 * NB * TP];
    static_assert(2 * SK * SP <= 2 * NB * TP, "LDS");
    double(*S)[NB][TP] = reinterpret_cast<double(*)[NB][TP]>(smem);
    double(*sA)[SK][SP] = reinterpret_cast<double(*)[SK][SP]>(smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t col = (int64_t)blockIdx.x * 64 + wave * 16 + (lane & 15);
    const bool live = col < ncol;
    double* Qc = Q + (live ? col : ncol - 1) + (lane >> 4) * ldQ;  // this lane's row of a 4-deep step
    constexpr int KB = NB2 / NB;                                   // blocks per panel
    for (int64_t K0 = 0; K0 < naux; K0 += NB2) {
        const int nrow = naux - K0 < NB2 ? (int)(naux - K0) : NB2, nb = (nrow + NB - 1) / NB;
        // leading dimensions and thread as if new in each panel: their multiples
        // held over the panels would not fit the registers
        int64_t ld = naux, step = 4 * ldQ;
        int t = tid;
        asm volatile("" : "+s"(ld), "+s"(step), "+v"(t));
        const double* Lp = L + K0 * ld;
        double* Qp = Qc + K0 * ldQ;
        double q[KB][16];  // block k, element e: row K0 + 64 k + 4 e + lane / 16
        if (nrow == NB2) {
            const double* p = Qp;
#pragma unroll
            for (int e = 0; e < 16 * KB; ++e, p += step) q[e >> 4][e & 15] = *p;
        } else {
            const double* p = Qp;
            asm volatile("" ::: "memory");  // stays a branch
#pragma unroll
            for (int e = 0; e < 16 * KB; ++e, p += step) q[e >> 4][e & 15] = 4 * e + (lane >> 4) < nrow ? *p : 0.0;
        }
        // ---- rows above the panel
        if (K0 > 0) {
            const int ar = t >> 4, akp = 2 * (t & 15);  // staged pairs: row ar + 16 j at k = akp
            const int64_t aoff = ar * ld + akp;
            double ra[NB2 / 16][2], rb[SK / 4];
            auto load_a = [&](int64_t kc) {
                if (nrow == NB2) {
#pragma unroll
                    for (int j = 0; j < NB2 / 16; ++j) __builtin_memcpy(ra[j], Lp + kc + 16 * j * ld + aoff, 16);
                } else {
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int j = 0; j < NB2 / 16; ++j) {
                        ra[j][0] = ra[j][1] = 0.0;
                        if (ar + 16 * j < nrow) __builtin_memcpy(ra[j], Lp + kc + 16 * j * ld + aoff, 16);
                    }
                }
            };
            // row k of a chunk keeps row m of L at m ^ (k & ~1): the 16 pairs of a store on
            // different banks
            auto store_a = [&](int buf) {
#pragma unroll
                for (int j = 0; j < NB2 / 16; ++j) {
                    sA[buf][akp][(ar + 16 * j) ^ akp] = -ra[j][0];
                    sA[buf][akp + 1][(ar + 16 * j) ^ akp] = -ra[j][1];
                }
            };
            auto load_b = [&](int64_t kc) {
                const double* Qk = Qc + kc * ldQ;
#pragma unroll
                for (int kk = 0; kk < SK / 4; ++kk) rb[kk] = Qk[kk * step];
            };
            v4d acc[KB][4];
#pragma unroll
            for (int h = 0; h < KB; ++h)
#pragma unroll
                for (int m = 0; m < 4; ++m) acc[h][m] = Mma<double>::zero();
            load_a(0);
            load_b(0);
            store_a(0);
            load_a(SK);  // K0 is a multiple of NB2: there are at least four chunks
            __syncthreads();
            int buf = 0;
            for (int64_t kc = 0; kc < K0; kc += SK) {
                double b[SK / 4];
#pragma unroll
                for (int kk = 0; kk < SK / 4; ++kk) b[kk] = rb[kk];
                if (kc + SK < K0) load_b(kc + SK);
#pragma unroll
                for (int kk = 0; kk < SK / 4; ++kk) {
                    const int kr = 4 * kk + (lane >> 4), ca = (lane & 15) ^ (4 * (kk & 3) + 2 * (lane >> 5));
#pragma unroll
                    for (int h = 0; h < KB; ++h) {
                        double a[4];
#pragma unroll
                        for (int m = 0; m < 4; ++m) a[m] = sA[buf][kr][16 * ((4 * h + m) ^ (kk >> 2)) + ca];
#pragma unroll
                        for (int m = 0; m < 4; ++m) acc[h][m] = Mma<double>::step(a[m], b[kk], acc[h][m]);
                    }
                }
                if (kc + SK < K0) {
                    store_a(buf ^ 1);
                    if (kc + 2 * SK < K0) load_a(kc + 2 * SK);
                }
                if ((kc + SK) % SFOLD == 0 || kc + SK == K0) {
#pragma unroll
                    for (int h = 0; h < KB; ++h)
#pragma unroll
                        for (int m = 0; m < 4; ++m) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) q[h][4 * m + r] += acc[h][m][r];
                            acc[h][m] = Mma<double>::zero();
                        }
                }
                buf ^= 1;
                __syncthreads();
            }
        }
        // ---- the panel's own triangle
        const double *Lt = Lp + K0, *Li = Linv + K0 * NB;
        Block64<kT> st;
        int rows = NB, buf = 0;
        bool neg = false;
        // the blocks in order of use: Linv_0, L_10, Linv_1
        auto fetch = [&](int k, int i) {  // block i == k: the inverse
            rows = i == k ? NB : min(nrow - 64 * i, NB);
            neg = i != k;
            if (i == k)
                st.load(Li + k * NB * NB, NB, NB, t);
            else
                st.load(Lt + 64 * i * ld + 64 * k, ld, rows, t);
        };
        fetch(0, 0);
        st.store(S[0], rows, neg, t);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KB; ++k) {
#pragma unroll
            for (int i = k; i < KB; ++i) {
                if (k >= nb || i >= nb) continue;
                const int kn = i + 1 < nb ? k : k + 1, in = i + 1 < nb ? i + 1 : k + 1;
                const bool more = kn < nb;
                if (more) fetch(kn, in);
                if (i == k) {
                    v4d acc[4];
#pragma unroll
                    for (int b = 0; b < 4; ++b) acc[b] = Mma<double>::zero();
#pragma unroll
                    for (int kk = 0; kk < 16; ++kk)
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            acc[b] = Mma<double>::step(oper(S[buf], b, kk, lane), q[k][kk], acc[b]);
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int r = 0; r < 4; ++r) q[k][4 * b + r] = acc[b][r];
                } else {
                    v4d acc[4];
#pragma unroll
                    for (int b = 0; b < 4; ++b) acc[b] = Mma<double>::zero();
#pragma unroll
                    for (int kk = 0; kk < 16; ++kk)
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            acc[b] = Mma<double>::step(oper(S[buf], b, kk, lane), q[k][kk], acc[b]);
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int r = 0; r < 4; ++r) q[i][4 * b + r] += acc[b][r];
                }
                if (more) st.store(S[buf ^ 1], rows, neg, t);
                buf ^= 1;
                __syncthreads();
            }
        }
        if (live) {
#pragma unroll
            for (int e = 0; e < 16 * KB; ++e, Qp += step)
                if (4 * e + (lane >> 4) < nrow) *Qp = q[e >> 4][e & 15];
        }
    }
}

}  // namespace

int form_B(int64_t naux, int64_t ncol, double* M, double* Q, int64_t ldQ, hipStream_t st) {
    // workspace: the flag and the 64 x 64 inverse of every diagonal block
    const int64_t nblk = cdiv(naux, NB);
    char* ws = nullptr;
    const size_t bytes = 256 + sizeof(double) * (size_t)(NB * NB * nblk);
    if (hipMalloc(&ws, bytes) != hipSuccess) {
        (void)hipGetLastError();
        set_error("dfjk_form_B: out of device memory");
        return DFJK_E_OOM;
    }
    int* flag = reinterpret_cast<int*>(ws);
    double* Linv_all = reinterpret_cast<double*>(ws + 256);
    int rc = DFJK_OK;
    if (hipMemsetAsync(flag, 0, sizeof(int), st) != hipSuccess) rc = DFJK_E_HIP;
    // Cholesky of M, in place
    for (int64_t k0 = 0; rc == DFJK_OK && k0 < naux; k0 += NB) {
        const int kb = (int)(naux - k0 < NB ? naux - k0 : NB);
        double* Linv = Linv_all + (k0 / NB) * NB * NB;
        chol_diag<<<1, kT, 0, st>>>(M, naux, k0, kb, Linv, flag);
        const int64_t n2 = naux - k0 - kb;  // kb = 64 when rows are left
        if (n2 > 0) {
            double* panel = M + (k0 + kb) * naux + k0;
            const int64_t nt = cdiv(n2, NB);
            chol_panel<<<dim3((unsigned)nt), kT, 0, st>>>(panel, naux, n2, Linv);
            chol_update<<<dim3((unsigned)(nt * (nt + 1) / 2)), kT, 0, st>>>(panel, M + (k0 + kb) * naux + k0 + kb,
                                                                            naux, n2);
        }
        if (hipGetLastError() != hipSuccess) rc = DFJK_E_HIP;
    }
    // strict upper triangle of M <- 0 (M holds L); rows in slabs of the grid's y limit
    for (int64_t i0 = 0; rc == DFJK_OK && i0 < naux; i0 += 32768) {
        const int64_t nr = naux - i0 < 32768 ? naux - i0 : 32768;
        zero_upper<<<dim3((unsigned)cdiv(naux, 256), (unsigned)nr), 256, 0, st>>>(M, naux, i0);
        if (hipGetLastError() != hipSuccess) rc = DFJK_E_HIP;
    }
    // forward substitution T = L^-1 Q, in place
    if (rc == DFJK_OK) {
        solve<<<dim3((unsigned)cdiv(ncol, 64)), kT, 0, st>>>(M, naux, Linv_all, Q, ldQ, ncol);
        if (hipGetLastError() != hipSuccess) rc = DFJK_E_HIP;
    }
    int host_flag = 0;
    if (rc == DFJK_OK &&
        (hipMemcpyAsync(&host_flag, flag, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess ||
         hipStreamSynchronize(st) != hipSuccess))
        rc = DFJK_E_HIP;
    (void)hipFree(ws);
    if (rc == DFJK_E_HIP) {
        set_error("dfjk_form_B: HIP error %s", hipGetErrorString(hipGetLastError()));
        return rc;
    }
    if (rc != DFJK_OK) return rc;
    if (host_flag) {
        set_error("dfjk_form_B: the metric is not positive definite (non-positive Cholesky pivot)");
        return DFJK_E_NONFINITE;
    }
    return DFJK_OK;
}

}  // namespace dfjk
