// Symmetric eigensolver for matrices that fit one CU's LDS (n <= kEigLdsN):
// two-sided cyclic Jacobi in the round-robin (tournament) order.
//
// A round rotates n/2 disjoint pairs.  Positions, not indices, are paired:
// pair k is (t_k, b_k) with t_k at position 2k and b_k at 2k + 1, and after
// each round every index moves to its next position, t_0 staying,
//   t_1 <- b_0,  t_k <- t_{k-1},  b_k <- b_{k+1},  b_{h-1} <- t_{h-1},
// so m - 1 rounds meet every pair once and bring the positions back (m = n
// rounded up to even; the extra index is a zero row).  The matrix is kept as
// the 2 x 2 blocks (pair k, pair kk), k <= kk, of its upper block triangle.
//
// What bounds it is the serial chain of (m - 1) x sweeps rounds, so a round is
// made short:
//   - a thread keeps the same blocks all along, and the positions its four
//     results go to are the same in every round: no index arithmetic;
//   - the rotations of the NEXT round are worked out by wavefronts of their
//     own while the others rotate the blocks: they need three blocks each (the
//     two diagonal blocks and the one holding the off-diagonal element of the
//     pair to come), rotated by this round's angles;
//   - with two copies of the matrix in LDS (h <= kEigDoubleH) a round needs one
//     barrier; larger matrices read, wait, write, wait;
//   - the eigenvectors do not take part: the rotations are logged and a second
//     kernel applies them, every column of V^T on a wavefront of its own.
// On MI355X, n = 128: 0.97 + 0.08 ms from the identity (about 0.95 us a round);
// averaged over the seven solutions of a six-iteration SCF, most of them
// started in the previous basis, 0.44 + 0.04 ms, against 2.36 ms for one
// workgroup that worked out indices, rotations and eigenvectors in turn.  The
// limit on n is LDS: one copy of 198 / 2 pairs' blocks is 158 KB.
#include "dense.h"

#include "numerics.h"

namespace dfjk {
namespace {

__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

constexpr int kEigThreads = 1024;
constexpr int kEigDoubleH = 69;  // pairs whose blocks fit LDS twice
constexpr int kEigLdsBytes = 160 * 1024 - 1024;  // dynamic LDS of the kernel at most (n = kEigLdsN: 161568)
constexpr double kEigTol = 1e-13;

// Next position of the index at position x (2k = t_k, 2k + 1 = b_k), h >= 2 pairs
__host__ __device__ inline int next_pos(int x, int h) {
    const int k = x >> 1;
    if ((x & 1) == 0) return k == 0 ? 0 : k < h - 1 ? x + 2 : x + 1;
    return k == 0 ? 2 : x - 2;
}
// Position whose index comes to position x
__host__ __device__ inline int prev_pos(int x, int h) {
    const int k = x >> 1;
    if ((x & 1) == 0) return k == 0 ? 0 : k == 1 ? 1 : x - 2;
    return k == h - 1 ? x - 1 : x + 2;
}
__host__ __device__ inline int blk_of(int k, int kk, int h) { return k * h - k * (k - 1) / 2 + (kk - k); }

// LDS place of the element (position i, position j): plane (row type, column
// type) and block, the block row first; the diagonal blocks keep (t, b) only
__host__ __device__ inline int place_of(int i, int j, int h, int nblk) {
    if ((i >> 1) > (j >> 1) || ((i >> 1) == (j >> 1) && i > j)) {
        const int t = i;
        i = j;
        j = t;
    }
    return ((i & 1) * 2 + (j & 1)) * nblk + blk_of(i >> 1, j >> 1, h);
}

// 1 / sqrt(x) and 1 / x to the last places for normal x well inside the range: the
// hardware's start (relative error below 2^-23) and one third-order step.  The residual
// 1 - x y^2 takes the rounding of x y along: without it the cosines were off to one
// side, and the norms of the vectors, which gather that over a thousand rotations,
// drifted: mean of |v|^2 - 1 at n=198 4.7e-14, with correctly rounded roots and
// divisions 3.2e-14, so -6e-16.
__device__ inline double rsqrt_near(double x) {
    const double y = __builtin_amdgcn_rsq(x), p = x * y;
    const double e = fma(-fma(x, y, -p), y, fma(-p, y, 1.0));
    return fma(y * e, fma(0.375, e, 0.5), y);
}
__device__ inline double rcp_near(double x) {
    const double y = __builtin_amdgcn_rcp(x), e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// Symmetric Schur rotation of (app, apq; apq, aqq) (Golub & Van Loan, 8.5.2).  It is
// the longest part of a round's chain, so with h = aqq - app and g = 2 apq the
// tangent is sign(h) g / (|h| + sqrt(h^2 + g^2)) by a reciprocal and two reciprocal
// roots: 16 molecules of 40 to 160 functions 1.02 ms a solution, 1.18 with three
// divisions and two square roots (at n = 128, where the blocks' LDS traffic of 200 KB a
// round bounds it, the same).  Differences whose squares would leave the range keep
// those.
__device__ inline void schur(double app, double apq, double aqq, double& c, double& s) {
    c = 1.0;
    s = 0.0;
    const double h = aqq - app, g = 2.0 * apq, m = fmax(fabs(h), fabs(g));
    if (__builtin_expect(m > 1e-140 && m < 1e140, 1)) {
        const double x = fma(h, h, g * g);
        const double d = fma(x, rsqrt_near(x), fabs(h));
        const double t = (h >= 0.0 ? g : -g) * rcp_near(d);
        c = rsqrt_near(fma(t, t, 1.0));
        s = t * c;
    } else if (apq != 0.0) {
        const double tau = h / g;
        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
        c = 1.0 / sqrt(1.0 + t * t);
        s = t * c;
    }
}

// (p, q) <- (c p - s q, s p + c q)
__device__ inline void rot(double c, double s, double& p, double& q) {
    const double x = c * p - s * q, y = s * p + c * q;
    p = x;
    q = y;
}

// One column of V^T through `rounds` logged rounds, on one wavefront: lane l
// holds the pairs R l .. R l + R - 1 of positions (xt, xb).
// U: rounds of rotations loaded ahead.
template <int R, int U>
__device__ inline void apply_rounds(const double2* __restrict__ log, int rounds, int h, double (&xt)[R],
                                    double (&xb)[R]) {
    const int lane = threadIdx.x & 63;
    auto up = [](double v) {  // value of the lane below
        const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xf, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xf, 0xf, false);
        return __hiloint2double(hi, lo);
    };
    auto down = [](double v) {  // value of the lane above
        const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xf, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130, 0xf, 0xf, false);
        return __hiloint2double(hi, lo);
    };
    double2 cs[U][R];
    auto load = [&](int r, double2 (&v)[R]) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int k = lane * R + q;
            v[q] = r < rounds && k < h ? log[(int64_t)r * h + k] : make_double2(1.0, 0.0);
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load(u, cs[u]);
    for (int r0 = 0; r0 < rounds; r0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r0 + u >= rounds) break;
            double last[R];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                rot(cs[u][q].x, cs[u][q].y, xt[q], xb[q]);
                last[q] = xt[q];
            }
            load(r0 + u + U, cs[u]);
            if (h == 1) continue;  // one pair: nothing moves
            const double t0 = xt[0];
            if (lane == 0) xt[0] = xb[0];  // b_0 moves to t_1
            const double in_t = up(xt[R - 1]), in_b = down(xb[0]);
#pragma unroll
            for (int q = R - 1; q > 0; --q) xt[q] = xt[q - 1];
            xt[0] = lane == 0 ? t0 : in_t;
#pragma unroll
            for (int q = 0; q + 1 < R; ++q) xb[q] = xb[q + 1];
            xb[R - 1] = in_b;
#pragma unroll
            for (int q = 0; q < R; ++q)
                if (lane * R + q == h - 1) xb[q] = last[q];  // t_{h-1} becomes b_{h-1}
        }
    }
}

template <int R>
__device__ inline void load_column(const double* __restrict__ V, bool identity, int n, int j, double (&xt)[R],
                                   double (&xb)[R]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = 2 * (lane * R + q);
        xt[q] = i < n ? (identity ? (i == j ? 1.0 : 0.0) : V[(int64_t)i * n + j]) : 0.0;
        xb[q] = i + 1 < n ? (identity ? (i + 1 == j ? 1.0 : 0.0) : V[(int64_t)(i + 1) * n + j]) : 0.0;
    }
}

template <int R>
__device__ inline void store_column(double* __restrict__ V, int n, int j, const double (&xt)[R],
                                    const double (&xb)[R]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = 2 * (lane * R + q);
        if (i < n) V[(int64_t)i * n + j] = xt[q];
        if (i + 1 < n) V[(int64_t)(i + 1) * n + j] = xb[q];
    }
}

// Eigenvalues of (X + X^T) / 2 (in ascending order in w, ties by index) and
// the log of rotations.  NB blocks per thread; DB: two copies of the matrix in
// LDS.
template <int NB, bool DB>
__device__ __forceinline__ void jacobi_solve(const double* __restrict__ X, int n, double2* __restrict__ log,
                                    int* __restrict__ iwork, double* __restrict__ w, char* smem,
                                    double (&red)[2][kEigThreads / 64]) {
    const int m = n + (n & 1), h = m / 2, nblk = h * (h + 1) / 2;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int na = 64 * (int)cdiv(h, 64);  // threads of the rotation wavefronts
    double2* cs = reinterpret_cast<double2*>(smem);  // [2][h]
    double* Abuf[2];
    Abuf[0] = reinterpret_cast<double*>(smem + 2 * h * sizeof(double2));
    Abuf[1] = DB ? Abuf[0] + 4 * nblk : Abuf[0];

    auto elem = [&](int i, int j) {
        return i < n && j < n ? 0.5 * (X[(int64_t)i * n + j] + X[(int64_t)j * n + i]) : 0.0;
    };
    auto self = [&](int j) { return tid - na + j * (nthr - na); };
    // blocks of this thread (negative: none) and where their results go
    int kk2[NB];  // k | kk << 16
    uint32_t to[NB][2];
    uint32_t top = 0;  // of the largest entry
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int b = self(j);
        kk2[j] = -1;
        if (tid >= na && b < nblk) {
            int k = 0, at = 0;
            while (at + (h - k) <= b) at += h - k++;
            const int kk = k + (b - at);
            kk2[j] = k | (kk << 16);
            uint32_t p[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 2 * k + (e >> 1), q = 2 * kk + (e & 1);
                p[e] = h > 1 ? (uint32_t)place_of(next_pos(i, h), next_pos(q, h), h, nblk) : (uint32_t)(e * nblk + b);
                const double x = elem(i, q);
                top = max(top, top_bits(x));
                Abuf[0][e * nblk + b] = x;
            }
            to[j][0] = p[0] | (p[1] << 16);
            to[j][1] = p[2] | (p[3] << 16);
        }
    }
    auto on_diag = [&](int j) { return (kk2[j] & 0xffff) == (kk2[j] >> 16); };
    // sources of the next round's pair of a rotation thread: positions u and v
    const int ak = tid < h ? tid : h - 1;
    const int u = h > 1 ? prev_pos(2 * ak, h) : 0, v = h > 1 ? prev_pos(2 * ak + 1, h) : 1;
    const int ku = u >> 1, kv = v >> 1;
    const int lo = ku < kv ? ku : kv, hi = ku < kv ? kv : ku;
    const int bu = blk_of(ku, ku, h), bv = blk_of(kv, kv, h), bx = blk_of(lo, hi, h);
    const bool rot_thread = tid < h;
    top = wave_max(top);
    if ((tid & 63) == 0) red[0][tid >> 6] = (double)top;
    __syncthreads();
    double topd = 0.0;
    for (int q = 0; q < nthr / 64; ++q) topd = fmax(topd, red[0][q]);
    const bool finite = topd < (double)kNotFinite;  // else there is nothing to solve: no sweep, NaN results
    const int ex = eig_exponent((uint32_t)topd);
    if (ex != 0) {  // scaled by 2^-ex: exact
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (kk2[j] >= 0)
#pragma unroll
                for (int e = 0; e < 4; ++e) Abuf[0][e * nblk + self(j)] *= pow2(-ex);
        __syncthreads();
    }
    double c = 1.0, s = 0.0;  // rotation thread: the rotation of the round to come
    if (rot_thread) {
        const int b = blk_of(ak, ak, h);
        const double* A = Abuf[0];
        schur(A[b], A[nblk + b], A[3 * nblk + b], c, s);
        cs[ak] = make_double2(c, s);
    }
    int cur = 0, par = 0, sweep = 0, logged = 0;
    __syncthreads();
    for (; finite && sweep < kEigMaxSweeps; ++sweep) {
        // off-diagonal norm against the full norm
        double off = 0.0, dia = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (kk2[j] >= 0) {
                const double* A = Abuf[cur] + self(j);
                const double x0 = A[0], x1 = A[nblk], x3 = A[3 * nblk];
                if (on_diag(j)) {
                    off = fma(2.0 * x1, x1, off);
                    dia = fma(x0, x0, fma(x3, x3, dia));
                } else {
                    const double x2 = A[2 * nblk];
                    off += 2.0 * (fma(x0, x0, x1 * x1) + fma(x2, x2, x3 * x3));
                }
            }
        off = wave_sum(off);
        dia = wave_sum(dia);
        if ((tid & 63) == 0) {
            red[0][tid >> 6] = off;
            red[1][tid >> 6] = dia;
        }
        __syncthreads();
        off = dia = 0.0;
        for (int q = 0; q < nthr / 64; ++q) {
            off += red[0][q];
            dia += red[1][q];
        }
        if (!(off > kEigTol * kEigTol * (off + dia))) break;
        for (int r = 0; r < m - 1; ++r, par ^= 1, ++logged) {
            const double* A = Abuf[cur];
            const double2* csr = cs + par * h;
            double x[NB][4];
            if (tid >= na) {
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    if (kk2[j] >= 0) {
                        const double* a = A + self(j);
                        x[j][0] = a[0], x[j][1] = a[nblk], x[j][3] = a[3 * nblk];
                        const bool diag = on_diag(j);
                        x[j][2] = diag ? x[j][1] : a[2 * nblk];
                        const double2 p = csr[kk2[j] & 0xffff], q = csr[kk2[j] >> 16];
                        rot(p.x, p.y, x[j][0], x[j][2]);  // rows t, b of the block
                        rot(p.x, p.y, x[j][1], x[j][3]);
                        rot(q.x, q.y, x[j][0], x[j][1]);  // columns
                        rot(q.x, q.y, x[j][2], x[j][3]);
                        if (diag) x[j][1] = x[j][2] = 0.0;  // by construction of the rotation
                    }
            } else if (rot_thread) {
                log[(int64_t)logged * h + ak] = make_double2(c, s);
                if (h > 1) {
                    const double2 p = csr[ku], q = csr[kv];
                    double d0 = A[bu], d1 = A[nblk + bu], d2 = d1, d3 = A[3 * nblk + bu];
                    rot(p.x, p.y, d0, d2);
                    rot(p.x, p.y, d1, d3);
                    rot(p.x, p.y, d0, d1);
                    rot(p.x, p.y, d2, d3);
                    const double app = (u & 1) ? d3 : d0;
                    d0 = A[bv], d1 = d2 = A[nblk + bv], d3 = A[3 * nblk + bv];
                    rot(q.x, q.y, d0, d2);
                    rot(q.x, q.y, d1, d3);
                    rot(q.x, q.y, d0, d1);
                    rot(q.x, q.y, d2, d3);
                    const double aqq = (v & 1) ? d3 : d0;
                    // element (u, v): block (lo, hi), rows of pair lo
                    const double2 pl = ku < kv ? p : q, ph = ku < kv ? q : p;
                    const int rl = ku < kv ? u : v, ch = ku < kv ? v : u;
                    double e0 = A[bx], e1 = A[nblk + bx], e2 = A[2 * nblk + bx], e3 = A[3 * nblk + bx];
                    rot(pl.x, pl.y, e0, e2);
                    rot(pl.x, pl.y, e1, e3);
                    rot(ph.x, ph.y, e0, e1);
                    rot(ph.x, ph.y, e2, e3);
                    const double apq = (rl & 1) ? ((ch & 1) ? e3 : e2) : ((ch & 1) ? e1 : e0);
                    schur(app, apq, aqq, c, s);
                } else {
                    c = 1.0;
                    s = 0.0;
                }
                cs[(par ^ 1) * h + ak] = make_double2(c, s);
            }
            if (!DB) __syncthreads();
            if (tid >= na) {
                double* B = Abuf[DB ? cur ^ 1 : 0];
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    if (kk2[j] >= 0) {
                        B[to[j][0] & 0xffffu] = x[j][0];
                        B[to[j][0] >> 16] = x[j][1];
                        if (!on_diag(j)) B[to[j][1] & 0xffffu] = x[j][2];
                        B[to[j][1] >> 16] = x[j][3];
                    }
            }
            __syncthreads();
            if (DB) cur ^= 1;
        }
    }
    // ascending order of the diagonal (ties by index); where it has none, the index
    __syncthreads();
    double* dg = reinterpret_cast<double*>(smem);  // overwrites cs, not the blocks
    double di = 0.0;
    if (tid < n) {
        const int b = blk_of(tid >> 1, tid >> 1, h);
        di = Abuf[cur][((tid & 1) ? 3 : 0) * nblk + b];
        dg[tid] = di;
    }
    __syncthreads();
    if (tid < n) {
        int rank = 0;
        for (int j = 0; j < n; ++j) rank += (dg[j] < di || (dg[j] == di && j < tid)) ? 1 : 0;
        if (!finite) {
            rank = tid;
            di = __builtin_nan("");
        }
        iwork[EigWork::rank_at(n) + tid] = rank;
        w[rank] = di * pow2(ex);
    }
    if (tid == 0) {
        iwork[0] = sweep;
        iwork[EigWork::rounds_at(n)] = finite ? logged : -1;
    }
}

template <int NB, bool DB>
__global__ __launch_bounds__(kEigThreads) void jacobi_lds(const double* __restrict__ X, int n,
                                                          double2* __restrict__ log, int* __restrict__ iwork,
                                                          double* __restrict__ w) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ double red[2][kEigThreads / 64];
    jacobi_solve<NB, DB>(X, n, log, iwork, w, smem, red);
}

// V^T <- J^T V^T with the logged rotations, one column per wavefront, and the
// ncol lowest eigenvectors as columns of out (mode 1: scaled by sqrt|w|, the
// signs of w to sign).
template <int R>
__device__ __forceinline__ void apply_log(const double2* __restrict__ log, const int* __restrict__ iwork, int n,
                                 int v_identity, double* __restrict__ V, const double* __restrict__ w, int ncol,
                                 int mode, double* __restrict__ out, double* __restrict__ sign) {
    const int col = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (col >= n) return;
    const int h = (n + 1) / 2;
    double xt[R], xb[R];
    load_column<R>(V, v_identity != 0, n, col, xt, xb);
    const int rounds = iwork[EigWork::rounds_at(n)];  // negative: no eigenvectors
    apply_rounds<R, 8>(log, rounds, h, xt, xb);
    store_column<R>(V, n, col, xt, xb);
#pragma unroll
    for (int q = 0; q < 2 * R; ++q) {
        const int i = 2 * (lane * R + (q >> 1)) + (q & 1);
        if (i >= n) continue;
        const int c = iwork[EigWork::rank_at(n) + i];
        if (c >= ncol) continue;
        const double x = (q & 1) ? xb[q >> 1] : xt[q >> 1];
        const double f = rounds < 0 ? __builtin_nan("") : mode == 1 ? sqrt(fabs(w[c])) : 1.0;
        out[(int64_t)col * ncol + c] = f * x;
        if (sign && col == 0) sign[c] = w[c] < 0.0 ? -1.0 : 1.0;
    }
}

template <int R>
__global__ __launch_bounds__(256) void jacobi_apply(const double2* __restrict__ log, const int* __restrict__ iwork,
                                                    int n, int v_identity, double* __restrict__ V,
                                                    const double* __restrict__ w, int ncol, int mode,
                                                    double* __restrict__ out, double* __restrict__ sign) {
    apply_log<R>(log, iwork, n, v_identity, V, w, ncol, mode, out, sign);
}

// The forms of jacobi_lds: one block per thread while the blocks fit a workgroup
// (fewer wavefronts to wait for), else three with two copies of the matrix in LDS, else six with one.
struct EigForm {
    int h, nblk, na, nb, threads;
    size_t lds;
    __host__ __device__ explicit EigForm(int n) {
        h = (n + 1) / 2;
        nblk = h * (h + 1) / 2;
        na = 64 * (int)cdiv(h, 64);
        const bool db = h <= kEigDoubleH;
        nb = nblk <= kEigThreads - na ? 1 : db ? 3 : 6;
        threads = nb == 1 ? na + 64 * (int)cdiv(nblk, 64) : kEigThreads;
        lds = 2 * sizeof(double2) * (size_t)h + (db ? 2 : 1) * 4 * sizeof(double) * (size_t)nblk;
    }
};

// One workgroup per molecule
__global__ __launch_bounds__(kEigThreads) void jacobi_many(const ScfMol* __restrict__ mols, MolPtrs X, int given) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ double red[2][kEigThreads / 64];
    const ScfMol& d = mols[blockIdx.x];
    const int n = d.n, nb = EigForm(n).nb;
    const double* x = as_global(given ? X.p[blockIdx.x] : d.Fx);
    double2* log = as_global(reinterpret_cast<double2*>(d.eig.log));
    int* iwork = as_global(d.eig.iwork);
    double* w = as_global(d.eig.w);
    if (nb == 1)
        jacobi_solve<1, true>(x, n, log, iwork, w, smem, red);
    else if (nb == 3)
        jacobi_solve<3, true>(x, n, log, iwork, w, smem, red);
    else
        jacobi_solve<6, false>(x, n, log, iwork, w, smem, red);
}

__global__ __launch_bounds__(256) void jacobi_apply_many(const ScfMol* __restrict__ mols, int v_identity) {
    const ScfMol& d = mols[blockIdx.y];
    const double2* log = as_global(reinterpret_cast<const double2*>(d.eig.log));
    const int* iwork = as_global(d.eig.iwork);
    if (d.n <= 128)
        apply_log<1>(log, iwork, d.n, v_identity, as_global(d.V), d.eig.w, d.nocc, 0, as_global(d.C), nullptr);
    else
        apply_log<2>(log, iwork, d.n, v_identity, as_global(d.V), d.eig.w, d.nocc, 0, as_global(d.C), nullptr);
}

}  // namespace

int eig_lds(hipStream_t st, const double* X, double* V, int n, bool v_identity, const EigWork& ws, int ncol,
            int mode, double* out, double* sign) {
    const EigForm f(n);
    double2* log = reinterpret_cast<double2*>(ws.log);
    auto launch = [&](auto kernel) -> int {
        // above 64 KB of dynamic LDS a kernel has to be told so
        DFJK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, kEigLdsBytes));
        kernel<<<1, f.threads, f.lds, st>>>(X, n, log, ws.iwork, ws.w);
        DFJK_LAUNCH_CHECK("jacobi_lds");
        return DFJK_OK;
    };
    int rc = f.nb == 1 ? launch(jacobi_lds<1, true>) : f.nb == 3 ? launch(jacobi_lds<3, true>) : launch(jacobi_lds<6, false>);
    if (rc) return rc;
    const dim3 grid((unsigned)cdiv(n, 4));
    if (f.h <= 64)
        jacobi_apply<1><<<grid, 256, 0, st>>>(log, ws.iwork, n, v_identity ? 1 : 0, V, ws.w, ncol, mode, out, sign);
    else
        jacobi_apply<2><<<grid, 256, 0, st>>>(log, ws.iwork, n, v_identity ? 1 : 0, V, ws.w, ncol, mode, out, sign);
    DFJK_LAUNCH_CHECK("jacobi_apply");
    return DFJK_OK;
}

int eig_lds_many(hipStream_t st, const ScfMol* mols, const MolPtrs* X, bool v_identity, int nmol, int max_n,
                 int lds_n) {
    // one launch holds all sizes, so its LDS is the most any of them takes (at lds_n)
    DFJK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(jacobi_many),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kEigLdsBytes));
    const MolPtrs none{};
    jacobi_many<<<(unsigned)nmol, EigForm(max_n).threads, EigForm(lds_n).lds, st>>>(mols, X ? *X : none, X ? 1 : 0);
    DFJK_LAUNCH_CHECK("jacobi_many");
    jacobi_apply_many<<<dim3((unsigned)cdiv(max_n, 4), (unsigned)nmol), 256, 0, st>>>(mols, v_identity ? 1 : 0);
    DFJK_LAUNCH_CHECK("jacobi_apply_many");
    return DFJK_OK;
}

size_t eig_lds_bytes(int n) { return EigForm(n).lds; }

}  // namespace dfjk
