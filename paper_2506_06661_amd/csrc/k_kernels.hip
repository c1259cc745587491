// Exchange matrix K on the matrix cores (FP64 MFMA, v_mfma_f64_16x16x4f64).
//
// For a factor C (nao x ncol) with column signs s_i and a scale a:
//   X_P = B_P C                                  (GEMM1, per auxiliary index P)
//   K   = a * sum_P sum_i s_i X_P[:,i] X_P[:,i]^T (GEMM2, a SYRK over (P,i))
// a = 2, s = +1 gives K for D = 2 C C^T (Eq. eq:df:eri contracted twice with
// the occupied orbitals).
//
// GEMM1 computes the transposed product X_P^T = C^T B_P so that each output
// row (P,i) is contiguous in mu; X is stored as rows k = P*ncol + i of length
// ldx.  B_P is read straight from the packed triangle: a 16 x 128 (nu, mu)
// chunk that lies wholly above or below the diagonal is a set of contiguous
// runs of one packed row, and is loaded along those runs.
//
// GEMM2 accumulates only the lower block triangle of K in 128 x 128 tiles,
// with the (P,i) contraction split over workgroups; each split writes its
// own partial tile, and a last kernel adds the splits in a fixed order and
// mirrors the result, so K is bitwise reproducible.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "mma.h"

namespace dfjk {

namespace {

constexpr int kThreads = 256;
constexpr int KC = 16;      // contraction chunk held in LDS
constexpr int SY_T = 128;   // SYRK output tile
constexpr int64_t kMaxSum32 = 16384;  // longest FP32 running sum in the SYRK

__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Storage element of B -> compute type (exact for every pair used here).
template <typename T, typename TS>
__device__ inline T to_compute(TS x) {
    return (T)x;
}
template <>
__device__ inline float to_compute<float, uint16_t>(uint16_t x) {  // bfloat16 bits
    return __uint_as_float((uint32_t)x << 16);
}
template <>
__device__ inline float to_compute<float, _Float16>(_Float16 x) {
    return (float)x;
}

// Keeps a branch that is rarely taken a branch: without it the compiler turns
// the zeroing of a last, partial chunk into selects on every chunk.
__device__ inline void rare_path() { asm volatile("" ::: "memory"); }

// ---------------------------------------------------------------- GEMM1
// Workgroup tile: BI = 16*NI rows i (all waves) x BM = 64*WM columns mu
// (each of the 4 waves owns 16*WM columns).  Per 16-deep nu chunk each thread
// stages 16 bytes of C per load (VC orbitals of a row) and up to 16 bytes of
// B_P (VB consecutive elements of a packed row: along nu below the diagonal,
// along mu above it; the GPU's global loads take unaligned addresses) in
// registers, then LDS.
//
// The products of a chunk keep the matrix cores busy for 64 (FP64) or 32 (FP32)
// cycles a step, so what costs is the vector work around them: an FP64 (7,1)
// chunk is 1792 cycles of products, and 64-bit addresses, bounds and selects of
// every element took longer than that.  So every address is a uniform base that
// advances in scalar registers plus a 32-bit thread offset that stays the same
// (C, and B below the diagonal) or takes one multiply-add (B above it: packed
// row T(nu0 + k) = T(nu0) + k nu0 + k(k+1)/2).  Columns past the operands are
// clamped to valid ones (their products are never stored); rows nu past nao are
// zeroed, in the last chunk only.  A chunk's loads are issued when the chunk
// before it has been stored to LDS, a whole chunk of products before they are
// used.  nao=1024, naux=4096, nocc=200, FP64: 35.1 -> 31.6 ms (matrix cores 74-79%
// busy at 2.2 GHz; the chip is at its power limit); nao=701, FP32: 5.37 -> 4.57.
template <typename T, typename TS, int NI, int WM>
struct G1 {
    static constexpr int VC = 16 / sizeof(T);     // orbitals per load
    static constexpr int VPR = 16 * NI / VC;      // loads per row of the C tile
    static constexpr int NV = KC * VPR;           // loads per chunk
    static constexpr int NC = (NV + kThreads - 1) / kThreads;  // per thread
    static constexpr int VB = 4 * WM < (int)(16 / sizeof(TS)) ? 4 * WM : (int)(16 / sizeof(TS));  // B elements per load
    static constexpr int NP = 4 * WM / VB;        // loads per thread per chunk
    static constexpr int TLO = KC / VB;           // below: threads per packed row mu
    static constexpr int RLO = kThreads / TLO;    // below: rows mu per pass
    static constexpr int TUP = 64 * WM / VB;      // above: threads per packed row nu
    static constexpr int RUP = kThreads / TUP;    // above: rows nu per pass
    // LDS rows are nu; an operand read covers 16 consecutive columns of 4 rows.
    // FP32: row pitches of 16 or 48 modulo 64 words put the four rows on
    // disjoint banks; FP64 (two rows per 256 bytes): 16 modulo 32 elements.
    static constexpr int G = sizeof(T) == 4 ? 64 : 32;
    static constexpr int PC = (16 * NI) % G % 32 == 16 ? 16 * NI : 16 * NI + 16;
    static constexpr int PB = 64 * WM + 16;
    // B below the diagonal is written transposed (VB rows from one thread), so
    // row k keeps column m at m ^ swz(k): the rows one store covers fall on
    // different banks.  FP32 moves whole groups of 16 columns (k / 4 is the
    // step number of a read); FP64 permutes pairs inside a group.
    __device__ static int swz(int k) { return sizeof(T) == 4 ? 16 * ((k >> 2) & 3) : 2 * ((k >> 1) & 7); }

    T c[NC][VC];
    TS b[NP][VB];
    uint32_t coff[NC];   // C: k * ldc + column
    uint32_t loff[NP];   // B below: T(mu) - T(mu0) + k
    uint32_t ucon[NP];   // B above: k(k+1)/2 + column
    int phase;           // of the chunk in b: 0 below, 1 crossing, 2 above the diagonal
    int klive;           // rows of the chunk below nao

    __device__ inline void init(int nao, int ldc, int mu0, int i0, int tid) {
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int e = tid + j * kThreads;
            const int k = e < NV ? e / VPR : 0, ii = (e % VPR) * VC;
            coff[j] = (uint32_t)(k * ldc + min(i0 + ii, ldc - VC));
        }
        const uint32_t t0 = (uint32_t)mu0 * (uint32_t)(mu0 + 1) / 2;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const uint32_t mu = (uint32_t)min(mu0 + tid / TLO + RLO * j, nao - 1);
            loff[j] = mu * (mu + 1) / 2 - t0 + (tid % TLO) * VB;
            const int k = tid / TUP + RUP * j;
            ucon[j] = (uint32_t)(k * (k + 1) / 2 + (tid % TUP) * VB);
        }
    }

    // chunk of rows nu0 .. nu0 + 15 (Cn: row nu0 of C)
    __device__ inline void load(const TS* __restrict__ Bp, const T* __restrict__ Cn, int nao, int ldc, int nu0,
                                int mu0, int tid) {
        klive = min(nao - nu0, KC);
        if (__builtin_expect(klive < KC, 0)) {
            rare_path();
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const int e = tid + j * kThreads, k = e < NV ? e / VPR : 0;  // as coff
                __builtin_memcpy(c[j], Cn + (coff[j] - (uint32_t)(max(k - klive + 1, 0) * ldc)), VC * sizeof(T));
            }
        } else {
#pragma unroll
            for (int j = 0; j < NC; ++j) __builtin_memcpy(c[j], Cn + coff[j], VC * sizeof(T));
        }
        phase = nu0 + KC <= mu0 ? 0 : nu0 < mu0 + 64 * WM ? 1 : 2;
        if (phase == 0) {
            // every nu < mu: packed row mu, columns nu0 .. nu0+15
            const TS* base = Bp + ((int64_t)mu0 * (mu0 + 1) / 2 + nu0);
#pragma unroll
            for (int j = 0; j < NP; ++j) __builtin_memcpy(b[j], base + loff[j], VB * sizeof(TS));
        } else if (phase == 2) {
            // every nu > mu: packed row nu, columns mu0 .. mu0+BM-1
            const TS* base = Bp + ((int64_t)nu0 * (nu0 + 1) / 2 + mu0);
            if (__builtin_expect(klive < KC, 0)) {
                rare_path();
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const int k = min(tid / TUP + RUP * j, klive - 1);
                    const uint32_t off = (uint32_t)(k * nu0 + k * (k + 1) / 2 + (tid % TUP) * VB);
                    __builtin_memcpy(b[j], base + off, VB * sizeof(TS));
                }
            } else {
#pragma unroll
                for (int j = 0; j < NP; ++j)
                    __builtin_memcpy(b[j], base + ((uint32_t)(tid / TUP + RUP * j) * (uint32_t)nu0 + ucon[j]),
                                     VB * sizeof(TS));
            }
        } else {
            // chunk crossing the diagonal (rows as above it, element loads)
            const TS* base = Bp + (int64_t)mu0 * (mu0 + 1) / 2;
            const int dnu = nu0 - mu0, dmax = nao - 1 - mu0;
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int k0 = tid / TUP + RUP * j;
#pragma unroll
                for (int q = 0; q < VB; ++q) {
                    // offsets from mu0: row hi, T(mu0 + hi) - T(mu0) = hi mu0 + hi(hi+1)/2
                    const int dm = min((tid % TUP) * VB + q, dmax), dn = min(dnu + k0, dmax);
                    const int hi = max(dm, dn), lo = min(dm, dn);
                    b[j][q] = base[(uint32_t)(hi * mu0 + hi * (hi + 1) / 2 + mu0 + lo)];
                }
            }
        }
    }

    // The loaded values are first looked at here, a chunk of products after
    // their loads were issued: zeroing the rows past nao while loading made the
    // wavefront wait for the loads before those products.
    __device__ inline void store(T (*sC)[PC], T (*sB)[PB], int tid) {
        if (__builtin_expect(klive < KC, 0)) {
            rare_path();
#pragma unroll
            for (int j = 0; j < NC; ++j)
#pragma unroll
                for (int q = 0; q < VC; ++q)
                    if ((tid + j * kThreads) / VPR >= klive) c[j][q] = T(0);
#pragma unroll
            for (int j = 0; j < NP; ++j)
#pragma unroll
                for (int q = 0; q < VB; ++q)
                    if (tid / TUP + RUP * j >= klive) b[j][q] = TS(0);
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int e = tid + j * kThreads;
            if (NV % kThreads == 0 || e < NV) __builtin_memcpy(&sC[e / VPR][(e % VPR) * VC], c[j], VC * sizeof(T));
        }
        if (phase == 0) {
            // element q of load j: row (tid % TLO) * VB + q, column mu
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int m = tid / TLO + RLO * j;
#pragma unroll
                for (int q = 0; q < VB; ++q) {
                    const int r = (tid % TLO) * VB + q;
                    sB[r][m ^ swz(r)] = to_compute<T, TS>(b[j][q]);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int r = tid / TUP + RUP * j, m = (tid % TUP) * VB;
                T v[VB];
#pragma unroll
                for (int q = 0; q < VB; ++q) v[q] = to_compute<T, TS>(b[j][q]);
                __builtin_memcpy(&sB[r][m ^ swz(r)], v, VB * sizeof(T));
            }
        }
    }
};

// Block order: consecutive hardware block ids go round-robin to the 8 XCDs.
// Renumber so that runs of consecutive logical ids share an XCD (and its L2):
// the i-blocks and mu-blocks of one P then read B_P through one L2.
__device__ inline int64_t xcd_logical(int64_t hw, int64_t nblk) {
    constexpr int64_t NX = 8;
    const int64_t per = nblk / NX, rem = nblk % NX;
    const int64_t x = hw % NX, q = hw / NX;
    // XCD x holds logical ids [x*per + min(x, rem), ...) ; blocks past per*NX keep their order
    if (q < per) return x * per + (x < rem ? x : rem) + q;
    return x * per + (x < rem ? x : rem) + per;  // only the first rem XCDs get one more block
}

// X[(P*ncol + i)*ldx + mu] = sum_nu C[nu][i] B_P[nu][mu]
// 1-D grid of nib * nmb * naux blocks; logical id -> (i block fastest, mu block, P)
// ldc is a multiple of VC.
template <typename T, typename TS, int NI, int WM>
__device__ __attribute__((always_inline)) inline void k_gemm1_body(int64_t lid, const TS* __restrict__ B, int64_t ldB, int64_t nao,
                                    const T* __restrict__ C, int64_t ldc, int64_t ncol,
                                    T* __restrict__ X, int64_t ldx, int64_t nib, int64_t nmb) {
    using S = G1<T, TS, NI, WM>;
    constexpr int BI = 16 * NI, BM = 64 * WM;
    __shared__ __attribute__((aligned(16))) T sC[2][KC][S::PC];
    __shared__ __attribute__((aligned(16))) T sB[2][KC][S::PB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t ib = lid % nib, mb = (lid / nib) % nmb, P = lid / (nib * nmb);
    const int64_t i0 = ib * BI, mu0 = mb * BM;
    const TS* Bp = B + P * ldB;

    typename Mma<T>::acc_t acc[NI][WM];
#pragma unroll
    for (int a = 0; a < NI; ++a)
#pragma unroll
        for (int b = 0; b < WM; ++b) acc[a][b] = Mma<T>::zero();

    // operand columns of this lane before the row's swizzle
    const int ca = lane & 15, cb = wave * 16 * WM + ((lane & 15) ^ (sizeof(T) == 8 ? 2 * (lane >> 5) : 0));
    S st;
    const int nao_ = (int)nao, ldc_ = (int)ldc, mu0_ = (int)mu0;
    st.init(nao_, ldc_, mu0_, (int)i0, tid);
    const T* Cn = C;
    st.load(Bp, Cn, nao_, ldc_, 0, mu0_, tid);
    st.store(sC[0], sB[0], tid);
    if (KC < nao_) st.load(Bp, Cn += KC * ldc, nao_, ldc_, KC, mu0_, tid);
    __syncthreads();
    int buf = 0;
    for (int nu0 = 0; nu0 < nao_; nu0 += KC, buf ^= 1) {
#pragma unroll
        for (int kk = 0; kk < KC / 4; ++kk) {
            const int kr = kk * 4 + (lane >> 4);
            T a[NI], b[WM];
#pragma unroll
            for (int t = 0; t < NI; ++t) a[t] = sC[buf][kr][t * 16 + ca];
#pragma unroll
            for (int t = 0; t < WM; ++t)
                b[t] = sB[buf][kr][sizeof(T) == 8 ? t * 16 + (cb ^ (4 * kk)) : (t * 16 + cb) ^ (16 * kk)];
#pragma unroll
            for (int ti = 0; ti < NI; ++ti)
#pragma unroll
                for (int tj = 0; tj < WM; ++tj) acc[ti][tj] = Mma<T>::step(a[ti], b[tj], acc[ti][tj]);
        }
        if (nu0 + KC < nao_) {
            st.store(sC[buf ^ 1], sB[buf ^ 1], tid);
            if (nu0 + 2 * KC < nao_) st.load(Bp, Cn += KC * ldc, nao_, ldc_, nu0 + 2 * KC, mu0_, tid);
        }
        __syncthreads();
    }
    T* Xp = X + (P * ncol + i0) * ldx + mu0;
#pragma unroll
    for (int tj = 0; tj < WM; ++tj) {
        const int m = wave * 16 * WM + tj * 16 + (lane & 15);
        if (mu0 + m >= nao) continue;
#pragma unroll
        for (int ti = 0; ti < NI; ++ti)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = ti * 16 + Mma<T>::row(lane, r);
                if (i0 + i < ncol) Xp[(int64_t)i * ldx + m] = acc[ti][tj][r];
            }
    }
}

// FP32 form on v_mfma_f32_32x32x2f32 (4096 flop per step; lane l supplies
// A[l%32][l/32] and B[l/32][l%32], result register r of lane l is row
// 8(r/4) + 4(l/32) + r%4, column l%32): wavefront tile 32*NJ orbital columns
// x 32*WJ basis functions, the four wavefronts stacked along mu.  Staging as
// k_gemm1_body with (NI, WM) = (2 NJ, 2 WJ).  A wavefront holds NJ*WJ
// independent 32 x 32 accumulators, whose longer steps keep the FP32 matrix
// cores busy with far fewer chains than the 16 x 16 x 4 form needs (measured
// register-only: 0.98 of the FP32 peak with 4 chains per wavefront).
typedef float v16f_k __attribute__((ext_vector_type(16)));

template <typename TS, int NJ, int WJ>
__device__ __attribute__((always_inline)) inline void k_gemm1w_body(int64_t lid, const TS* __restrict__ B, int64_t ldB, int64_t nao,
                                     const float* __restrict__ C, int64_t ldc, int64_t ncol,
                                     float* __restrict__ X, int64_t ldx, int64_t nib, int64_t nmb) {
    constexpr int NI = 2 * NJ, WM = 2 * WJ;
    using S = G1<float, TS, NI, WM>;
    constexpr int BI = 16 * NI, BM = 64 * WM;
    __shared__ __attribute__((aligned(16))) float sC[2][KC][S::PC];
    __shared__ __attribute__((aligned(16))) float sB[2][KC][S::PB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t ib = lid % nib, mb = (lid / nib) % nmb, P = lid / (nib * nmb);
    const int64_t i0 = ib * BI, mu0 = mb * BM;
    const TS* Bp = B + P * ldB;

    v16f_k acc[NJ][WJ];
#pragma unroll
    for (int a = 0; a < NJ; ++a)
#pragma unroll
        for (int b = 0; b < WJ; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

    S st;
    const int nao_ = (int)nao, ldc_ = (int)ldc, mu0_ = (int)mu0;
    st.init(nao_, ldc_, mu0_, (int)i0, tid);
    const float* Cn = C;
    st.load(Bp, Cn, nao_, ldc_, 0, mu0_, tid);
    st.store(sC[0], sB[0], tid);
    if (KC < nao_) st.load(Bp, Cn += KC * ldc, nao_, ldc_, KC, mu0_, tid);
    __syncthreads();
    int buf = 0;
    for (int nu0 = 0; nu0 < nao_; nu0 += KC, buf ^= 1) {
#pragma unroll
        for (int kp = 0; kp < KC / 2; ++kp) {
            const int kr = kp * 2 + (lane >> 5);
            float a[NJ], b[WJ];
#pragma unroll
            for (int t = 0; t < NJ; ++t) a[t] = sC[buf][kr][t * 32 + (lane & 31)];
#pragma unroll
            for (int t = 0; t < WJ; ++t)
                b[t] = sB[buf][kr][(wave * 32 * WJ + t * 32 + (lane & 31)) ^ (16 * (kp >> 1))];
#pragma unroll
            for (int ti = 0; ti < NJ; ++ti)
#pragma unroll
                for (int tj = 0; tj < WJ; ++tj)
                    acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ti], b[tj], acc[ti][tj], 0, 0, 0);
        }
        if (nu0 + KC < nao_) {
            st.store(sC[buf ^ 1], sB[buf ^ 1], tid);
            if (nu0 + 2 * KC < nao_) st.load(Bp, Cn += KC * ldc, nao_, ldc_, nu0 + 2 * KC, mu0_, tid);
        }
        __syncthreads();
    }
#pragma unroll
    for (int ti = 0; ti < NJ; ++ti)
#pragma unroll
        for (int tj = 0; tj < WJ; ++tj)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t i = i0 + ti * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                const int64_t mu = mu0 + wave * 32 * WJ + tj * 32 + (lane & 31);
                if (i < ncol && mu < nao) X[(P * ncol + i) * ldx + mu] = acc[ti][tj][r];
            }
}

template <typename TS, int NJ, int WJ>
__global__ __launch_bounds__(kThreads) void k_gemm1w(const TS* __restrict__ B, int64_t ldB, int64_t nao,
                                                      const float* __restrict__ C, int64_t ldc, int64_t ncol,
                                                      float* __restrict__ X, int64_t ldx, int64_t nib,
                                                      int64_t nmb, int64_t nblk) {
    k_gemm1w_body<TS, NJ, WJ>(xcd_logical(blockIdx.x, nblk), B, ldB, nao, C, ldc, ncol, X, ldx, nib, nmb);
}

// Waves per SIMD the register allocation is held to (LDS allows them):
// FP64 (7,1) 3 instead of 2 (nao=1024, nocc=200: 35.5 -> 34.6 ms for the
// GEMM1 phase); FP32 (13,1) on 16-bit B 4 instead of 3 (nao=2048, nocc=400:
// 309 -> 299 ms, with a 48-byte spill; on FP32 B the same bound ran slower,
// 18.95 -> 19.70 ms, so that tile keeps 3).
template <typename T, typename TS, int NI, int WM>
constexpr int g1_waves() {
    return (sizeof(T) == 8 && NI == 7 && WM == 1) ? 3
           : (sizeof(T) == 4 && sizeof(TS) == 2 && NI == 13 && WM == 1) ? 4
                                                                          : 1;
}

template <typename T, typename TS, int NI, int WM>
__global__ __launch_bounds__(kThreads, (g1_waves<T, TS, NI, WM>())) void k_gemm1(const TS* __restrict__ B, int64_t ldB, int64_t nao,
                                                     const T* __restrict__ C, int64_t ldc, int64_t ncol,
                                                     T* __restrict__ X, int64_t ldx, int64_t nib,
                                                     int64_t nmb, int64_t nblk) {
    k_gemm1_body<T, TS, NI, WM>(xcd_logical(blockIdx.x, nblk), B, ldB, nao, C, ldc, ncol, X, ldx, nib, nmb);
}

// ---------------------------------------------------------------- GEMM2 (SYRK)
// GEMM2 modes.  SY_SYM: K = sum_k s_k x_k x_k^T over the rows of one X,
// lower tiles.  For two factors (D = L R^T) X holds X_L (rows 0..n) and then
// X_R (rows n..2n), and row k of the second operand is row (k + n) mod 2n:
// SY_PAIR_FULL contracts k < n over all tiles (sum_k xL_k xR_k^T);
// SY_PAIR_LOWER contracts k < 2n over the lower tiles, which adds the
// transpose (sum_k xL_k xR_k^T + xR_k xL_k^T, a symmetric result), or k < n
// where the sum is symmetric by itself.
enum { SY_SYM = 0, SY_PAIR_LOWER = 1, SY_PAIR_FULL = 2 };

// Edge of a partial tile's slot: where one lower tile holds all of K, no more than
// its 16-wide blocks.
__host__ __device__ inline int sy_slot(int64_t nao, bool full) {
    return !full && nao < SY_T ? (int)(nao + 15) / 16 * 16 : SY_T;
}

// Staging of one KC-deep chunk of a 128-wide operand panel: 16-byte loads (rows
// of X start 16-byte aligned: ldx is a multiple of V), 8 elements per thread.
// Addresses are a uniform base plus a 32-bit offset that stays the same for
// every chunk; columns past the rows are clamped to the last vector of a row
// (they feed output rows or columns at or past nao, which are never read);
// contraction rows past kend are zeroed, in the last chunk only.
constexpr int SY_P = SY_T + 16;  // LDS pitch: 16 modulo 64 floats / 32 doubles, so a read's rows use different banks

template <typename T>
struct SyPanel {
    static constexpr int V = 16 / sizeof(T);          // elements per load
    static constexpr int TPR = SY_T / V;              // threads per panel row
    static constexpr int RPP = kThreads / TPR;        // rows per pass
    static constexpr int NP = KC / RPP;               // passes per chunk
    T v[NP][V];
    uint32_t off[NP];

    __device__ inline void init(int64_t ldx, int64_t col0, int tid) {
        const int64_t c = col0 + (tid % TPR) * V <= ldx - V ? col0 + (tid % TPR) * V : ldx - V;
#pragma unroll
        for (int p = 0; p < NP; ++p) off[p] = (uint32_t)((tid / TPR + RPP * p) * ldx + c);
    }
    // rows base .. base + 15 (base: uniform)
    __device__ inline void load(const T* __restrict__ base) {
#pragma unroll
        for (int p = 0; p < NP; ++p) __builtin_memcpy(v[p], base + off[p], 16);
    }
    // the same with klive < 16 rows (the others repeat the last one), and
    // `shift` more elements for the rows at or past `from`
    __device__ inline void load_part(const T* __restrict__ base, int klive, int64_t ldx, int tid, int from,
                                     int64_t shift) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int k = tid / TPR + RPP * p;
            const T* src = base + off[p];
            if (k >= klive) src -= (k - klive + 1) * ldx;
            if (min(k, klive - 1) >= from) src += shift;
            __builtin_memcpy(v[p], src, 16);
        }
    }
    // (the loaded values are first looked at here, a chunk of products after their loads)
    __device__ inline void store(T (*s)[SY_P], int klive, int tid) {
        if (__builtin_expect(klive < KC, 0)) {
            rare_path();
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if (tid / TPR + RPP * p >= klive)
#pragma unroll
                    for (int e = 0; e < V; ++e) v[p][e] = T(0);
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) __builtin_memcpy(&s[tid / TPR + RPP * p][(tid % TPR) * V], v[p], 16);
    }
};

// The chunk loop of one output tile: stages the panels and calls step(sA, sB,
// kr) for every 4-deep step.  A chunk's loads are issued when the chunk before
// it has been stored, so they have a whole chunk of products to arrive.  ONE:
// both operands are the same panel (a diagonal tile of an unsigned symmetric
// product), staged once.
template <typename T, int MODE, bool SIGN, bool ONE, typename F>
__device__ __attribute__((always_inline)) inline void sy_loop(const T* __restrict__ X, int64_t ldx, int64_t mu0, int64_t nu0, int64_t ncol,
                                                              const double* __restrict__ sign, int64_t kbeg, int64_t kend,
                                                              int64_t boff, T (*sA)[KC][SY_P], T (*sB)[KC][SY_P],
                                                              F&& step) {
    if (kbeg >= kend) return;
    using S = SyPanel<T>;
    const int tid = threadIdx.x, lane = tid & 63;
    S pa, pb;
    pa.init(ldx, mu0, tid);
    if (!ONE) pb.init(ldx, nu0, tid);
    const T* base = X + kbeg * ldx;      // next chunk to load
    int rows = (int)(kend - kbeg);       // rows from there on
    int64_t left = boff - kbeg;          // rows from there on below boff (pairs)
    int klive = KC;                      // rows of the chunk in the panels
    // signs: their upper halves, and the column of each row staged, moved on by a chunk
    // at a time (whole values spilled, and a remainder of 64-bit numbers per load took
    // longer than a short chunk's products)
    uint32_t sg[S::NP];
    int scol[S::NP];
    const int sstep = SIGN ? KC % (int)ncol : 0;
    if (SIGN) {
#pragma unroll
        for (int p = 0; p < S::NP; ++p) scol[p] = (int)((kbeg + tid / S::TPR + S::RPP * p) % ncol);
    }
    auto load = [&]() {
        klive = min(rows, KC);
        if (__builtin_expect(klive < KC, 0)) {
            rare_path();
            pa.load_part(base, klive, ldx, tid, KC, 0);
        } else {
            pa.load(base);
        }
        if (!ONE) {
            // pairs: row k goes with row (k + boff) mod 2 boff
            const T* bb = MODE == SY_SYM ? base : left > 0 ? base + boff * ldx : base - boff * ldx;
            if (__builtin_expect(klive < KC || (MODE != SY_SYM && left > 0 && left < KC), 0)) {
                rare_path();
                const bool wraps = MODE != SY_SYM && left > 0 && left < KC;
                pb.load_part(bb, klive, ldx, tid, wraps ? (int)left : KC, -2 * boff * ldx);
            } else {
                pb.load(bb);
            }
        }
        if (SIGN) {
#pragma unroll
            for (int p = 0; p < S::NP; ++p) {
                sg[p] = reinterpret_cast<const uint32_t*>(sign)[2 * scol[p] + 1];  // (rows past the last are zeroed whatever their sign)
                scol[p] += sstep;
                if (scol[p] >= (int)ncol) scol[p] -= (int)ncol;
            }
        }
        base += KC * ldx;
        rows -= KC;
        left -= KC;
    };
    auto store = [&](int buf) {
        pa.store(sA[buf], klive, tid);
        if (ONE) return;
        if (SIGN) {
#pragma unroll
            for (int p = 0; p < S::NP; ++p)
#pragma unroll
                for (int e = 0; e < S::V; ++e) pb.v[p][e] = sg[p] > 0x80000000u ? -pb.v[p][e] : pb.v[p][e];
        }
        pb.store(sB[buf], klive, tid);
    };
    int todo = (int)cdiv(kend - kbeg, KC);  // chunks not yet multiplied
    load();
    store(0);
    if (todo > 1) load();
    __syncthreads();
    for (int buf = 0; todo > 0; --todo, buf ^= 1) {
#pragma unroll
        for (int kk = 0; kk < KC / 4; ++kk) {
            const int kr = kk * 4 + (lane >> 4);
            step(sA[buf][kr], ONE ? sA[buf][kr] : sB[buf][kr]);
        }
        if (todo > 1) {
            store(buf ^ 1);
            if (todo > 2) load();
        }
        __syncthreads();
    }
}

// partial[(s*ntl + t)][m][n] = sum_{k in split s} X[k][mu0+m] * sign_k * X[k'][nu0+n]
// (k' = k, or the row paired with k for two factors); block id = s*ntl + t,
// t a lower tile (I >= J) or, for SY_PAIR_FULL, any tile (I = t / nt).
// Three forms, all computing the 16 x 16 blocks the finish reads, every block
// summed over k in the same 4-deep steps:
//   whole tiles: 2 x 2 wavefronts of 64 x 64 (4 x 4 blocks);
//   diagonal tiles of a symmetric result: the 36 blocks on or below the
//     diagonal dealt to the four wavefronts, 9 each (fewer at the edge of K);
//   tiles with rows past nao: each wavefront takes two block columns and the
//     block rows below nao, so no wavefront idles.
// One loop with a branch per product and 64-bit addresses took 16.2 ms at
// nao=1024, naux=4096, nocc=200 in FP64 (every product sat between two jumps and
// waited for its own operands); this takes 14.1 (61 TFLOP/s, matrix cores 80%
// busy).  nao=701 in FP32, whose rows were not 16-byte aligned before ldx was
// padded: 2.62 -> 1.83 ms.
template <typename T, int MODE, bool SIGN>
__device__ __attribute__((always_inline)) inline void k_syrk_body(int64_t lid, const T* __restrict__ X, int64_t ldx, int64_t nrows,
                                   int64_t nao, int64_t ncol, const double* __restrict__ sign,
                                   int64_t kchunk, int64_t ntl, T* __restrict__ part, int64_t boff = 0) {
    __shared__ __attribute__((aligned(16))) T sA[2][KC][SY_P];
    __shared__ __attribute__((aligned(16))) T sB[2][KC][SY_P];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t t = lid % ntl, s = lid / ntl;
    int64_t I, J;
    if (MODE == SY_PAIR_FULL) {
        const int64_t nt = cdiv(nao, SY_T);
        I = t / nt;
        J = t % nt;
    } else {
        I = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
        while (I * (I + 1) / 2 > t) --I;
        while ((I + 1) * (I + 2) / 2 <= t) ++I;
        J = t - I * (I + 1) / 2;
    }
    const int64_t mu0 = I * SY_T, nu0 = J * SY_T;
    const int64_t kbeg = s * kchunk, kend = kbeg + kchunk < nrows ? kbeg + kchunk : nrows;
    const int nbr = nao - mu0 < SY_T ? (int)cdiv(nao - mu0, 16) : SY_T / 16;  // block rows below nao
    const int lc = lane & 15;
    auto put = [&](const typename Mma<T>::acc_t& a, int br, int bc, int edge = SY_T) {
        T* out = part + (s * ntl + t) * (int64_t)(edge * edge);
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(br * 16 + Mma<T>::row(lane, r)) * edge + bc * 16 + lc] = a[r];
    };
    if (MODE != SY_PAIR_FULL && I == J) {
        constexpr int NB = 9;
        const int total = nbr * (nbr + 1) / 2;
        int br[NB], bc[NB];
        typename Mma<T>::acc_t acc[NB];
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int b = wave + 4 * q;
            int i = 0;
            while ((i + 1) * (i + 2) / 2 <= b) ++i;
            br[q] = b < total ? i : 0;
            bc[q] = b < total ? b - i * (i + 1) / 2 : 0;
            acc[q] = Mma<T>::zero();
        }
        const int mine = (total - wave + 3) / 4;
        sy_loop<T, MODE, SIGN, MODE == SY_SYM && !SIGN>(
            X, ldx, mu0, nu0, ncol, sign, kbeg, kend, boff, sA, sB, [&](const T* ra, const T* rb) {
                T a[NB], b[NB];
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    a[q] = ra[br[q] * 16 + lc];
                    b[q] = rb[bc[q] * 16 + lc];
                }
                if (mine == NB) {
#pragma unroll
                    for (int q = 0; q < NB; ++q) acc[q] = Mma<T>::step(a[q], b[q], acc[q]);
                } else {
#pragma unroll
                    for (int q = 0; q < NB; ++q)
                        if (q < mine) acc[q] = Mma<T>::step(a[q], b[q], acc[q]);
                }
            });
        const int slot = sy_slot(nao, false);
#pragma unroll
        for (int q = 0; q < NB; ++q)
            if (q < mine) put(acc[q], br[q], bc[q], slot);
    } else if (nbr < SY_T / 16) {
        typename Mma<T>::acc_t acc[8][2];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i][0] = acc[i][1] = Mma<T>::zero();
        sy_loop<T, MODE, SIGN, false>(X, ldx, mu0, nu0, ncol, sign, kbeg, kend, boff, sA, sB,
                                      [&](const T* ra, const T* rb) {
                                          const T b0 = rb[wave * 32 + lc], b1 = rb[wave * 32 + 16 + lc];
                                          T a[8];
#pragma unroll
                                          for (int i = 0; i < 8; ++i) a[i] = ra[i * 16 + lc];
#pragma unroll
                                          for (int i = 0; i < 8; ++i)
                                              if (i < nbr) {
                                                  acc[i][0] = Mma<T>::step(a[i], b0, acc[i][0]);
                                                  acc[i][1] = Mma<T>::step(a[i], b1, acc[i][1]);
                                              }
                                      });
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < nbr) {
                put(acc[i][0], i, 2 * wave);
                put(acc[i][1], i, 2 * wave + 1);
            }
    } else {
        const int wm = wave >> 1, wn = wave & 1;
        typename Mma<T>::acc_t acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = Mma<T>::zero();
        sy_loop<T, MODE, SIGN, false>(X, ldx, mu0, nu0, ncol, sign, kbeg, kend, boff, sA, sB,
                                      [&](const T* ra, const T* rb) {
                                          T a[4], b[4];
#pragma unroll
                                          for (int q = 0; q < 4; ++q) {
                                              a[q] = ra[wm * 64 + q * 16 + lc];
                                              b[q] = rb[wn * 64 + q * 16 + lc];
                                          }
#pragma unroll
                                          for (int i = 0; i < 4; ++i)
#pragma unroll
                                              for (int j = 0; j < 4; ++j) acc[i][j] = Mma<T>::step(a[i], b[j], acc[i][j]);
                                      });
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) put(acc[i][j], wm * 4 + i, wn * 4 + j);
    }
}

// Waves per SIMD the registers are held to.  FP32 pairs on the lower tiles and signed
// rows carry a second panel, row offsets or signs more than the plain form: at 4 they
// spilled 36 and 87 registers (nao=128, naux=512, 24 columns: K 98 and 85 us; 76 and 54 at 3).
template <typename T, int MODE, bool SIGN>
constexpr int sy_waves() { return sizeof(T) == 8 ? 2 : MODE == SY_PAIR_LOWER || SIGN ? 3 : 4; }

template <typename T, int MODE, bool SIGN = false>
__global__ __launch_bounds__(kThreads, (sy_waves<T, MODE, SIGN>())) void k_syrk(const T* __restrict__ X, int64_t ldx, int64_t nrows,
                                                    int64_t nao, int64_t ncol,
                                                    const double* __restrict__ sign, int64_t kchunk,
                                                    int64_t ntl, int64_t nblk, T* __restrict__ part,
                                                    int64_t boff) {
    // all tiles of one split run on one XCD and share its L2 copy of the X rows
    k_syrk_body<T, MODE, SIGN>(xcd_logical(blockIdx.x, nblk), X, ldx, nrows, nao, ncol, sign, kchunk, ntl, part,
                         boff);
}

// K[mu][nu] = K[nu][mu] = scale * sum_s partial[s][t][m][n] over the lower
// triangle (on diagonal tiles only m >= n is used, so K is exactly symmetric).
template <typename T>
__device__ __attribute__((always_inline)) inline void k_syrk_finish_body(int64_t t, int sub, int nsub, const T* __restrict__ part,
                                          int64_t nsplit, int64_t ntl, int64_t nao, double scale,
                                          double* __restrict__ K) {
    int64_t I = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (I * (I + 1) / 2 > t) --I;
    while ((I + 1) * (I + 2) / 2 <= t) ++I;
    const int64_t J = t - I * (I + 1) / 2;
    const int slot = sy_slot(nao, false), n2 = slot * slot, per = (n2 + nsub - 1) / nsub;
    const int64_t stride = ntl * n2;
    const int e1 = min((sub + 1) * per, n2);
    for (int e = sub * per + (int)threadIdx.x; e < e1; e += kThreads) {
        const int m = slot == SY_T ? e / SY_T : e / slot, n = e - m * slot;
        const int64_t mu = I * SY_T + m, nu = J * SY_T + n;
        if (mu >= nao || nu >= nao) continue;
        if (I == J && m < n) continue;
        const T* p = part + t * n2 + e;
        double v = 0.0;
#pragma unroll 8
        for (int64_t s = 0; s < nsplit; ++s) v += (double)p[s * stride];  // fixed order
        v *= scale;
        K[mu * nao + nu] = v;
        K[nu * nao + mu] = v;
    }
}

// Workgroups per output tile of the finish: kFinSub, or 64 (one element per
// thread) when a few tiles would leave most CUs idle: a thread's sums over the
// splits are a serial chain.
int fin_sub(int64_t ntl) { return ntl * kFinSub < 256 ? 64 : kFinSub; }

// grid: nsub blocks per lower tile, each adding up a contiguous slice of it
template <typename T>
__global__ __launch_bounds__(kThreads) void k_syrk_finish(const T* __restrict__ part, int64_t nsplit,
                                                           int64_t ntl, int64_t nao, double scale, int nsub,
                                                           double* __restrict__ K) {
    k_syrk_finish_body<T>(blockIdx.x / nsub, (int)(blockIdx.x % nsub), nsub, part, nsplit, ntl, nao, scale, K);
}

// Full-tile finish (two factors, no symmetry): K[mu][nu] = scale * sum_s
// partial[s][t][m][n] with t = I * nt + J.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_pair_finish(const T* __restrict__ part, int64_t nsplit,
                                                           int64_t nt, int64_t nao, double scale,
                                                           double* __restrict__ K) {
    constexpr int per = SY_T * SY_T / kFinSub;
    const int64_t t = blockIdx.x / kFinSub;
    const int sub = (int)(blockIdx.x % kFinSub);
    const int64_t I = t / nt, J = t % nt;
    const int64_t stride = nt * nt * (int64_t)(SY_T * SY_T);
    for (int e = sub * per + (int)threadIdx.x; e < (sub + 1) * per; e += kThreads) {
        const int m = e / SY_T, n = e % SY_T;
        const int64_t mu = I * SY_T + m, nu = J * SY_T + n;
        if (mu >= nao || nu >= nao) continue;
        const T* p = part + t * (int64_t)(SY_T * SY_T) + e;
        double v = 0.0;
#pragma unroll 8
        for (int64_t s = 0; s < nsplit; ++s) v += (double)p[s * stride];  // fixed order
        K[mu * nao + nu] = v * scale;
    }
}

template <typename T, typename TS, int NI, int WM>
int launch_gemm1(const dfjk_ctx* h, const void* C, int64_t ldc, int64_t ncol, void* X, int64_t ldx) {
    const int64_t nib = cdiv(ncol, 16 * NI), nmb = cdiv(h->nao, 64 * WM);
    const int64_t nblk = nib * nmb * h->naux;
    k_gemm1<T, TS, NI, WM><<<dim3((unsigned)nblk), kThreads, 0, h->stream>>>(
        static_cast<const TS*>(h->B), h->ldB, h->nao, static_cast<const T*>(C), ldc, ncol,
        static_cast<T*>(X), ldx, nib, nmb, nblk);
    DFJK_LAUNCH_CHECK("k_gemm1");
    return DFJK_OK;
}

template <typename TS, int NJ, int WJ>
int launch_gemm1w(const dfjk_ctx* h, const void* C, int64_t ldc, int64_t ncol, void* X, int64_t ldx) {
    const int64_t nib = cdiv(ncol, 32 * NJ), nmb = cdiv(h->nao, 128 * WJ);
    const int64_t nblk = nib * nmb * h->naux;
    k_gemm1w<TS, NJ, WJ><<<dim3((unsigned)nblk), kThreads, 0, h->stream>>>(
        static_cast<const TS*>(h->B), h->ldB, h->nao, static_cast<const float*>(C), ldc, ncol,
        static_cast<float*>(X), ldx, nib, nmb, nblk);
    DFJK_LAUNCH_CHECK("k_gemm1w");
    return DFJK_OK;
}

// Compiled GEMM1 tiles: (NI, WM) = (i tiles of 16, mu tiles of 16 per wave),
// one launcher per B storage type (FP64 on the FP64 matrix cores; FP32, BF16
// and FP16 dequantised exactly on load and run on the FP32 matrix cores).
typedef int (*G1Launch)(const dfjk_ctx*, const void*, int64_t, int64_t, void*, int64_t);
struct G1Tile {
    int ni, wm;
    G1Launch by_dtype[4];  // indexed by dfjk_dtype
};
#define G1T(a, b)                                                                              \
    {                                                                                          \
        a, b, {                                                                                \
            launch_gemm1<double, double, a, b>, launch_gemm1<float, float, a, b>,              \
                launch_gemm1<float, uint16_t, a, b>, launch_gemm1<float, _Float16, a, b>       \
        }                                                                                      \
    }
// Tiles 14..16: the FP32 32 x 32 x 2 form, (NI, WM) = (2 NJ, 2 WJ); no FP64
// launcher (FP64 has no 32 x 32 step).  Not defaults: at nao=1024,
// naux=4096, nocc=200 (FP32 B) on MI355X they took 24.9 / 29.7 / 28.0 ms
// against 21.5 ms for (13,1) on 16 x 16 x 4 steps (both with one element
// per staging load; (13,1) takes 19.1-19.3 ms with the wide staging).
#define G1W(a, b)                                                                              \
    {                                                                                          \
        2 * a, 2 * b, {                                                                        \
            nullptr, launch_gemm1w<float, a, b>, launch_gemm1w<uint16_t, a, b>,                \
                launch_gemm1w<_Float16, a, b>                                                  \
        }                                                                                      \
    }
const G1Tile kG1Tiles[] = {
    G1T(1, 2), G1T(2, 2), G1T(3, 2), G1T(4, 2), G1T(5, 2), G1T(6, 2),
    G1T(7, 2), G1T(8, 2), G1T(13, 1), G1T(4, 4), G1T(7, 1), G1T(5, 1), G1T(6, 1), G1T(3, 1),
    G1W(2, 1), G1W(1, 2), G1W(2, 2),
    G1T(1, 1), G1T(2, 1), G1T(4, 1), G1T(8, 1), G1T(9, 1), G1T(10, 1), G1T(11, 1), G1T(12, 1),
};
#undef G1T
#undef G1W
constexpr int kNumG1Tiles = sizeof(kG1Tiles) / sizeof(kG1Tiles[0]);

// Copy of C (nao x ncol) with rows ldc apart, FP32 with one rounding per
// element (the columns past ncol stay as they are: GEMM1 does not store their
// products).
template <typename T>
__global__ void c_rows(const double* __restrict__ x, int64_t nao, int64_t ncol, int64_t ldc, T* __restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nao * ncol) y[i / ncol * ldc + i % ncol] = (T)x[i];
}

// Row stride of C for GEMM1: whole 16-byte vectors.  FP64 reads the caller's C
// when that holds already (an even ncol), else a copy; FP32 always a copy.
int64_t c_stride(int64_t ncol, bool f32) { return f32 ? cdiv(ncol, 4) * 4 : cdiv(ncol, 2) * 2; }
template <typename T>
int c_operand(dfjk_ctx* h, const double* C, int64_t ncol, T* copy, const T** out) {
    const int64_t ldc = c_stride(ncol, sizeof(T) == 4);
    if (sizeof(T) == 8 && ldc == ncol) {
        *out = reinterpret_cast<const T*>(C);
        return DFJK_OK;
    }
    c_rows<T><<<dim3((unsigned)cdiv(h->nao * ncol, 256)), 256, 0, h->stream>>>(C, h->nao, ncol, ldc, copy);
    DFJK_LAUNCH_CHECK("c_rows");
    *out = copy;
    return DFJK_OK;
}
// Bytes of the copies of n factors
size_t c_bytes(const dfjk_ctx* h, int64_t ncol, int n) {
    const bool f32 = h->dtype != DFJK_F64;
    if (!f32 && c_stride(ncol, false) == ncol) return 0;
    return (f32 ? 4 : 8) * (size_t)(n * h->nao * c_stride(ncol, f32));
}

// Default tile: one launch of tiles 64 basis functions wide (nao is padded to
// 64 only; two i blocks or fewer take 128, a wavefront needs independent
// products) and ni <= 13 blocks of 16 orbitals (13 accumulator blocks keep two
// FP64 or four FP32 wavefronts on a SIMD), ni chosen for the least padded
// columns, each tile costing another read of B's chunk: weight 1 + w / ni.
// Counting padded columns, FP32 tiles of 13 / 7 / 5 / 3 blocks run at 125 / 122 /
// 119 / 112 TFLOP/s (w = 0.35), the FP64 ones at 57 / 58 / 61 / 55 (w = 0.1: the
// matrix cores bound them all).  Useful TFLOP/s on MI355X, the rule's tile
// first: nocc=200, nao=1024, FP32: (13,1) 120, (7,2) 110, (5,2) 101; FP64: (13,1)
// 55, (7,1) + (6,1) in two launches, B read twice, 55, (5,2) 48; nocc=96,
// nao=500, FP64: (6,1) 55, (3,2) 49; 400 columns, nao=400, FP64: (5,1) 52, (13,1) 48.
int pick_g1_tile(int64_t ncol, bool f32) {
    int best = 0;
    double best_cost = 1e300;
    for (int t = 0; t < kNumG1Tiles; ++t) {
        const int ni = kG1Tiles[t].ni;
        if (ni > 13 || kG1Tiles[t].wm != (ni <= 2 ? 2 : 1) || !kG1Tiles[t].by_dtype[DFJK_F64]) continue;
        const double cost = (double)(cdiv(ncol, 16 * ni) * 16 * ni) * (1.0 + (f32 ? 0.35 : 0.1) / ni);
        if (cost < best_cost) {
            best_cost = cost;
            best = t;
        }
    }
    return best;
}

// X = (B_P C)^T for every P in one launch, with the handle's forced tile or
// pick_g1_tile's (profiled as the GEMM1 phase).
int run_gemm1(dfjk_ctx* h, const void* C, int64_t ncol, void* X, int64_t ldx, bool f32) {
    const int64_t ldc = c_stride(ncol, f32);
    if (h->g1_tile >= 0 && h->g1_tile < kNumG1Tiles) {
        const G1Launch f = kG1Tiles[h->g1_tile].by_dtype[h->dtype];
        if (!f) {
            set_error("GEMM1 tile %d has no FP64 form", h->g1_tile);
            return DFJK_E_INVALID;
        }
        return f(h, C, ldc, ncol, X, ldx);
    }
    return kG1Tiles[pick_g1_tile(ncol, f32)].by_dtype[h->dtype](h, C, ldc, ncol, X, ldx);
}

// Splits of a GEMM2 contraction of nrows terms over ntl output tiles.
// FP64: 512 workgroups are resident; about 4096 of them even out the tiles'
// unequal lengths, and up to 8192 while a split keeps 2048 rows.  Every split
// costs a partial tile to write and to add: nao=1024, naux=4096, nocc=200 GEMM2 +
// finish took 16.9 / 15.3 / 14.7 / 14.4 / 14.5 ms with about 1024 / 2048 / 4096 /
// 8192 / 16384 workgroups, two factors at nao=500 2.36 / 2.08 / 2.10 / 2.21 / 2.28.
// Short contractions keep 384 rows a split (naux=103 at nao=1024) unless that
// leaves CUs idle: then down to kMinRows64 rows.  A repeated K, us, with 384 and with
// fewer rows: nao=112, 7680 rows 92, 38; nao=128, 6144 rows 67, 35; nao=200, 1920
// rows 78, 36.
// Partials above kSmallPart make a new handle's first J and K 0.50 ms, not 0.24 (the
// allocation), so they stay within it where that costs no more than every second
// split: nao=64, naux=256, nocc=16 takes 64, not 86, 39 us repeated either way.
// FP32: about 16384 workgroups, no split shorter than 384 rows and no running
// sum longer than kMaxSum32 terms (the split partials are added in FP64).
constexpr int64_t kMinRows64 = 48, kSmallPart = 2 << 20;
int64_t syrk_max_splits(int64_t nrows, int64_t ntl, int64_t slot, bool f32) {  // never falls as nrows grows
    int64_t nsplit;
    if (f32) {
        nsplit = std::min(std::max(cdiv(16384, ntl), cdiv(nrows, kMaxSum32)), cdiv(nrows, 384));
    } else {
        nsplit = std::max(cdiv(4096, ntl), std::min(cdiv(8192, ntl), nrows / 2048));
        const int64_t fit = kSmallPart / (8 * slot * slot * ntl);
        int64_t more = std::min(cdiv(512, ntl), cdiv(nrows, kMinRows64));
        if (more <= 2 * fit) more = std::min(more, fit);
        nsplit = std::min(nsplit, std::max(cdiv(nrows, 384), more));
    }
    return std::max<int64_t>(nsplit, 1);
}
void syrk_splits(int64_t nrows, int64_t ntl, int64_t slot, bool f32, int64_t* nsplit_out, int64_t* kchunk_out) {
    const int64_t nsplit = syrk_max_splits(nrows, ntl, slot, f32);
    const int64_t kchunk = cdiv(cdiv(nrows, nsplit), KC) * KC;
    *nsplit_out = cdiv(nrows, kchunk);
    *kchunk_out = kchunk;
}

// Workspace of one K build: X rows of nao elements and the GEMM2 split
// partials (nrows contraction terms over ntl output tiles), in bytes.
struct KBytes {
    size_t X, kpart;
};
// Row stride of X: whole 16-byte vectors, for the SYRK's loads
int64_t x_stride(const dfjk_ctx* h, size_t elem) {
    const int64_t V = 16 / (int64_t)elem;
    return cdiv(h->nao, V) * V;
}
KBytes k_bytes(const dfjk_ctx* h, size_t elem, int64_t xrows, int64_t nrows, int64_t ntl, bool full = false) {
    int64_t nsplit, kchunk;
    const size_t slot = (size_t)sy_slot(h->nao, full);
    syrk_splits(nrows, ntl, (int64_t)slot, elem == 4, &nsplit, &kchunk);
    return KBytes{elem * (size_t)xrows * (size_t)x_stride(h, elem), elem * (size_t)(nsplit * ntl) * slot * slot};
}

template <typename T>
int k_build_t(dfjk_ctx* h, const double* C_in, int64_t ncol, const double* sign, double scale, double* K) {
    const int64_t ldx = x_stride(h, sizeof(T));
    const int64_t nrows = h->naux * ncol;
    const int64_t nt = cdiv(h->nao, SY_T);
    const int64_t ntl = nt * (nt + 1) / 2;
    const KBytes need = k_bytes(h, sizeof(T), nrows, nrows, ntl);
    int rc;
    if ((rc = h->X.ensure(need.X)) || (rc = h->kpart.ensure(need.kpart)) || (rc = h->Cw.ensure(c_bytes(h, ncol, 1))))
        return rc;
    T* X = static_cast<T*>(h->X.ptr);

    const T* C = nullptr;
    if ((rc = c_operand<T>(h, C_in, ncol, static_cast<T*>(h->Cw.ptr), &C))) return rc;
    h->prof.begin(PH_K, h->stream);
    h->prof.begin(PH_K_GEMM1, h->stream);
    rc = run_gemm1(h, C, ncol, X, ldx, sizeof(T) == 4);
    h->prof.end(PH_K_GEMM1, h->stream);
    if (rc) return rc;

    int64_t nsplit, kchunk;
    syrk_splits(nrows, ntl, sy_slot(h->nao, false), sizeof(T) == 4, &nsplit, &kchunk);
    T* part = static_cast<T*>(h->kpart.ptr);
    h->prof.begin(PH_K_SYRK, h->stream);
    if (sign)
        k_syrk<T, SY_SYM, true><<<dim3((unsigned)(ntl * nsplit)), kThreads, 0, h->stream>>>(
            X, ldx, nrows, h->nao, ncol, sign, kchunk, ntl, ntl * nsplit, part, 0);
    else
        k_syrk<T, SY_SYM><<<dim3((unsigned)(ntl * nsplit)), kThreads, 0, h->stream>>>(
            X, ldx, nrows, h->nao, ncol, nullptr, kchunk, ntl, ntl * nsplit, part, 0);
    h->prof.end(PH_K_SYRK, h->stream);
    DFJK_LAUNCH_CHECK("k_syrk");
    h->prof.begin(PH_K_FINISH, h->stream);
    const int nsub = fin_sub(ntl);
    k_syrk_finish<T><<<dim3((unsigned)(ntl * nsub)), kThreads, 0, h->stream>>>(part, nsplit, ntl, h->nao, scale,
                                                                                nsub, K);
    h->prof.end(PH_K_FINISH, h->stream);
    h->prof.end(PH_K, h->stream);
    DFJK_LAUNCH_CHECK("k_syrk_finish");
    return DFJK_OK;
}

// Two factors, D = L R^T (L, R: nao x ncol): X_L = (B_P L)^T and X_R =
// (B_P R)^T are stored one after the other, then
//   sym = 0: K = scale * sum_P X_L^T X_R            (all output tiles)
//   sym = 1: K = scale * sum_P (X_L^T X_R + X_R^T X_L)  (lower tiles, mirrored)
template <typename T>
int k_build_pair_t(dfjk_ctx* h, const double* L_in, const double* R_in, int64_t ncol, int sym, double scale, double* K) {
    const int64_t ldx = x_stride(h, sizeof(T));
    const int64_t n1 = h->naux * ncol;  // rows of X_L (and of X_R)
    const int64_t nt = cdiv(h->nao, SY_T);
    const int64_t ntl = sym ? nt * (nt + 1) / 2 : nt * nt;
    const int64_t nrows = sym ? 2 * n1 : n1;  // contraction length
    const KBytes need = k_bytes(h, sizeof(T), 2 * n1, nrows, ntl, !sym);
    int rc;
    if ((rc = h->X.ensure(need.X)) || (rc = h->kpart.ensure(need.kpart)) || (rc = h->Cw.ensure(c_bytes(h, ncol, 2))))
        return rc;
    T* X = static_cast<T*>(h->X.ptr);

    const T *L = nullptr, *R = nullptr;
    T* copy = static_cast<T*>(h->Cw.ptr);
    if ((rc = c_operand<T>(h, L_in, ncol, copy, &L)) ||
        (rc = c_operand<T>(h, R_in, ncol, copy + h->nao * c_stride(ncol, sizeof(T) == 4), &R)))
        return rc;
    h->prof.begin(PH_K, h->stream);
    h->prof.begin(PH_K_GEMM1, h->stream);
    rc = run_gemm1(h, L, ncol, X, ldx, sizeof(T) == 4);
    if (!rc) rc = run_gemm1(h, R, ncol, X + n1 * ldx, ldx, sizeof(T) == 4);
    h->prof.end(PH_K_GEMM1, h->stream);
    if (rc) return rc;

    int64_t nsplit, kchunk;
    syrk_splits(nrows, ntl, sy_slot(h->nao, !sym), sizeof(T) == 4, &nsplit, &kchunk);
    T* part = static_cast<T*>(h->kpart.ptr);
    const dim3 grid((unsigned)(ntl * nsplit));
    h->prof.begin(PH_K_SYRK, h->stream);
    if (sym)
        k_syrk<T, SY_PAIR_LOWER><<<grid, kThreads, 0, h->stream>>>(X, ldx, nrows, h->nao, ncol, nullptr, kchunk, ntl,
                                                                     ntl * nsplit, part, n1);
    else
        k_syrk<T, SY_PAIR_FULL><<<grid, kThreads, 0, h->stream>>>(X, ldx, nrows, h->nao, ncol, nullptr, kchunk, ntl,
                                                                    ntl * nsplit, part, n1);
    h->prof.end(PH_K_SYRK, h->stream);
    DFJK_LAUNCH_CHECK("k_syrk (two factors)");
    h->prof.begin(PH_K_FINISH, h->stream);
    const int nsub = fin_sub(ntl);
    if (sym)
        k_syrk_finish<T><<<dim3((unsigned)(ntl * nsub)), kThreads, 0, h->stream>>>(part, nsplit, ntl, h->nao, scale,
                                                                                    nsub, K);
    else
        k_pair_finish<T><<<dim3((unsigned)(ntl * kFinSub)), kThreads, 0, h->stream>>>(part, nsplit, nt, h->nao,
                                                                                       scale, K);
    h->prof.end(PH_K_FINISH, h->stream);
    h->prof.end(PH_K, h->stream);
    DFJK_LAUNCH_CHECK("k finish (two factors)");
    return DFJK_OK;
}

// ---------------------------------------------------------------- K of a density
// X[(P, i)][mu] = B_P[i][mu] from the packed triangle (rows ldx apart): 64 x 64
// tiles (I >= J) of every P, written as read and transposed through LDS.
template <typename T, typename TS>
__global__ __launch_bounds__(kThreads) void unpack_rows(const TS* __restrict__ B, int64_t ldB, int64_t nao,
                                                         int64_t naux, T* __restrict__ X, int64_t ldx) {
    constexpr int UT = 64;
    __shared__ T tile[UT][UT + 1];
    const int64_t t = blockIdx.x;
    int64_t I = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (I * (I + 1) / 2 > t) --I;
    while ((I + 1) * (I + 2) / 2 <= t) ++I;
    const int64_t i0 = I * UT, j0 = (t - I * (I + 1) / 2) * UT;
    const int c = threadIdx.x % UT, r0 = threadIdx.x / UT;
    for (int64_t P = blockIdx.y; P < naux; P += gridDim.y) {
        const TS* Bp = B + P * ldB;
        T* Xp = X + P * nao * ldx;
#pragma unroll
        for (int q = 0; q < UT / 4; ++q) {
            const int64_t i = i0 + r0 + 4 * q, j = j0 + c;
            T v = T(0);
            if (i < nao && j <= i) {
                v = to_compute<T, TS>(Bp[i * (i + 1) / 2 + j]);
                Xp[i * ldx + j] = v;
            }
            tile[r0 + 4 * q][c] = v;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < UT / 4; ++q) {
            const int64_t j = j0 + r0 + 4 * q, i = i0 + c;
            if (i < nao && j < i) Xp[j * ldx + i] = tile[c][r0 + 4 * q];
        }
        __syncthreads();
    }
}

// K = sum_P B_P D B_P for a symmetric D (nao x nao) as the product of the rows of
// D B_P (GEMM1 with D for C) and those of B_P itself.  FP64: one contraction over
// (P, i) on the lower tiles.  FP32: D B_P times B_P and B_P times D B_P, half each,
// as for the two factors (D, I), which it equals bit for bit: the product of B_P
// and I is B_P, so only the reading of it is left out.
// nao=400, naux=1600, FP64: J and K 13.3 -> 7.7 ms (GEMM1 with I 3.3 ms -> 0.8 of copying,
// the contraction half as long).
template <typename T>
int k_build_density_t(dfjk_ctx* h, const double* D, double* K) {
    const int64_t nao = h->nao, ldx = x_stride(h, sizeof(T)), n1 = h->naux * nao;
    const int64_t nt = cdiv(nao, SY_T), ntl = nt * (nt + 1) / 2;
    const bool f32 = sizeof(T) == 4;
    const int64_t nrows = f32 ? 2 * n1 : n1;
    const KBytes need = k_bytes(h, sizeof(T), 2 * n1, nrows, ntl);
    int rc;
    if ((rc = h->X.ensure(need.X)) || (rc = h->kpart.ensure(need.kpart)) || (rc = h->Cw.ensure(c_bytes(h, nao, 1))))
        return rc;
    T* X = static_cast<T*>(h->X.ptr);
    T* XR = X + n1 * ldx;
    const T* Dw = nullptr;
    if ((rc = c_operand<T>(h, D, nao, static_cast<T*>(h->Cw.ptr), &Dw))) return rc;
    const hipStream_t st = h->stream;
    h->prof.begin(PH_K, st);
    h->prof.begin(PH_K_GEMM1, st);
    rc = run_gemm1(h, Dw, nao, X, ldx, f32);
    if (!rc) {
        const int64_t nu = cdiv(nao, 64);
        const dim3 grid((unsigned)(nu * (nu + 1) / 2), (unsigned)std::min<int64_t>(h->naux, 65535));
        auto unpack = [&](auto* B) {
            using TS = std::remove_const_t<std::remove_pointer_t<decltype(B)>>;
            unpack_rows<T, TS><<<grid, kThreads, 0, st>>>(B, h->ldB, nao, h->naux, XR, ldx);
        };
        if constexpr (sizeof(T) == 8)
            unpack(static_cast<const double*>(h->B));
        else if (h->dtype == DFJK_F32)
            unpack(static_cast<const float*>(h->B));
        else if (h->dtype == DFJK_BF16)
            unpack(static_cast<const uint16_t*>(h->B));
        else
            unpack(static_cast<const _Float16*>(h->B));
    }
    h->prof.end(PH_K_GEMM1, st);
    if (rc) return rc;
    DFJK_LAUNCH_CHECK("unpack_rows");
    int64_t nsplit, kchunk;
    syrk_splits(nrows, ntl, sy_slot(nao, false), f32, &nsplit, &kchunk);
    T* part = static_cast<T*>(h->kpart.ptr);
    h->prof.begin(PH_K_SYRK, st);
    k_syrk<T, SY_PAIR_LOWER><<<dim3((unsigned)(ntl * nsplit)), kThreads, 0, st>>>(X, ldx, nrows, nao, nao, nullptr,
                                                                                  kchunk, ntl, ntl * nsplit, part, n1);
    h->prof.end(PH_K_SYRK, st);
    DFJK_LAUNCH_CHECK("k_syrk (density)");
    h->prof.begin(PH_K_FINISH, st);
    const int nsub = fin_sub(ntl);
    k_syrk_finish<T><<<dim3((unsigned)(ntl * nsub)), kThreads, 0, st>>>(part, nsplit, ntl, nao, f32 ? 0.5 : 1.0, nsub,
                                                                        K);
    h->prof.end(PH_K_FINISH, st);
    h->prof.end(PH_K, st);
    DFJK_LAUNCH_CHECK("k_syrk_finish");
    return DFJK_OK;
}

// ---------------------------------------------------------------- batched
__global__ __launch_bounds__(kThreads) void kb_kernel(int kind, const MolDesc* __restrict__ mols, PhaseList pl) {
    const int64_t b = blockIdx.x;
    const int j = find_mol(pl.prefix, pl.n, b);
    const MolDesc& d = mols[pl.ids[j]];
    const int64_t lid = b - pl.prefix[j];
    if (kind == BP_CF32) {
        const int64_t e = lid * kThreads + threadIdx.x;
        if (e < d.nao * d.nocc) as_global(d.Cf)[e / d.nocc * d.ldcf + e % d.nocc] = (float)as_global(d.C)[e];
    } else if (kind == BP_KFIN) {
        k_syrk_finish_body<float>(lid / kFinSub, (int)(lid % kFinSub), kFinSub, as_global(d.kpart), d.nsplit, d.ntl,
                                  d.nao, 2.0, as_global(d.K));
    }
}

// GEMM2 of every molecule: 4 waves per SIMD, as the single one.  A kernel of its
// own: beside the other phases its registers spilled.
__global__ __launch_bounds__(kThreads, 4) void kb_syrk(const MolDesc* __restrict__ mols, PhaseList pl) {
    const int64_t b = xcd_runs(blockIdx.x, pl.nblk);
    const int j = find_mol(pl.prefix, pl.n, b);
    const MolDesc& d = mols[pl.ids[j]];
    k_syrk_body<float, SY_SYM, false>(b - pl.prefix[j], as_global(d.X), d.ldx, d.naux * d.nocc, d.nao, d.nocc,
                                      nullptr, d.kchunk, d.ntl, as_global(d.kpart));
}

// Batched GEMM1 tiles with at most 8 accumulator blocks are held to 5 waves
// per SIMD (their LDS allows 6); larger ones would spill.
template <int NI, int WM>
constexpr int kb_g1_waves() { return NI * WM <= 8 ? 5 : 1; }

template <typename TS, int NI, int WM>
__global__ __launch_bounds__(kThreads, (kb_g1_waves<NI, WM>())) void kb_gemm1(const MolDesc* __restrict__ mols,
                                                                             PhaseList pl) {
    const int64_t b = xcd_runs(blockIdx.x, pl.nblk);
    const int j = find_mol(pl.prefix, pl.n, b);
    const MolDesc& d = mols[pl.ids[j]];
    k_gemm1_body<float, TS, NI, WM>(b - pl.prefix[j], as_global(static_cast<const TS*>(d.B)), d.ldB, d.nao,
                                    as_global(d.Cf), d.ldcf, d.nocc, as_global(d.X), d.ldx, d.g1_nib, d.g1_nmb);
}

template <int NI, int WM>
int launch_kb_gemm1(hipStream_t st, int dtype, const MolDesc* mols, const PhaseList& pl) {
    const dim3 grid((unsigned)pl.nblk);
    switch (dtype) {
        case DFJK_F32: kb_gemm1<float, NI, WM><<<grid, kThreads, 0, st>>>(mols, pl); break;
        case DFJK_BF16: kb_gemm1<uint16_t, NI, WM><<<grid, kThreads, 0, st>>>(mols, pl); break;
        case DFJK_F16: kb_gemm1<_Float16, NI, WM><<<grid, kThreads, 0, st>>>(mols, pl); break;
        default: set_error("batched builds take FP32, BF16 or FP16 B"); return DFJK_E_DTYPE;
    }
    DFJK_LAUNCH_CHECK("kb_gemm1");
    return DFJK_OK;
}

template <typename TS, int NJ, int WJ>
__global__ __launch_bounds__(kThreads) void kb_gemm1w(const MolDesc* __restrict__ mols, PhaseList pl) {
    const int64_t b = xcd_runs(blockIdx.x, pl.nblk);
    const int j = find_mol(pl.prefix, pl.n, b);
    const MolDesc& d = mols[pl.ids[j]];
    k_gemm1w_body<TS, NJ, WJ>(b - pl.prefix[j], as_global(static_cast<const TS*>(d.B)), d.ldB, d.nao,
                              as_global(d.Cf), d.ldcf, d.nocc, as_global(d.X), d.ldx, d.g1_nib, d.g1_nmb);
}

template <int NJ, int WJ>
int launch_kb_gemm1w(hipStream_t st, int dtype, const MolDesc* mols, const PhaseList& pl) {
    const dim3 grid((unsigned)pl.nblk);
    switch (dtype) {
        case DFJK_F32: kb_gemm1w<float, NJ, WJ><<<grid, kThreads, 0, st>>>(mols, pl); break;
        case DFJK_BF16: kb_gemm1w<uint16_t, NJ, WJ><<<grid, kThreads, 0, st>>>(mols, pl); break;
        case DFJK_F16: kb_gemm1w<_Float16, NJ, WJ><<<grid, kThreads, 0, st>>>(mols, pl); break;
        default: set_error("batched builds take FP32, BF16 or FP16 B"); return DFJK_E_DTYPE;
    }
    DFJK_LAUNCH_CHECK("kb_gemm1w");
    return DFJK_OK;
}

typedef int (*KbLaunch)(hipStream_t, int, const MolDesc*, const PhaseList&);
#define KBT(a, b) launch_kb_gemm1<a, b>
const KbLaunch kKbTiles[] = {KBT(1, 2), KBT(2, 2), KBT(3, 2), KBT(4, 2), KBT(5, 2), KBT(6, 2),
                             KBT(7, 2), KBT(8, 2), KBT(13, 1), KBT(4, 4), KBT(7, 1), KBT(5, 1),
                             KBT(6, 1), KBT(3, 1), launch_kb_gemm1w<2, 1>, launch_kb_gemm1w<1, 2>,
                             launch_kb_gemm1w<2, 2>, KBT(1, 1), KBT(2, 1), KBT(4, 1), KBT(8, 1), KBT(9, 1),
                             KBT(10, 1), KBT(11, 1), KBT(12, 1)};
#undef KBT
static_assert(sizeof(kKbTiles) / sizeof(kKbTiles[0]) == kNumG1Tiles, "tile tables differ");

}  // namespace

int k_batch_phase(hipStream_t st, int kind, int dtype, const MolDesc* mols, const PhaseList& pl) {
    (void)dtype;
    if (pl.nblk <= 0) return DFJK_OK;
    if (kind == BP_SYRK)
        kb_syrk<<<dim3((unsigned)pl.nblk), kThreads, 0, st>>>(mols, pl);
    else
        kb_kernel<<<dim3((unsigned)pl.nblk), kThreads, 0, st>>>(kind, mols, pl);
    DFJK_LAUNCH_CHECK("kb_kernel");
    return DFJK_OK;
}

int k_batch_gemm1(hipStream_t st, int dtype, int tile, const MolDesc* mols, const PhaseList& pl) {
    if (pl.nblk <= 0) return DFJK_OK;
    if (tile < 0 || tile >= kNumG1Tiles) {
        set_error("tile %d out of range", tile);
        return DFJK_E_INVALID;
    }
    return kKbTiles[tile](st, dtype, mols, pl);
}

int pick_tile(int64_t ncol) { return pick_g1_tile(ncol, true); }

int tile_nb(int tile, int64_t nao, int64_t ncol, int64_t* nib, int64_t* nmb) {
    if (tile < 0 || tile >= kNumG1Tiles) return DFJK_E_INVALID;
    *nib = cdiv(ncol, 16 * kG1Tiles[tile].ni);
    *nmb = cdiv(nao, 64 * kG1Tiles[tile].wm);
    return DFJK_OK;
}

int k_build_factored(dfjk_ctx* h, const double* C, int64_t ncol, const double* sign, double scale,
                     double* K) {
    if (h->dtype == DFJK_F64) return k_build_t<double>(h, C, ncol, sign, scale, K);
    if ((h->dtype == DFJK_BF16 || h->dtype == DFJK_F16) && h->opts.k16 && !sign)
        return k_build_16(h, C, ncol, scale, K);
    // FP32 compute for FP32, BF16 and FP16 storage of B
    return k_build_t<float>(h, C, ncol, sign, scale, K);
}

int k_build_pair(dfjk_ctx* h, const double* L, const double* R, int64_t ncol, int sym, double scale, double* K) {
    if (h->dtype == DFJK_F64) return k_build_pair_t<double>(h, L, R, ncol, sym, scale, K);
    // FP32 compute for FP32, BF16 and FP16 storage of B (also with the k16
    // option: the 16-bit exchange takes one factor)
    return k_build_pair_t<float>(h, L, R, ncol, sym, scale, K);
}

int k_build_density(dfjk_ctx* h, const double* D, double* K) {
    return h->dtype == DFJK_F64 ? k_build_density_t<double>(h, D, K) : k_build_density_t<float>(h, D, K);
}

int k_reserve(dfjk_ctx* h, int64_t max_ncol) {
    const size_t elem = h->dtype == DFJK_F64 ? 8 : 4;
    const int64_t nt = cdiv(h->nao, SY_T), lower = nt * (nt + 1) / 2;
    const int64_t n1 = h->naux * max_ncol, half = h->naux * (max_ncol / 2);
    // one factor of max_ncol columns; two factors of max_ncol / 2 each (the
    // symmetric form contracts both over the lower tiles, the general one
    // half of the rows over every tile)
    const KBytes a = k_bytes(h, elem, n1, n1, lower);
    const KBytes b = k_bytes(h, elem, 2 * half, 2 * half, lower);
    // the partials by the splits aimed at, not those that whole chunks leave: a
    // call of fewer columns may be cut into more of them (24600 rows into 385,
    // 24576 into 512)
    const auto partials = [&](int64_t nrows, int64_t ntl, bool full) {
        const size_t slot = (size_t)sy_slot(h->nao, full);
        return elem * (size_t)(syrk_max_splits(nrows, ntl, (int64_t)slot, elem == 4) * ntl) * slot * slot;
    };
    const size_t kp =
        std::max({partials(n1, lower, false), partials(2 * half, lower, false), partials(half, nt * nt, true)});
    int rc;
    if ((rc = h->X.ensure(a.X > b.X ? a.X : b.X))) return rc;
    if ((rc = h->kpart.ensure(kp))) return rc;
    // copies of C: one factor of up to max_ncol columns or two of half as many
    // (an FP64 copy is only made for an odd number of columns; a call may use
    // fewer columns than reserved)
    const size_t f = h->dtype == DFJK_F64 ? 8 : 4;
    const size_t one = f * (size_t)(h->nao * c_stride(max_ncol, f == 4));
    const size_t two = 2 * f * (size_t)(h->nao * c_stride(max_ncol / 2, f == 4));
    if ((rc = h->Cw.ensure(one > two ? one : two))) return rc;
    return DFJK_OK;
}

int k_tile_count() { return kNumG1Tiles; }

bool k_tile_has_dtype(int t, int dtype) {
    return t >= 0 && t < kNumG1Tiles && dtype >= 0 && dtype < 4 && kG1Tiles[t].by_dtype[dtype] != nullptr;
}

int k_tile_info(int t, int* ni, int* wm) {
    if (t < 0 || t >= kNumG1Tiles) return DFJK_E_INVALID;
    *ni = kG1Tiles[t].ni;
    *wm = kG1Tiles[t].wm;
    return DFJK_OK;
}

}  // namespace dfjk
