// One 16 x 16 tile of a small FP64 product on the matrix cores.
#pragma once

#include <hip/hip_runtime.h>

#include "mma.h"

namespace dfjk {

// C = alpha op(A) op(B) + beta C for small products (the SCF's nao x nao ones):
// one 16 x 16 tile per workgroup of 256 threads, the contraction split over its
// four wavefronts and added in order, operands straight from L2 into the
// matrix-core layout.  Latency bounds these, so every load is independent and
// there is one barrier: nao=128 4 us (tiles of 64 and 128 leave one to four
// workgroups with a serial loop of staged chunks: 7 to 16 and 24 us).
template <bool TA, bool TB>
__device__ inline void gemm_tile16(int M, int N, int K, double alpha, const double* __restrict__ A, int64_t lda,
                                   const double* __restrict__ B, int64_t ldb, double beta, double* __restrict__ C,
                                   int64_t ldc) {
    __shared__ double red[4][16][17];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;
    const int gm = min(m0 + (lane & 15), M - 1), gn = min(n0 + (lane & 15), N - 1);
    const int per = (K + 15) / 16 * 4;  // contraction terms per wavefront, in whole steps
    const int kb = wave * per, ke = min(kb + per, K);
    const double *Ak = TA ? A + gm : A + gm * lda, *Bk = TB ? B + gn * ldb : B + gn;
    const int64_t sa = TA ? lda : 1, sb = TB ? 1 : ldb;
    v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
    int k0 = kb;
    for (; k0 + 32 <= ke; k0 += 32) {  // eight steps' loads in flight
        double a[8], b[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t k = k0 + 4 * j + (lane >> 4);
            a[j] = Ak[k * sa];
            b[j] = Bk[k * sb];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) acc = Mma<double>::step(a[j], b[j], acc);
    }
    for (; k0 < ke; k0 += 4) {
        const int k = k0 + (lane >> 4);
        double a = 0.0, b = 0.0;
        if (k < ke) a = Ak[k * sa], b = Bk[k * sb];
        acc = Mma<double>::step(a, b, acc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][Mma<double>::row(lane, r)][lane & 15] = acc[r];
    __syncthreads();
    const int r = tid >> 4, c = tid & 15;
    if (m0 + r < M && n0 + c < N) {
        const double v = ((red[0][r][c] + red[1][r][c]) + red[2][r][c]) + red[3][r][c];
        double* dst = C + (m0 + r) * ldc + n0 + c;
        *dst = alpha * v + (beta == 0.0 ? 0.0 : beta * *dst);
    }
}

}  // namespace dfjk
