// Learned initial guess: a three-layer perceptron (d_in -> H -> H -> 1, SiLU)
// that maps features of a basis-function pair to a correction of the
// core-Hamiltonian guess density.  The paper's mean-field runs accept any
// guess density (Sec. IV.A.1), so the prediction is used as given.
//
// All arithmetic is FP32 on the matrix cores (products) and vector units
// (activations, reductions, Adam); with the BF16 compute mode the three
// hidden-layer products (forward, input gradient, weight gradient) round
// their FP32 operands to bfloat16 and run on the 16-bit matrix cores with
// FP32 sums.  Weight gradients contract over the batch with the batch split
// into slabs whose partial products are added in a fixed order, so a training
// step is bitwise reproducible.  A step at 65536 rows and 256 hidden units is
// three products of 91-136 us and three passes over the activations of 17-47
// us, 0.45 ms with its sums (23.9 ms with one launch per slab and one pass per
// elementwise operation).
#include <algorithm>
#include <new>
#include <vector>

#include "dense.h"
#include "numerics.h"

namespace dfjk {
namespace {

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

__device__ inline float silu(float z) { return z / (1.f + __expf(-z)); }
// The row passes below give a lane 4 consecutive hidden units of a row (16-byte
// loads and stores) and a wavefront 256 of them; units at or past h are read
// as zero and never written.
__device__ inline void row4(float (&v)[4], const float* __restrict__ row, int c, int h) {
    if (c + 4 <= h) {
        __builtin_memcpy(v, row + c, 16);
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = c + q < h ? row[c + q] : 0.f;
    }
}
__device__ inline void put4(float* __restrict__ row, int c, int h, const float (&v)[4]) {
    if (c + 4 <= h) {
        __builtin_memcpy(row + c, v, 16);
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (c + q < h) row[c + q] = v[q];
    }
}

// Layer 1: Z = X W^T + b and A = silu(Z), kL1Rows rows per wavefront and 256
// hidden units.  The contraction is d_in (8) long, so this is bound by the
// stores of Z and A: a lane keeps the weights of its 4 units and its sums in
// registers, the row of X is a uniform load.  Z may be null (a plain forward
// pass does not need it).
constexpr int kL1Rows = 8;
__global__ __launch_bounds__(256) void layer1(const float* __restrict__ X, int64_t n, int d,
                                              const float* __restrict__ W, const float* __restrict__ b, int h,
                                              float* __restrict__ Z, float* __restrict__ A) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = blockIdx.y * 256 + 4 * (threadIdx.x & 63);
    const int64_t r0 = ((int64_t)blockIdx.x * 4 + wave) * kL1Rows;
    if (r0 >= n) return;
    float z[kL1Rows][4], bc[4];
    row4(bc, b, c, h);
#pragma unroll
    for (int r = 0; r < kL1Rows; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) z[r][q] = 0.f;
    for (int k0 = 0; k0 < d; k0 += 8) {
        float w[4][8];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k)
                w[q][k] = c + q < h && k0 + k < d ? W[(int64_t)(c + q) * d + k0 + k] : 0.f;
#pragma unroll
        for (int r = 0; r < kL1Rows; ++r) {
            const int64_t row = r0 + r < n ? r0 + r : n - 1;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k0 + k < d) {
                    const float x = X[row * d + k0 + k];
#pragma unroll
                    for (int q = 0; q < 4; ++q) z[r][q] = __builtin_fmaf(x, w[q][k], z[r][q]);
                }
        }
    }
#pragma unroll
    for (int r = 0; r < kL1Rows; ++r)
        if (r0 + r < n) {
            float s[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                z[r][q] += bc[q];
                s[q] = silu(z[r][q]);
            }
            if (Z) put4(Z + (r0 + r) * h, c, h, z[r]);
            put4(A + (r0 + r) * h, c, h, s);
        }
}

// Output layer: y[i] = silu(Z2[i,:]) . w + b, one wavefront per row
__global__ void head(const float* __restrict__ Z2, const float* __restrict__ w, const float* __restrict__ b,
                     int64_t n, int h, float* __restrict__ y) {
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n) return;
    float s = 0.f;
    for (int k = lane; k < h; k += 64) s = __builtin_fmaf(silu(Z2[row * h + k]), w[k], s);
    s = wave_sum(s);
    if (lane == 0) y[row] = s + b[0];
}

// Output layer with the loss and everything of the backward pass that hangs
// on one row: y as above, gy = 2 (y - t) / n, gZ2 = gy w silu'(Z2), and the
// column sums gb2 = sum gZ2, gw = sum gy silu(Z2), with the sums of gy and of
// (y - t)^2.  One wavefront per row, the row (4 NC values per lane) in
// registers between its dot product and its gradient, so Z2 is read once and
// gZ2 written once (bound by those 2 x 4 n h bytes).  A workgroup takes `per`
// rows; its sums go to part[block][0..h) gb2, [h..2h) gw, [2h] sum gy, [2h+1]
// loss: the order of the parameters.  Rows and columns are fixed per wavefront
// and lane: reproducible.
template <int NC>
__global__ __launch_bounds__(256) void head_grad(const float* __restrict__ Z2, const float* __restrict__ w,
                                                 const float* __restrict__ b, const float* __restrict__ t,
                                                 int64_t n, int h, int64_t per, float* __restrict__ gZ2,
                                                 float* __restrict__ part) {
    __shared__ float red[4][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * per, r1 = r0 + per < n ? r0 + per : n;
    const float b0 = b[0], two_n = 2.f / (float)n;
    float wr[NC][4], gw[NC][4], gb[NC][4];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        row4(wr[c], w, c * 256 + 4 * lane, h);
#pragma unroll
        for (int q = 0; q < 4; ++q) gw[c][q] = gb[c][q] = 0.f;
    }
    float sgy = 0.f;
    double loss = 0.0;  // one value per row for the whole wavefront: FP64 costs nothing here
    float zn[NC][4];  // the next row, loaded while this one is worked on
    auto load = [&](int64_t i) {
#pragma unroll
        for (int c = 0; c < NC; ++c) row4(zn[c], Z2 + i * h, c * 256 + 4 * lane, h);
    };
    if (r0 + wave < r1) load(r0 + wave);
    for (int64_t i = r0 + wave; i < r1; i += 4) {
        float sg[NC][4], sl[NC][4], s = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float z = zn[c][q];
                const float g = 1.f / (1.f + __expf(-z));
                sl[c][q] = z * g;
                sg[c][q] = g * (1.f + z * (1.f - g));
                s = __builtin_fmaf(sl[c][q], wr[c][q], s);
            }
        if (i + 4 < r1) load(i + 4);
        s = wave_sum(s);
        const float d = (s + b0) - t[i];
        const float gy = two_n * d;
        loss = fma((double)d, (double)d, loss);
        sgy += gy;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            float g[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                g[q] = gy * wr[c][q] * sg[c][q];
                gw[c][q] = __builtin_fmaf(gy, sl[c][q], gw[c][q]);
                gb[c][q] += g[q];
            }
            put4(gZ2 + i * h, c * 256 + 4 * lane, h, g);
        }
    }
    float* out = part + (int64_t)blockIdx.x * (2 * h + 2);
    auto emit = [&](const float (&v)[4], float* dst, int c, int lim) {
#pragma unroll
        for (int q = 0; q < 4; ++q) red[wave][4 * lane + q] = v[q];
        __syncthreads();
        const int e = threadIdx.x;
        if (c + e < lim) dst[c + e] = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
        __syncthreads();
    };
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        emit(gb[c], out, c * 256, h);
        emit(gw[c], out + h, c * 256, h);
    }
    const float last[4] = {sgy, (float)loss, 0.f, 0.f};  // lane 0's columns
    emit(last, out + 2 * h, 0, 2);
}

// Weight and bias gradient of layer 1: part[block] holds sum gZ1[i][c] X[i][k]
// (c < h, k < d) and then sum gZ1[i][c], over the block's `per` rows.  Bound by
// the one read of gZ1; rows round-robin over the four wavefronts, 8 columns of
// X (uniform loads) at a time.
__global__ __launch_bounds__(256) void layer1_grad(const float* __restrict__ G, const float* __restrict__ X,
                                                   int64_t n, int h, int d, int64_t per,
                                                   float* __restrict__ part) {
    __shared__ float red[4][256 * 9];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cb = blockIdx.y * 256, c = cb + 4 * lane;
    const int64_t r0 = (int64_t)blockIdx.x * per, r1 = r0 + per < n ? r0 + per : n;
    float* out = part + (int64_t)blockIdx.x * (h * (int64_t)d + h);
    for (int k0 = 0; k0 < d; k0 += 8) {
        float s[9][4];
#pragma unroll
        for (int k = 0; k < 9; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) s[k][q] = 0.f;
#pragma unroll 4
        for (int64_t i = r0 + wave; i < r1; i += 4) {
            float g[4];
            row4(g, G + i * h, c, h);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float x = k0 + k < d ? X[i * d + k0 + k] : 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) s[k][q] = __builtin_fmaf(g[q], x, s[k][q]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) s[8][q] += g[q];
        }
        __syncthreads();  // the previous group's sums have been read
#pragma unroll
        for (int k = 0; k < 9; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) red[wave][(4 * lane + q) * 9 + k] = s[k][q];
        __syncthreads();
        for (int e = threadIdx.x; e < 256 * 9; e += 256) {
            const int u = cb + e / 9, k = e % 9;
            if (u >= h) continue;
            const float v = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
            if (k == 8)
                out[(int64_t)h * d + u] = v;  // the same sum for every group of columns
            else if (k0 + k < d)
                out[(int64_t)u * d + k0 + k] = v;
        }
    }
}

// out[c] = sum_p part[p * ld + c] for c < cols, in FP64 and a fixed order: a
// workgroup adds 64 columns, its four wavefronts a quarter of the parts each.  With
// loss, the column past them is the sum of squares: loss = inv_n times it.
__global__ __launch_bounds__(256) void sum_parts(const float* __restrict__ part, int64_t np, int64_t ld,
                                                 int64_t cols, float* __restrict__ out, float* __restrict__ loss,
                                                 double inv_n) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * 64 + lane;
    const int64_t q = (np + 3) / 4, p0 = wave * q, p1 = p0 + q < np ? p0 + q : np;
    double s = 0.0;
    if (c < cols + (loss ? 1 : 0)) {
#pragma unroll 8
        for (int64_t p = p0; p < p1; ++p) s += (double)part[p * ld + c];
    }
    red[wave][lane] = s;
    __syncthreads();
    const double v = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    if (wave == 0 && c < cols) out[c] = (float)v;
    if (wave == 0 && c == cols && loss) loss[0] = (float)(v * inv_n);
}

__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                            float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Pair features of one system (mu <= nu, packed order p = nu(nu+1)/2 + mu):
// [Dcore_mn, H_mn, (H_mm + H_nn)/2, |H_mm - H_nn|, r/10, exp(-r^2),
//  delta_mn, (rank_m + rank_n) / (2 nao)] with rank = position of H_mm in
// ascending order of the diagonal of H.
__global__ void pair_features(const double* __restrict__ H, const double* __restrict__ Dc,
                              const double* __restrict__ R, int64_t nao, float* __restrict__ X) {
    const int64_t nu = blockIdx.x;
    const double hnn = H[nu * nao + nu];
    int rn = 0;
    for (int64_t k = 0; k < nao; ++k) {
        const double hk = H[k * nao + k];
        rn += (hk < hnn || (hk == hnn && k < nu)) ? 1 : 0;
    }
    for (int64_t mu = threadIdx.x; mu <= nu; mu += blockDim.x) {
        const double hmm = H[mu * nao + mu];
        int rm = 0;
        for (int64_t k = 0; k < nao; ++k) {
            const double hk = H[k * nao + k];
            rm += (hk < hmm || (hk == hmm && k < mu)) ? 1 : 0;
        }
        const double dx = R[3 * mu] - R[3 * nu], dy = R[3 * mu + 1] - R[3 * nu + 1],
                     dz = R[3 * mu + 2] - R[3 * nu + 2];
        const double r2 = dx * dx + dy * dy + dz * dz;
        float* x = X + (nu * (nu + 1) / 2 + mu) * 8;
        x[0] = (float)Dc[mu * nao + nu];
        x[1] = (float)H[mu * nao + nu];
        x[2] = (float)(0.5 * (hmm + hnn));
        x[3] = (float)fabs(hmm - hnn);
        x[4] = (float)(sqrt(r2) * 0.1);
        x[5] = (float)exp(-r2);
        x[6] = mu == nu ? 1.f : 0.f;
        x[7] = (float)((rm + rn) * 0.5 / (double)nao);
    }
}

// D[mu][nu] = D[nu][mu] = Dcore[mu][nu] + y[p(mu,nu)]
__global__ void assemble_guess(const float* __restrict__ y, const double* __restrict__ Dc, int64_t nao,
                               double* __restrict__ D) {
    const int64_t nu = blockIdx.x;
    for (int64_t mu = threadIdx.x; mu <= nu; mu += blockDim.x) {
        const double v = Dc[mu * nao + nu] + (double)y[nu * (nu + 1) / 2 + mu];
        D[mu * nao + nu] = v;
        D[nu * nao + mu] = v;
    }
}

// t[p(mu,nu)] = D[mu][nu] - Dcore[mu][nu] for mu <= nu (FP32 training target)
__global__ void guess_target(const double* __restrict__ D, const double* __restrict__ Dc, int64_t nao,
                             float* __restrict__ t) {
    const int64_t nu = blockIdx.x;
    for (int64_t mu = threadIdx.x; mu <= nu; mu += blockDim.x)
        t[nu * (nu + 1) / 2 + mu] = (float)(D[mu * nao + nu] - Dc[mu * nao + nu]);
}

// One workgroup: out[0] = tr D (fixed-order sum), out[1] = number of
// non-finite entries of D.
__global__ __launch_bounds__(256) void guess_check(const double* __restrict__ D, int64_t nao,
                                                   double* __restrict__ out) {
    __shared__ double s_tr[256];
    __shared__ double s_bad[256];
    double tr = 0.0, bad = 0.0;
    for (int64_t e = threadIdx.x; e < nao * nao; e += 256) {
        const double v = D[e];
        if (!isfinite(v)) bad += 1.0;
        if (e / nao == e % nao) tr += v;
    }
    s_tr[threadIdx.x] = tr;
    s_bad[threadIdx.x] = bad;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            s_tr[threadIdx.x] += s_tr[threadIdx.x + w];
            s_bad[threadIdx.x] += s_bad[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = s_tr[0];
        out[1] = s_bad[0];
    }
}

// Y[r][:] = X[idx[r]][:] (rows of d FP32 values)
__global__ void gather_rows(const float* __restrict__ X, const int64_t* __restrict__ idx, int64_t n, int d,
                            float* __restrict__ Y) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * d) return;
    const int64_t r = e / d;
    Y[e] = X[idx[r] * d + (e - r * d)];
}

// Batch rows per partial sum of the weight gradient: at least kSlab and, while no FP32
// running sum gets longer than kMaxSlab rows for it, at most kMaxSlabs partials (a
// 256 x 256 gradient then has 4 x 128 workgroups at 65536 rows, two per CU, and
// 64 MB of partials up to 524288 rows).
constexpr int64_t kSlab = 512, kMaxSlab = 2048, kMaxSlabs = 256;
inline int64_t slab_of(int64_t n) {
    return std::min(std::max(kSlab, cdiv(cdiv(n, kMaxSlabs), 16) * 16), kMaxSlab);
}
// Most partials that any batch of up to n rows takes
inline int64_t max_slabs(int64_t n) { return std::max(std::min(cdiv(n, kSlab), kMaxSlabs), cdiv(n, kMaxSlab)); }
// Rows per workgroup of the row passes (head_grad, layer1_grad): about 1024
// workgroups, four per CU
constexpr int64_t kRowParts = 1024;
inline int64_t rows_of(int64_t n) { return std::max<int64_t>(16, cdiv(n, kRowParts)); }

}  // namespace
}  // namespace dfjk

struct dfjk_mlp_ctx {
    hipStream_t stream = nullptr;
    int d_in = 0, hidden = 0;
    int64_t max_batch = 0, nparam = 0;
    dfjk::DevBuf params, grads, m1, m2, act, part;
    int64_t step = 0;
    int compute = DFJK_F32;  // DFJK_BF16: hidden-layer products on the 16-bit matrix cores
    // parameter blocks inside `params` / `grads`
    int64_t oW1, ob1, oW2, ob2, oW3, ob3;
};

using namespace dfjk;

namespace {

struct Act {
    float *Z1, *A1, *Z2, *gZ2, *gZ1, *loss;
};

Act act_of(dfjk_mlp_ctx* m) {
    const int64_t nH = m->max_batch * m->hidden;
    float* b = static_cast<float*>(m->act.ptr);
    Act a;
    a.Z1 = b;
    a.A1 = b + nH;
    a.Z2 = b + 2 * nH;
    a.gZ2 = b + 3 * nH;
    a.gZ1 = b + 4 * nH;
    a.loss = b + 5 * nH;
    return a;
}

// Z2 of the batch (and Z1, A1 of the training pass)
int hidden_layers(dfjk_mlp_ctx* m, const float* X, int64_t n, Act& a, bool keep) {
    const hipStream_t st = m->stream;
    const float* P = static_cast<const float*>(m->params.ptr);
    const int H = m->hidden;
    layer1<<<dim3((unsigned)cdiv(n, 4 * kL1Rows), (unsigned)cdiv(H, 256)), 256, 0, st>>>(
        X, n, m->d_in, P + m->oW1, P + m->ob1, H, keep ? a.Z1 : nullptr, a.A1);
    DFJK_LAUNCH_CHECK("layer1");
    GemmEpi e;
    e.bias = P + m->ob2;
    return net_gemm(st, m->compute == DFJK_BF16, false, true, n, H, H, a.A1, H, P + m->oW2, H, a.Z2, H, 0,
                    EPI_BIAS, e);
}

int add_parts(dfjk_mlp_ctx* m, const float* part, int64_t np, int64_t ld, int64_t cols, float* out,
              float* loss = nullptr, double inv_n = 0.0) {
    sum_parts<<<dim3((unsigned)cdiv(cols + 1, 64)), 256, 0, m->stream>>>(part, np, ld, cols, out, loss, inv_n);
    DFJK_LAUNCH_CHECK("sum_parts");
    return DFJK_OK;
}

int check(const dfjk_mlp_ctx* m, int64_t n) {
    if (!m) {
        set_error("null MLP handle");
        return DFJK_E_INVALID;
    }
    if (n < 1 || n > m->max_batch) {
        set_error("batch of %lld rows outside [1, %lld]", (long long)n, (long long)m->max_batch);
        return DFJK_E_INVALID;
    }
    return DFJK_OK;
}

}  // namespace

extern "C" {

int dfjk_mlp_init(dfjk_mlp* out, int d_in, int hidden, int64_t max_batch, void* stream) {
    clear_error();
    if (!out || d_in < 1 || d_in > 64 || hidden < 16 || hidden > 1024 || max_batch < 1 ||
        max_batch > (int64_t(1) << 24)) {
        set_error("dfjk_mlp_init: sizes out of range");
        return DFJK_E_INVALID;
    }
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) {
        (void)hipGetLastError();
        set_error("dfjk_mlp_init: no HIP device available");
        return DFJK_E_NO_DEVICE;
    }
    dfjk_mlp_ctx* m = new (std::nothrow) dfjk_mlp_ctx();
    if (!m) {
        set_error("dfjk_mlp_init: host allocation failed");
        return DFJK_E_OOM;
    }
    m->stream = (hipStream_t)stream;
    m->d_in = d_in;
    m->hidden = hidden;
    m->max_batch = max_batch;
    const int64_t H = hidden;
    m->oW1 = 0;
    m->ob1 = m->oW1 + H * d_in;
    m->oW2 = m->ob1 + H;
    m->ob2 = m->oW2 + H * H;
    m->oW3 = m->ob2 + H;
    m->ob3 = m->oW3 + H;
    m->nparam = m->ob3 + 1;
    const size_t pb = sizeof(float) * (size_t)m->nparam;
    // partial sums: weight-gradient slabs, then the row passes' workgroups
    // (every batch up to max_batch takes at most as many)
    const int64_t nslab = max_slabs(max_batch);
    const int64_t nrow = std::min<int64_t>(cdiv(max_batch, 16), kRowParts);
    int rc;
    if ((rc = m->params.ensure(pb)) || (rc = m->grads.ensure(pb)) || (rc = m->m1.ensure(pb)) ||
        (rc = m->m2.ensure(pb)) ||
        (rc = m->act.ensure(sizeof(float) * (size_t)(5 * max_batch * H + 64))) ||
        (rc = m->part.ensure(sizeof(float) *
                             (size_t)std::max(nslab * H * H, nrow * (H * std::max<int64_t>(d_in + 1, 2) + 2))))) {
        dfjk_mlp_destroy(m);
        return rc;
    }
    *out = m;
    return DFJK_OK;
}

int64_t dfjk_mlp_nparam(dfjk_mlp m) { return m ? m->nparam : -1; }

int dfjk_mlp_set_params(dfjk_mlp m, const float* host) {
    clear_error();
    if (!m || !host) {
        set_error("dfjk_mlp_set_params: null argument");
        return DFJK_E_INVALID;
    }
    const size_t pb = sizeof(float) * (size_t)m->nparam;
    DFJK_HIP_TRY(hipMemcpy(m->params.ptr, host, pb, hipMemcpyHostToDevice));
    std::vector<float> zero((size_t)m->nparam, 0.f);
    DFJK_HIP_TRY(hipMemcpy(m->m1.ptr, zero.data(), pb, hipMemcpyHostToDevice));
    DFJK_HIP_TRY(hipMemcpy(m->m2.ptr, zero.data(), pb, hipMemcpyHostToDevice));
    m->step = 0;
    return DFJK_OK;
}

int dfjk_mlp_get(dfjk_mlp m, int which, float* host) {
    clear_error();
    if (!m || !host || which < 0 || which > 1) {
        set_error("dfjk_mlp_get: bad arguments");
        return DFJK_E_INVALID;
    }
    DFJK_HIP_TRY(hipStreamSynchronize(m->stream));
    DFJK_HIP_TRY(hipMemcpy(host, which == 0 ? m->params.ptr : m->grads.ptr,
                           sizeof(float) * (size_t)m->nparam, hipMemcpyDeviceToHost));
    return DFJK_OK;
}

int dfjk_mlp_forward(dfjk_mlp m, const float* X_dev, int64_t n, float* y_dev) {
    clear_error();
    if (int rc = check(m, n)) return rc;
    if (!X_dev || !y_dev) {
        set_error("dfjk_mlp_forward: null argument");
        return DFJK_E_INVALID;
    }
    Act a = act_of(m);
    if (int rc = hidden_layers(m, X_dev, n, a, false)) return rc;
    const float* P = static_cast<const float*>(m->params.ptr);
    head<<<dim3((unsigned)cdiv(n, 4)), 256, 0, m->stream>>>(a.Z2, P + m->oW3, P + m->ob3, n, m->hidden, y_dev);
    DFJK_LAUNCH_CHECK("head");
    return DFJK_OK;
}

int dfjk_mlp_loss_grad(dfjk_mlp m, const float* X, const float* t, int64_t n, float* loss_dev) {
    clear_error();
    if (int rc = check(m, n)) return rc;
    if (!X || !t) {
        set_error("dfjk_mlp_loss_grad: null argument");
        return DFJK_E_INVALID;
    }
    const hipStream_t st = m->stream;
    Act a = act_of(m);
    int rc;
    if ((rc = hidden_layers(m, X, n, a, true))) return rc;
    const int H = m->hidden, d = m->d_in;
    const float* P = static_cast<const float*>(m->params.ptr);
    float* G = static_cast<float*>(m->grads.ptr);
    float* part = static_cast<float*>(m->part.ptr);
    const bool bf = m->compute == DFJK_BF16;
    const int64_t per = rows_of(n), nrow = cdiv(n, per);
    // output layer: gradients of w3, b3 and b2, and gZ2 (the row passes'
    // registers hold hidden / 64 values per lane)
    if (H <= 256)
        head_grad<1><<<dim3((unsigned)nrow), 256, 0, st>>>(a.Z2, P + m->oW3, P + m->ob3, t, n, H, per, a.gZ2, part);
    else
        head_grad<4><<<dim3((unsigned)nrow), 256, 0, st>>>(a.Z2, P + m->oW3, P + m->ob3, t, n, H, per, a.gZ2, part);
    DFJK_LAUNCH_CHECK("head_grad");
    // b2, W3 and b3 lie one after the other in the parameters, as in the parts
    if ((rc = add_parts(m, part, nrow, 2 * H + 2, 2 * H + 1, G + m->ob2, a.loss, 1.0 / (double)n))) return rc;
    // layer 2
    const int64_t slab = slab_of(n);
    if ((rc = net_gemm(st, bf, true, false, H, H, n, a.gZ2, H, a.A1, H, part, H, slab))) return rc;
    if ((rc = add_parts(m, part, cdiv(n, slab), (int64_t)H * H, (int64_t)H * H, G + m->oW2))) return rc;
    // layer 1: gZ1 = (gZ2 W2) silu'(Z1), then its d_in columns
    GemmEpi e;
    e.Z = a.Z1;
    if ((rc = net_gemm(st, bf, false, false, n, H, H, a.gZ2, H, P + m->oW2, H, a.gZ1, H, 0, EPI_DSILU, e))) return rc;
    layer1_grad<<<dim3((unsigned)nrow, (unsigned)cdiv(H, 256)), 256, 0, st>>>(a.gZ1, X, n, H, d, per, part);
    DFJK_LAUNCH_CHECK("layer1_grad");
    // W1 and b1 lie one after the other in the parameters, as in the parts
    if ((rc = add_parts(m, part, nrow, (int64_t)H * d + H, (int64_t)H * d + H, G + m->oW1))) return rc;
    if (loss_dev)
        DFJK_HIP_TRY(hipMemcpyAsync(loss_dev, a.loss, sizeof(float), hipMemcpyDeviceToDevice, st));
    return DFJK_OK;
}

int dfjk_mlp_set_compute(dfjk_mlp m, int dtype) {
    clear_error();
    if (!m || (dtype != DFJK_F32 && dtype != DFJK_BF16)) {
        set_error("dfjk_mlp_set_compute: null handle or dtype other than DFJK_F32 / DFJK_BF16");
        return DFJK_E_INVALID;
    }
    m->compute = dtype;
    return DFJK_OK;
}

int dfjk_mlp_adam(dfjk_mlp m, float lr, float beta1, float beta2, float eps) {
    clear_error();
    if (!m || !(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) ||
        !(eps > 0.f)) {
        set_error("dfjk_mlp_adam: bad arguments");
        return DFJK_E_INVALID;
    }
    m->step += 1;
    const float c1 = 1.f - powf(beta1, (float)m->step), c2 = 1.f - powf(beta2, (float)m->step);
    adam_kernel<<<dim3((unsigned)cdiv(m->nparam, 256)), 256, 0, m->stream>>>(
        static_cast<float*>(m->params.ptr), static_cast<const float*>(m->grads.ptr),
        static_cast<float*>(m->m1.ptr), static_cast<float*>(m->m2.ptr), m->nparam, lr, beta1, beta2, eps,
        c1, c2);
    DFJK_LAUNCH_CHECK("adam_kernel");
    return DFJK_OK;
}

int dfjk_guess_features(const double* H, const double* Dcore, const double* R, int64_t nao, float* X,
                        void* stream) {
    clear_error();
    if (!H || !Dcore || !R || !X || nao < 1 || nao > 65535) {
        set_error("dfjk_guess_features: bad arguments");
        return DFJK_E_INVALID;
    }
    pair_features<<<dim3((unsigned)nao), 128, 0, (hipStream_t)stream>>>(H, Dcore, R, nao, X);
    DFJK_LAUNCH_CHECK("pair_features");
    return DFJK_OK;
}

int dfjk_guess_assemble(const float* y, const double* Dcore, int64_t nao, double* D, void* stream) {
    clear_error();
    if (!y || !Dcore || !D || nao < 1 || nao > 65535) {
        set_error("dfjk_guess_assemble: bad arguments");
        return DFJK_E_INVALID;
    }
    assemble_guess<<<dim3((unsigned)nao), 128, 0, (hipStream_t)stream>>>(y, Dcore, nao, D);
    DFJK_LAUNCH_CHECK("assemble_guess");
    return DFJK_OK;
}

int dfjk_guess_target(const double* D, const double* Dcore, int64_t nao, float* t, void* stream) {
    clear_error();
    if (!D || !Dcore || !t || nao < 1 || nao > 65535) {
        set_error("dfjk_guess_target: bad arguments");
        return DFJK_E_INVALID;
    }
    guess_target<<<dim3((unsigned)nao), 128, 0, (hipStream_t)stream>>>(D, Dcore, nao, t);
    DFJK_LAUNCH_CHECK("guess_target");
    return DFJK_OK;
}

int dfjk_guess_check(const double* D, int64_t nao, double* out, void* stream) {
    clear_error();
    if (!D || !out || nao < 1 || nao > 65535) {
        set_error("dfjk_guess_check: bad arguments");
        return DFJK_E_INVALID;
    }
    guess_check<<<1, 256, 0, (hipStream_t)stream>>>(D, nao, out);
    DFJK_LAUNCH_CHECK("guess_check");
    return DFJK_OK;
}

int dfjk_gather_rows(const float* X, const int64_t* idx, int64_t n, int d, float* Y, void* stream) {
    clear_error();
    if (!X || !idx || !Y || n < 0 || d < 1) {
        set_error("dfjk_gather_rows: bad arguments");
        return DFJK_E_INVALID;
    }
    if (n == 0) return DFJK_OK;
    gather_rows<<<dim3((unsigned)cdiv(n * d, 256)), 256, 0, (hipStream_t)stream>>>(X, idx, n, d, Y);
    DFJK_LAUNCH_CHECK("gather_rows");
    return DFJK_OK;
}

void dfjk_mlp_destroy(dfjk_mlp m) {
    if (!m) return;
    (void)hipStreamSynchronize(m->stream);
    m->params.release();
    m->grads.release();
    m->m1.release();
    m->m2.release();
    m->act.release();
    m->part.release();
    delete m;
}

}  // extern "C"
