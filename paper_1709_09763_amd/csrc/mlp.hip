// Learned surrogate theta -> G_l(theta): an MLP K -> H -> H -> N_obs with
// erf-GELU, trained on the GPU from (theta, G_l(theta)) pairs the sampler
// produces, and used as the first stage of delayed-acceptance pCN (two-stage
// Metropolis-Hastings: the surrogate screens proposals, the FEM solve judges
// the survivors).  Matrix products run on the CDNA4 matrix cores as BF16
// MFMA with FP32 accumulation; master weights and Adam moments are FP32.
#include <algorithm>
#include <cmath>
#include <numeric>
#include <random>

#include "common.h"

namespace mls {

typedef float flt4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// ------------------------------------------------------------------ GEMM --
// C[M x N] = sum_k A(m,k) B(k,n) with A(m,k) = TA ? A[k lda + m] : A[m lda + k]
// and B(k,n) = TB ? B[n ldb + k] : B[k ldb + n]; operands are rounded to
// BF16 as the fragments are loaded (v_mfma_f32_16x16x32_bf16 lanes: A rows
// lane%16, k = 8(lane/16)+0..7; B cols lane%16, same k; D[4(lane/16)+v][lane%16]).
// Epilogues: 0 store; 1 +bias, store Z to C and GELU(Z) to C2; 2 +bias;
// 3 multiply by GELU'(Zin[m][n]) (backward through the activation); 4 store,
// and (TA only) also write the row sums over k of A, sum_k A(m,k), to C2[m]:
// the bias gradient of a layer comes out of its weight-gradient product.
enum { EPI_STORE = 0, EPI_BIAS_GELU = 1, EPI_BIAS = 2, EPI_DGELU = 3, EPI_STORE_ASUM = 4 };

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float z)
{
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.3989422804014327f;
}

// Each wave owns one 16x16 tile of C, a workgroup 32x32.  The k loop loads
// the fragments of MLP_U consecutive 32-wide k steps before it issues their
// MFMAs, so one round of memory latency covers MLP_U steps (K <= 256 in the
// surrogate: at most two rounds).
constexpr int MLP_U = 4;

template <bool TA, bool TB, int EPI>
__global__ __launch_bounds__(256) void mlp_gemm(int M, int N, int K, const float* __restrict__ A, int lda,
                                                const float* __restrict__ B, int ldb,
                                                const float* __restrict__ bias, float* __restrict__ C,
                                                float* __restrict__ C2, const float* __restrict__ Zin,
                                                int ldc)
{
    static_assert(EPI != EPI_STORE_ASUM || TA, "row sums of A are taken for the transposed-A form");
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r = lane & 15, kq = lane >> 4;
    const int m0 = blockIdx.y * 32 + 16 * (wv >> 1);
    const int n0 = blockIdx.x * 32 + 16 * (wv & 1);
    const bool asum = EPI == EPI_STORE_ASUM && blockIdx.x == 0 && (wv & 1) == 0;
    flt4 acc = {0.f, 0.f, 0.f, 0.f};
    float rs = 0.f;
    const int am = m0 + r, bn = n0 + r;
    for (int k0 = 0; k0 < K; k0 += 32 * MLP_U) {
        bf16x8 a[MLP_U], b[MLP_U];
#pragma unroll
        for (int u = 0; u < MLP_U; ++u) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int k = k0 + 32 * u + 8 * kq + t;
                float av = 0.f, bv = 0.f;
                if (am < M && k < K) av = TA ? A[(int64_t)k * lda + am] : A[(int64_t)am * lda + k];
                if (bn < N && k < K) bv = TB ? B[(int64_t)bn * ldb + k] : B[(int64_t)k * ldb + bn];
                if (EPI == EPI_STORE_ASUM) rs += av;
                a[u][t] = (__bf16)av;
                b[u][t] = (__bf16)bv;
            }
        }
#pragma unroll
        for (int u = 0; u < MLP_U; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b[u], acc, 0, 0, 0);
    }
    if (EPI == EPI_STORE_ASUM) {
        // lanes r, r+16, r+32, r+48 hold the partial sums of row am
        rs += __shfl_xor(rs, 16);
        rs += __shfl_xor(rs, 32);
        if (asum && kq == 0 && am < M) C2[am] = rs;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int m = m0 + 4 * kq + v, n = n0 + r;
        if (m >= M || n >= N) continue;
        float z = acc[v];
        const int64_t o = (int64_t)m * ldc + n;
        if (EPI == EPI_BIAS_GELU) {
            z += bias[n];
            C[o] = z;
            C2[o] = gelu(z);
        } else if (EPI == EPI_BIAS) {
            C[o] = z + bias[n];
        } else if (EPI == EPI_DGELU) {
            C[o] = z * gelu_d(Zin[o]);
        } else {
            C[o] = z;
        }
    }
}

template <bool TA, bool TB, int EPI>
static int gemm(int M, int N, int K, const float* A, int lda, const float* B, int ldb, const float* bias,
                float* C, float* C2, const float* Zin, int ldc, hipStream_t s)
{
    if (M == 0 || N == 0) return MLS2MC_OK;
    dim3 grid((unsigned)((N + 31) / 32), (unsigned)((M + 31) / 32));
    mlp_gemm<TA, TB, EPI><<<grid, 256, 0, s>>>(M, N, K, A, lda, B, ldb, bias, C, C2, Zin, ldc);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// ------------------------------------------------------- small kernels --
// delta = (out - t) * scale, loss = scale * sum (out - t)^2 / 2 (one workgroup)
__global__ __launch_bounds__(1024) void loss_delta_kernel(int64_t n, const float* __restrict__ out,
                                                          const float* __restrict__ t, float scale,
                                                          float* __restrict__ delta, float* __restrict__ loss)
{
    __shared__ double red[16];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) {
        const float d = out[i] - t[i];
        delta[i] = d * scale;
        s += 0.5 * (double)d * (double)d;
    }
    s = block_sum<1024>(s, red);
    if (threadIdx.x == 0) loss[0] = (float)(s * scale);
}

// One Adam update; the contractions are spelled out so that every kernel
// rounds alike.
__device__ __forceinline__ float adam_update(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                                             int64_t i, float gi, float lr, float b1, float b2, float c1, float c2,
                                             float eps)
{
    const float mi = fmaf(1.f - b1, gi, b1 * m[i]);
    const float vi = fmaf(gi, (1.f - b2) * gi, b2 * v[i]);
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    return pi;
}

__global__ void adam_kernel(int64_t n, float* __restrict__ p, const float* __restrict__ g,
                            float* __restrict__ m, float* __restrict__ v, float lr, float b1, float b2,
                            float c1, float c2, float eps)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    (void)adam_update(p, m, v, i, g[i], lr, b1, b2, c1, c2, eps);
}

// rows idx[b] (or b) of a double matrix, standardised, to float
__global__ void standardize_kernel(int64_t B, int D, const int32_t* __restrict__ idx,
                                   const double* __restrict__ src, const float* __restrict__ mu,
                                   const float* __restrict__ sd, float* __restrict__ dst)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= B * D) return;
    const int64_t b = t / D;
    const int k = (int)(t - b * D);
    const int64_t row = idx ? idx[b] : b;
    const double v = src[row * D + k];
    dst[t] = mu ? (float)((v - (double)mu[k]) / (double)sd[k]) : (float)v;
}

__global__ void unstandardize_kernel(int64_t B, int O, const float* __restrict__ out,
                                     const float* __restrict__ mu, const float* __restrict__ sd,
                                     double* __restrict__ G)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= B * O) return;
    const int o = (int)(t % O);
    G[t] = (double)mu[o] + (double)sd[o] * (double)out[t];
}

// column mean and standard deviation of an n x D double matrix (one block per column)
__global__ __launch_bounds__(256) void col_stats_kernel(int64_t n, int D, const double* __restrict__ X,
                                                        float* __restrict__ mu, float* __restrict__ sd)
{
    __shared__ double red[4];
    const int k = blockIdx.x;
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) s += X[i * D + k];
    const double mean = block_sum<256>(s, red) / (double)n;
    double q = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double d = X[i * D + k] - mean;
        q += d * d;
    }
    const double var = block_sum<256>(q, red) / (double)n;
    if (threadIdx.x == 0) {
        mu[k] = (float)mean;
        sd[k] = (float)(var > 1e-30 ? sqrt(var) : 1.0);
    }
}

__global__ void f2d_kernel(int64_t n, const float* __restrict__ a, double* __restrict__ b)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) b[i] = (double)a[i];
}

__global__ void f2f_scaled_kernel(int64_t n, const double* __restrict__ z, float scale, float* __restrict__ out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] = scale * (float)z[i];
}

// ----------------------------------------------------------- surrogate --
struct Surrogate {
    int D = 0, H = 0, O = 0;
    int64_t np = 0;
    float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
    float *mu_x = nullptr, *sd_x = nullptr, *mu_y = nullptr, *sd_y = nullptr;
    int64_t adam_t = 0;
    bool standardized = false;
    // dataset ring
    int64_t cap = 0, count = 0, head = 0;
    double *ds_th = nullptr, *ds_G = nullptr;
    // activations for up to bmax rows
    int64_t bmax = 0;
    float *X = nullptr, *Z1 = nullptr, *H1 = nullptr, *Z2 = nullptr, *H2 = nullptr, *OUT = nullptr;
    float *T = nullptr, *D3 = nullptr, *D2 = nullptr, *D1 = nullptr, *loss = nullptr;
    int32_t* perm = nullptr;
    // fused path: BF16 copies of the weights as MFMA operands (null: the
    // layer-by-layer products), and the transposed batch for the weight
    // gradients (see MlpDims)
    __bf16* w16 = nullptr;
    char* tr = nullptr;
    int64_t tr_rows = 0;
    double* lossp = nullptr;
    float* W1() const { return p; }
    float* b1() const { return p + (int64_t)H * D; }
    float* W2() const { return b1() + H; }
    float* b2() const { return W2() + (int64_t)H * H; }
    float* W3() const { return b2() + H; }
    float* b3() const { return W3() + (int64_t)O * H; }
};

static void sur_free(Surrogate* S)
{
    void* ptrs[] = {S->p, S->g, S->m, S->v, S->mu_x, S->sd_x, S->mu_y, S->sd_y, S->ds_th, S->ds_G,
                    S->X, S->Z1, S->H1, S->Z2, S->H2, S->OUT, S->T, S->D3, S->D2, S->D1, S->loss, S->perm,
                    S->w16, S->tr, S->lossp};
    for (void* q : ptrs)
        if (q) (void)hipFree(q);
    *S = Surrogate();
}

void surrogate_destroy(mls2mc_ctx* ctx)
{
    if (ctx->sur) {
        sur_free(ctx->sur);
        delete ctx->sur;
        ctx->sur = nullptr;
    }
}

static int sur_ensure_batch(Surrogate* S, int64_t B)
{
    if (B <= S->bmax) return MLS2MC_OK;
    float** acts[] = {&S->X, &S->Z1, &S->H1, &S->Z2, &S->H2, &S->OUT, &S->T, &S->D3, &S->D2, &S->D1};
    for (float** a : acts)
        if (*a) { (void)hipFree(*a); *a = nullptr; }
    const int64_t w = std::max<int64_t>(std::max(S->D, S->H), S->O);
    for (float** a : acts) MLS_CHECK_HIP(hipMalloc(a, sizeof(float) * (size_t)B * w));
    S->bmax = B;
    return MLS2MC_OK;
}

// forward of B standardised rows in S->X; outputs in S->OUT (standardised)
static int sur_forward(Surrogate* S, int64_t B, hipStream_t s)
{
    const int D = S->D, H = S->H, O = S->O;
    MLS_TRY((gemm<false, true, EPI_BIAS_GELU>((int)B, H, D, S->X, D, S->W1(), D, S->b1(), S->Z1, S->H1, nullptr, H, s)));
    MLS_TRY((gemm<false, true, EPI_BIAS_GELU>((int)B, H, H, S->H1, H, S->W2(), H, S->b2(), S->Z2, S->H2, nullptr, H, s)));
    MLS_TRY((gemm<false, true, EPI_BIAS>((int)B, O, H, S->H2, H, S->W3(), H, S->b3(), S->OUT, nullptr, nullptr, O, s)));
    return MLS2MC_OK;
}

// gradient of mean (out - t)^2 / 2 w.r.t. all parameters into S->g; T holds targets
static int sur_backward(Surrogate* S, int64_t B, hipStream_t s)
{
    const int D = S->D, H = S->H, O = S->O;
    const float scale = 1.0f / (float)(B * O);
    loss_delta_kernel<<<1, 1024, 0, s>>>(B * O, S->OUT, S->T, scale, S->D3, S->loss);
    MLS_CHECK_HIP(hipGetLastError());
    float *gW1 = S->g, *gb1 = gW1 + (int64_t)H * D, *gW2 = gb1 + H, *gb2 = gW2 + (int64_t)H * H,
          *gW3 = gb2 + H, *gb3 = gW3 + (int64_t)O * H;
    // layer 3: dW3 = D3^T H2 and db3 = colsum D3 in one product; dH2 = D3 W3 (then * GELU'(Z2))
    MLS_TRY((gemm<true, false, EPI_STORE_ASUM>(O, H, (int)B, S->D3, O, S->H2, H, nullptr, gW3, gb3, nullptr, H, s)));
    MLS_TRY((gemm<false, false, EPI_DGELU>((int)B, H, O, S->D3, O, S->W3(), H, nullptr, S->D2, nullptr, S->Z2, H, s)));
    // layer 2
    MLS_TRY((gemm<true, false, EPI_STORE_ASUM>(H, H, (int)B, S->D2, H, S->H1, H, nullptr, gW2, gb2, nullptr, H, s)));
    MLS_TRY((gemm<false, false, EPI_DGELU>((int)B, H, H, S->D2, H, S->W2(), H, nullptr, S->D1, nullptr, S->Z1, H, s)));
    // layer 1
    MLS_TRY((gemm<true, false, EPI_STORE_ASUM>(H, D, (int)B, S->D1, H, S->X, D, nullptr, gW1, gb1, nullptr, D, s)));
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// ------------------------------------------------------ fused passes --
// A training step on 256 rows is 0.16 GFLOP, microseconds of the matrix
// cores; as twelve launches, each a chain of strided scalar loads, it took
// 172 us (100 -> 256 -> 256 -> 49).  Now 34: everything before the weight
// gradients is row-local, so one kernel (24 us; a chain of five layers'
// load latencies in 16 workgroups bounds it; with 512 threads 27 us) takes 16
// rows through standardisation, the three layers, the loss and the two
// backward products with the activations in LDS, and a second one (9 us)
// forms all weight gradients and applies Adam in their epilogue.
// Weights are read as BF16 copies (rounding the FP32 master as the fragments
// were loaded before gives the same operands), which every call that changes
// the parameters brings in line on its own stream: the initialisation, new
// parameters, the Adam epilogue.  A call that only reads them never has to, so
// a captured one replays with the parameters of the day.  The batch is handed
// over transposed, so every fragment is one or two 16-byte loads.  The MFMA tiles, their k order and the FP32 epilogues are
// those of mlp_gemm, so the parameters are bitwise the same.
struct MlpDims {
    int D, H, O;     // inputs, hidden width (a multiple of 16), outputs
    int Dp, Hp, Op;  // as k extents: padded to 32
    int Or;          // outputs as rows: padded to 16
    // element offsets of the BF16 copies: rows x padded k
    int64_t w1() const { return 0; }                         // H x Dp
    int64_t w2() const { return (int64_t)H * Dp; }           // H x Hp
    int64_t w3() const { return w2() + (int64_t)H * Hp; }    // Or x Hp
    int64_t w2t() const { return w3() + (int64_t)Or * Hp; }  // H x Hp
    int64_t w3t() const { return w2t() + (int64_t)H * Hp; }  // H x Op
    int64_t total() const { return w3t() + (int64_t)H * Op; }
    // bytes of LDS of the row kernel: X, H1, H2 (later D2), D3 in BF16 rows
    // padded against bank conflicts, Z1 and Z2 in FP32, the loss partials
    size_t lds() const
    {
        return 2 * 16 * (size_t)(Dp + 8 + 2 * (Hp + 8) + Op + 8) + 2 * 4 * 16 * (size_t)H + 64;
    }
};
static MlpDims mlp_dims(const Surrogate* S)
{
    auto up = [](int x, int m) { return (x + m - 1) / m * m; };
    return {S->D, S->H, S->O, up(S->D, 32), up(S->H, 32), up(S->O, 32), up(S->O, 16)};
}

struct MlpRows {
    int D, H, O, Dp, Hp, Op, Or;
    const __bf16 *w1, *w2, *w3, *w2t, *w3t;
    const float *b1, *b2, *b3;
    int64_t B, Bp;           // rows, and padded to 32 (the batch's k extent)
    const int32_t* idx;      // rows of th and G (null: 0 .. B - 1)
    const double *th, *G;    // inputs, targets (G: outputs in a prediction)
    const float *mux, *sdx, *muy, *sdy;  // standardisation, or null
    double* out;             // prediction: B x O
    float scale;
    __bf16 *xt, *h1t, *h2t;  // training: features x Bp
    float *d3t, *d2t, *d1t;
    double* lossp;           // per workgroup
};

// C[16 x 16 tile n0] = A (LDS, 16 rows of lda) x W^T (rows n0 .. n0+15 of Kp)
__device__ __forceinline__ flt4 row_tile(const __bf16* a, int lda, const __bf16* __restrict__ w, int Kp, int n0)
{
    const int lane = threadIdx.x & 63, r = lane & 15, kq = lane >> 4;
    const bf16x8* ap = reinterpret_cast<const bf16x8*>(a + r * lda + 8 * kq);
    const bf16x8* wp = reinterpret_cast<const bf16x8*>(w + (int64_t)(n0 + r) * Kp + 8 * kq);
    flt4 acc = {0.f, 0.f, 0.f, 0.f};
    int k = 0;
    for (; k + 8 <= Kp / 32; k += 8) {  // a round of loads in flight, then its MFMAs
        bf16x8 wf[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) wf[u] = wp[4 * (k + u)];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[4 * (k + u)], wf[u], acc, 0, 0, 0);
    }
    for (; k + 2 <= Kp / 32; k += 2) {
        const bf16x8 w0 = wp[4 * k], w1 = wp[4 * k + 4];
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[4 * k], w0, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[4 * k + 4], w1, acc, 0, 0, 0);
    }
    for (; k < Kp / 32; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[4 * k], wp[4 * k], acc, 0, 0, 0);
    return acc;
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store4(float* p, const float (&v)[4])
{
    *reinterpret_cast<flt4*>(p) = flt4{v[0], v[1], v[2], v[3]};
}
__device__ __forceinline__ void store4(__bf16* p, const float (&v)[4])
{
    *reinterpret_cast<bf16x4*>(p) = bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
}

extern __shared__ __align__(16) char mlp_lds[];

constexpr int kRowThreads = 1024;
template <bool TRAIN>
__global__ __launch_bounds__(kRowThreads) void mlp_rows_kernel(MlpRows P)
{
    __shared__ double red[kRowThreads / 64];
    const int ldx = P.Dp + 8, ldh = P.Hp + 8, ldo = P.Op + 8;
    __bf16* X = reinterpret_cast<__bf16*>(mlp_lds);
    __bf16* H1 = X + 16 * ldx;
    __bf16* H2 = H1 + 16 * ldh;  // D2 in the backward products
    __bf16* D3 = H2 + 16 * ldh;
    float* Z1 = reinterpret_cast<float*>(D3 + 16 * ldo);
    float* Z2 = Z1 + 16 * P.H;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r = lane & 15, kq = lane >> 4;
    constexpr int NW = kRowThreads / 64;
    const int64_t b0 = blockIdx.x * (int64_t)16;
    // standardised inputs; the padded k columns and rows past the batch are zero
    for (int q = tid; q < 16 * P.Dp; q += kRowThreads) {
        const int row = q / P.Dp, k = q - row * P.Dp;
        float x = 0.f;
        if (b0 + row < P.B && k < P.D) {
            const int64_t src = P.idx ? P.idx[b0 + row] : b0 + row;
            const double v = P.th[src * P.D + k];
            x = P.mux ? (float)((v - (double)P.mux[k]) / (double)P.sdx[k]) : (float)v;
        }
        X[row * ldx + k] = (__bf16)x;
    }
    for (int q = tid; q < 16 * (P.Hp - P.H); q += kRowThreads) {
        const int row = q / (P.Hp - P.H), k = P.H + q % (P.Hp - P.H);
        H1[row * ldh + k] = H2[row * ldh + k] = (__bf16)0.f;
    }
    if (TRAIN)
        for (int q = tid; q < 16 * P.Op; q += kRowThreads) D3[(q / P.Op) * ldo + q % P.Op] = (__bf16)0.f;
    __syncthreads();
    if (TRAIN)
        for (int q = tid; q < 2 * P.D; q += kRowThreads) {  // X transposed, eight rows per store
            const int k = q >> 1, row = 8 * (q & 1);
            bf16x8 v;
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = X[(row + u) * ldx + k];
            *reinterpret_cast<bf16x8*>(P.xt + k * P.Bp + b0 + row) = v;
        }
    auto hidden = [&](const __bf16* a, int lda, const __bf16* w, int Kp, const float* b, float* Z, __bf16* Hout,
                      __bf16* ht) {
        for (int n0 = 16 * wv; n0 < P.H; n0 += 16 * NW) {
            const flt4 acc = row_tile(a, lda, w, Kp, n0);
            const int n = n0 + r;
            float h[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float z = acc[v];
                z += b[n];
                h[v] = gelu(z);
                if (TRAIN) Z[(4 * kq + v) * P.H + n] = z;
                Hout[(4 * kq + v) * ldh + n] = (__bf16)h[v];
            }
            if (TRAIN) store4(ht + n * P.Bp + b0 + 4 * kq, h);
        }
        __syncthreads();
    };
    hidden(X, ldx, P.w1, P.Dp, P.b1, Z1, H1, P.h1t);
    hidden(H1, ldh, P.w2, P.Hp, P.b2, Z2, H2, P.h2t);
    double loss = 0.0;
    for (int n0 = 16 * wv; n0 < P.Or; n0 += 16 * NW) {
        const flt4 acc = row_tile(H2, ldh, P.w3, P.Hp, n0);
        const int n = n0 + r;
        if (n >= P.O) continue;
        float d3[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t row = b0 + 4 * kq + v;
            const float o = acc[v] + P.b3[n];
            d3[v] = 0.f;
            if (row < P.B) {
                if (TRAIN) {
                    const int64_t src = P.idx ? P.idx[row] : row;
                    const double g = P.G[src * P.O + n];
                    const float t = P.muy ? (float)((g - (double)P.muy[n]) / (double)P.sdy[n]) : (float)g;
                    const float d = o - t;
                    d3[v] = d * P.scale;
                    loss += 0.5 * (double)d * (double)d;
                } else {
                    P.out[row * P.O + n] = P.muy ? (double)P.muy[n] + (double)P.sdy[n] * (double)o : (double)o;
                }
            }
            if (TRAIN) D3[(4 * kq + v) * ldo + n] = (__bf16)d3[v];
        }
        if (TRAIN) store4(P.d3t + n * P.Bp + b0 + 4 * kq, d3);
    }
    if (!TRAIN) return;
    loss = block_sum<kRowThreads>(loss, red);  // its barriers end the layer
    if (tid == 0) P.lossp[blockIdx.x] = loss;
    auto backward = [&](const __bf16* a, int lda, const __bf16* w, int Kp, const float* Z, __bf16* Dout, float* dt) {
        for (int n0 = 16 * wv; n0 < P.H; n0 += 16 * NW) {
            const flt4 acc = row_tile(a, lda, w, Kp, n0);
            const int n = n0 + r;
            float d[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                d[v] = acc[v] * gelu_d(Z[(4 * kq + v) * P.H + n]);
                if (Dout) Dout[(4 * kq + v) * ldh + n] = (__bf16)d[v];
            }
            store4(dt + n * P.Bp + b0 + 4 * kq, d);
        }
    };
    backward(D3, ldo, P.w3t, P.Op, Z2, H2, P.d2t);
    __syncthreads();
    backward(H2, ldh, P.w2t, P.Hp, Z1, nullptr, P.d1t);
}

// Weight gradients dW = D^T H of the three layers and the bias gradients
// (row sums of D^T), one 16 x 16 tile per wave, with the Adam update and the
// refreshed BF16 copies in the epilogue (ADAM), or stored to g.
struct MlpGrad {
    int M[3], N[3];                       // outs x ins per layer
    int tiles[3], tn[3];                  // 16 x 16 tiles, tiles per row
    const float* dt[3];                   // M x Bp
    const __bf16* ht[3];                  // N x Bp
    int64_t w[3], b[3];                   // parameter offsets
    __bf16* c[3];                         // BF16 copy, M x ldc
    __bf16* ct[3];                        // transposed copy, N x ldt (or null)
    int ldc[3], ldt[3];
    int64_t Bp;
    float *p, *m, *v, *g;
    float lr, b1, b2, c1, c2, eps;
};

template <bool ADAM>
__global__ __launch_bounds__(256) void mlp_grad_kernel(MlpGrad P)
{
    int t = blockIdx.x * 4 + (threadIdx.x >> 6), l = 0;
    while (l < 3 && t >= P.tiles[l]) t -= P.tiles[l++];
    if (l == 3) return;
    const int lane = threadIdx.x & 63, r = lane & 15, kq = lane >> 4;
    const int M = P.M[l], N = P.N[l];
    const int m0 = 16 * (t / P.tn[l]), n0 = 16 * (t % P.tn[l]);
    const int am = m0 + r, bn = n0 + r;
    // rows past the layer's sizes repeat the last one; their products are not stored
    const float* dp = P.dt[l] + (int64_t)(am < M ? am : M - 1) * P.Bp + 8 * kq;
    const __bf16* hp = P.ht[l] + (int64_t)(bn < N ? bn : N - 1) * P.Bp + 8 * kq;
    flt4 acc = {0.f, 0.f, 0.f, 0.f};
    float rs = 0.f;
    for (int64_t k0 = 0; k0 < P.Bp; k0 += 128) {
        flt4 a0[4], a1[4];
        bf16x8 b[4];
        const int nu = P.Bp - k0 < 128 ? (int)(P.Bp - k0) / 32 : 4;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (u < nu) {
                a0[u] = *reinterpret_cast<const flt4*>(dp + k0 + 32 * u);
                a1[u] = *reinterpret_cast<const flt4*>(dp + k0 + 32 * u + 4);
                b[u] = *reinterpret_cast<const bf16x8*>(hp + k0 + 32 * u);
            }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (u < nu) {
                bf16x8 a;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    a[q] = (__bf16)a0[u][q];
                    a[4 + q] = (__bf16)a1[u][q];
                }
                if (n0 == 0) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) rs += a0[u][q];
#pragma unroll
                    for (int q = 0; q < 4; ++q) rs += a1[u][q];
                }
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[u], acc, 0, 0, 0);
            }
    }
    auto step = [&](int64_t i, float gi) {
        return adam_update(P.p, P.m, P.v, i, gi, P.lr, P.b1, P.b2, P.c1, P.c2, P.eps);
    };
    if (n0 == 0) {
        rs += __shfl_xor(rs, 16);
        rs += __shfl_xor(rs, 32);
        if (kq == 0 && am < M) {
            if (ADAM) (void)step(P.b[l] + am, rs);
            else P.g[P.b[l] + am] = rs;
        }
    }
    const int n = n0 + r;
    if (n >= N) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int m = m0 + 4 * kq + v;
        if (m >= M) continue;
        const int64_t i = P.w[l] + (int64_t)m * N + n;
        if (ADAM) {
            const __bf16 w = (__bf16)step(i, acc[v]);
            P.c[l][(int64_t)m * P.ldc[l] + n] = w;
            if (P.ct[l]) P.ct[l][(int64_t)n * P.ldt[l] + m] = w;
        } else {
            P.g[i] = acc[v];
        }
    }
}

// the BF16 copies of a layer's M x N weights
__global__ void mlp_copy_kernel(int M, int N, const float* __restrict__ w, __bf16* __restrict__ c, int ldc,
                                __bf16* __restrict__ ct, int ldt)
{
    const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (i >= (int64_t)M * N) return;
    const int m = (int)(i / N), n = (int)(i - (int64_t)m * N);
    const __bf16 v = (__bf16)w[i];
    c[(int64_t)m * ldc + n] = v;
    if (ct) ct[(int64_t)n * ldt + m] = v;
}

__global__ void zero16_kernel(int64_t n, __bf16* __restrict__ p)
{
    const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (i < n) p[i] = (__bf16)0.f;
}

__global__ __launch_bounds__(256) void loss_sum_kernel(int n, const double* __restrict__ part, float scale,
                                                       float* __restrict__ loss)
{
    __shared__ double red[4];
    double s = 0.0;
    for (int k = threadIdx.x; k < n; k += 256) s += part[k];
    s = block_sum<256>(s, red);
    if (threadIdx.x == 0) loss[0] = (float)(s * scale);
}

// The row kernel's LDS must fit beside its static array; wider networks keep
// the layer-by-layer products.
static bool mlp_fits(const mls2mc_ctx* ctx) { return mlp_dims(ctx->sur).lds() <= (size_t)ctx->max_lds; }

// the BF16 copies of the parameters, made anew (a network of the layer-by-layer
// products has none)
static int mlp_copies(const Surrogate* S, hipStream_t s)
{
    if (!S->w16) return MLS2MC_OK;
    const MlpDims d = mlp_dims(S);
    auto copy = [&](int M, int N, const float* w, int64_t c, int ldc, int64_t ct, int ldt) {
        mlp_copy_kernel<<<(unsigned)(((int64_t)M * N + 255) / 256), 256, 0, s>>>(M, N, w, S->w16 + c, ldc,
                                                                                ct >= 0 ? S->w16 + ct : nullptr, ldt);
    };
    copy(d.H, d.D, S->W1(), d.w1(), d.Dp, -1, 0);
    copy(d.H, d.H, S->W2(), d.w2(), d.Hp, d.w2t(), d.Hp);
    copy(d.O, d.H, S->W3(), d.w3(), d.Hp, d.w3t(), d.Op);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

static MlpRows mlp_rows(const Surrogate* S, int64_t B)
{
    const MlpDims d = mlp_dims(S);
    MlpRows P = {};
    P.D = d.D; P.H = d.H; P.O = d.O; P.Dp = d.Dp; P.Hp = d.Hp; P.Op = d.Op; P.Or = d.Or;
    P.w1 = S->w16 + d.w1(); P.w2 = S->w16 + d.w2(); P.w3 = S->w16 + d.w3();
    P.w2t = S->w16 + d.w2t(); P.w3t = S->w16 + d.w3t();
    P.b1 = S->b1(); P.b2 = S->b2(); P.b3 = S->b3();
    P.B = B;
    P.Bp = (B + 31) / 32 * 32;
    return P;
}

// loss and gradient of B rows of the training arrays: into the parameters
// (an Adam step) or into S->g
static int mlp_step(Surrogate* S, int64_t B, const int32_t* idx, const double* th, const double* G, bool standardise,
                    bool adam, float lr, float b1, float b2, float c1, float c2, float eps, hipStream_t s)
{
    const MlpDims d = mlp_dims(S);
    MlpRows P = mlp_rows(S, B);
    if (S->tr_rows < P.Bp) {
        if (S->tr) MLS_CHECK_HIP(hipFree(S->tr));
        if (S->lossp) MLS_CHECK_HIP(hipFree(S->lossp));
        S->tr = nullptr;
        S->lossp = nullptr;
        S->tr_rows = 0;
        MLS_CHECK_HIP(hipMalloc(&S->tr, (size_t)P.Bp * (4 * (2 * d.H + d.O) + 2 * (2 * d.H + d.D))));
        MLS_CHECK_HIP(hipMalloc(&S->lossp, sizeof(double) * (size_t)(P.Bp / 16)));
        S->tr_rows = P.Bp;
    }
    P.d3t = reinterpret_cast<float*>(S->tr);
    P.d2t = P.d3t + d.O * P.Bp;
    P.d1t = P.d2t + d.H * P.Bp;
    P.h1t = reinterpret_cast<__bf16*>(P.d1t + d.H * P.Bp);
    P.h2t = P.h1t + d.H * P.Bp;
    P.xt = P.h2t + d.H * P.Bp;
    P.lossp = S->lossp;
    P.idx = idx; P.th = th; P.G = G;
    if (standardise) { P.mux = S->mu_x; P.sdx = S->sd_x; P.muy = S->mu_y; P.sdy = S->sd_y; }
    P.scale = 1.0f / (float)(B * d.O);
    const unsigned wg = (unsigned)(P.Bp / 16);
    mlp_rows_kernel<true><<<wg, kRowThreads, d.lds(), s>>>(P);
    MLS_CHECK_HIP(hipGetLastError());
    MlpGrad g = {};
    const int Ms[3] = {d.H, d.H, d.O}, Ns[3] = {d.D, d.H, d.H};
    const float* dts[3] = {P.d1t, P.d2t, P.d3t};
    const __bf16* hts[3] = {P.xt, P.h1t, P.h2t};
    const float *ws[3] = {S->W1(), S->W2(), S->W3()}, *bs[3] = {S->b1(), S->b2(), S->b3()};
    __bf16* cs[3] = {S->w16 + d.w1(), S->w16 + d.w2(), S->w16 + d.w3()};
    __bf16* cts[3] = {nullptr, S->w16 + d.w2t(), S->w16 + d.w3t()};
    int tiles = 0;
    for (int l = 0; l < 3; ++l) {
        g.M[l] = Ms[l]; g.N[l] = Ns[l];
        g.tn[l] = (Ns[l] + 15) / 16;
        g.tiles[l] = g.tn[l] * ((Ms[l] + 15) / 16);
        g.dt[l] = dts[l]; g.ht[l] = hts[l];
        g.w[l] = ws[l] - S->p; g.b[l] = bs[l] - S->p;
        g.c[l] = cs[l]; g.ct[l] = cts[l];
        g.ldc[l] = l == 0 ? d.Dp : d.Hp;
        g.ldt[l] = l == 1 ? d.Hp : d.Op;
        tiles += g.tiles[l];
    }
    g.Bp = P.Bp;
    g.p = S->p; g.m = S->m; g.v = S->v; g.g = S->g;
    g.lr = lr; g.b1 = b1; g.b2 = b2; g.c1 = c1; g.c2 = c2; g.eps = eps;
    if (adam) mlp_grad_kernel<true><<<(tiles + 3) / 4, 256, 0, s>>>(g);
    else mlp_grad_kernel<false><<<(tiles + 3) / 4, 256, 0, s>>>(g);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// the loss of the last mlp_step on B rows into S->loss
static int mlp_loss(Surrogate* S, int64_t B, hipStream_t s)
{
    loss_sum_kernel<<<1, 256, 0, s>>>((int)((B + 31) / 32 * 2), S->lossp, 1.0f / (float)(B * S->O), S->loss);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

// ------------------------------------------------ delayed acceptance --
// stage-1 potential of the surrogate: beta * Phi(G~)
__global__ void da_psis_kernel(int64_t N, int nobs, const double* __restrict__ Gs, const double* __restrict__ y,
                               double inv_sigma, double beta, double* __restrict__ psis)
{
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= N) return;
    double s = 0.0;
    for (int o = 0; o < nobs; ++o) {
        const double r = (y[o] - Gs[j * nobs + o]) * inv_sigma;
        s += r * r;
    }
    psis[j] = beta * 0.5 * s;
}

// Stage 1 and compaction in one workgroup: thread k owns the contiguous chunk
// [k N / BS, (k+1) N / BS); survivors keep their ascending order in idx.
__global__ __launch_bounds__(1024) void da_stage1_kernel(int64_t N, const double* __restrict__ u1,
                                                         const double* __restrict__ ps_old,
                                                         const double* __restrict__ ps_new,
                                                         int32_t* __restrict__ idx, int64_t* __restrict__ count,
                                                         uint8_t* __restrict__ acc, uint8_t* __restrict__ pass1,
                                                         int64_t* __restrict__ n_lo, int64_t* __restrict__ n_hi)
{
    __shared__ int64_t part[1024];
    const int64_t lo = (int64_t)threadIdx.x * N / 1024, hi = (int64_t)(threadIdx.x + 1) * N / 1024;
    int64_t c = 0;
    for (int64_t j = lo; j < hi; ++j) {
        const bool s1 = log(u1[j]) < -(ps_new[j] - ps_old[j]);
        c += s1 ? 1 : 0;
        acc[j] = 0;
        if (pass1) pass1[j] = s1 ? 1 : 0;
    }
    part[threadIdx.x] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t a = 0;
        for (int k = 0; k < 1024; ++k) {
            const int64_t v = part[k];
            part[k] = a;
            a += v;
        }
        count[0] = a;
        if (n_lo) n_lo[0] += a;
        if (n_hi) n_hi[0] += a;
    }
    __syncthreads();
    int64_t o = part[threadIdx.x];
    for (int64_t j = lo; j < hi; ++j)
        if (log(u1[j]) < -(ps_new[j] - ps_old[j])) idx[o++] = (int32_t)j;
}

__global__ void gather_count_kernel(int64_t N, int ncols, const int32_t* __restrict__ idx,
                                    const int64_t* __restrict__ count, const double* __restrict__ src,
                                    double* __restrict__ dst)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t c = t / ncols;
    if (c >= N || c >= count[0]) return;
    const int k = (int)(t - c * ncols);
    dst[t] = src[(int64_t)idx[c] * ncols + k];
}

// Error of the surrogate against the FEM solve that judges it in stage 2:
// e_c = ||G~(theta'_j) - G(theta'_j)||_2 / sigma_n for the survivors c <
// count (j = idx[c]); acc[0] += sum e, acc[1] = max(acc[1], max e),
// acc[2] += number of survivors.  One workgroup, deterministic sums.
__global__ __launch_bounds__(256) void da_err_kernel(int64_t N, const int64_t* __restrict__ count,
                                                     const int32_t* __restrict__ idx, int nobs,
                                                     const double* __restrict__ Gs, const double* __restrict__ Gf,
                                                     double inv_sigma, double* __restrict__ acc)
{
    __shared__ double red[4];
    const int64_t n = count[0] < N ? count[0] : N;
    double sum = 0.0, mx = 0.0;
    for (int64_t c = threadIdx.x; c < n; c += 256) {
        const int64_t j = idx[c];
        double e2 = 0.0;
        for (int o = 0; o < nobs; ++o) {
            const double d = Gs[j * nobs + o] - Gf[c * nobs + o];
            e2 += d * d;
        }
        const double e = sqrt(e2) * inv_sigma;
        sum += e;
        mx = fmax(mx, e);
    }
    sum = block_sum<256>(sum, red);
    mx = block_max<256>(mx, red);
    if (threadIdx.x == 0) {
        acc[0] += sum;
        acc[1] = fmax(acc[1], mx);
        acc[2] += (double)n;
    }
}

// stage 2 for the survivors: Psi of the FEM solve corrected by the surrogate
__global__ void da_stage2_kernel(int64_t N, const int64_t* __restrict__ count, const int32_t* __restrict__ idx,
                                 int K, int nobs, int mode, double beta, double zeta,
                                 const double* __restrict__ u2, const double* __restrict__ ps_old,
                                 const double* __restrict__ ps_new, const double* __restrict__ thn,
                                 const double* __restrict__ Gcl, const double* __restrict__ Gch,
                                 const double* __restrict__ pcl, const double* __restrict__ pch,
                                 const int8_t* __restrict__ stl, const int8_t* __restrict__ sth,
                                 double* __restrict__ th, double* __restrict__ Gl, double* __restrict__ Gh,
                                 double* __restrict__ pl, double* __restrict__ ph, uint8_t* __restrict__ acc)
{
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= N || c >= count[0]) return;
    const int64_t j = idx[c];
    const bool need_lo = mode != 2, need_hi = mode != 0;
    double po, pn;
    if (mode == 0) {
        po = beta * pl[j];
        pn = beta * pcl[c];
    } else if (mode == 1) {
        po = beta * ((1.0 - zeta) * pl[j] + zeta * ph[j]);
        pn = beta * ((1.0 - zeta) * pcl[c] + zeta * pch[c]);
    } else {
        po = beta * ph[j];
        pn = beta * pch[c];
    }
    bool ok = true;
    if (need_lo && stl[c] != 0) ok = false;
    if (need_hi && sth[c] != 0) ok = false;
    const bool a = ok && (log(u2[j]) < -(pn - po) + (ps_new[j] - ps_old[j]));
    if (!a) return;
    for (int k = 0; k < K; ++k) th[j * K + k] = thn[j * K + k];
    if (need_lo) {
        for (int o = 0; o < nobs; ++o) Gl[j * nobs + o] = Gcl[c * nobs + o];
        pl[j] = pcl[c];
    }
    if (need_hi) {
        for (int o = 0; o < nobs; ++o) Gh[j * nobs + o] = Gch[c * nobs + o];
        ph[j] = pch[c];
    }
    acc[j] = 1;
}

}  // namespace mls

using namespace mls;

extern "C" {

int mls2mc_surrogate_init(mls2mc_ctx* ctx, int hidden, int64_t capacity, uint64_t seed, void* stream)
{
    MLS_REQUIRE(ctx != nullptr, "null context");
    MLS_REQUIRE(hidden >= 16 && hidden <= 1024 && hidden % 16 == 0, "surrogate_init: hidden must be a multiple of 16 in [16, 1024]");
    MLS_REQUIRE(capacity >= 1 && capacity <= (int64_t(1) << 24), "surrogate_init: capacity in [1, 2^24]");
    const hipStream_t s = (hipStream_t)stream;
    surrogate_destroy(ctx);
    ctx->sur = new Surrogate();
    Surrogate* S = ctx->sur;
    S->D = ctx->prob.K;
    S->H = hidden;
    S->O = ctx->nobs;
    const int D = S->D, H = S->H, O = S->O;
    S->np = (int64_t)H * D + H + (int64_t)H * H + H + (int64_t)O * H + O;
    for (float** a : {&S->p, &S->g, &S->m, &S->v}) MLS_CHECK_HIP(hipMalloc(a, sizeof(float) * S->np));
    for (float** a : {&S->mu_x, &S->sd_x}) MLS_CHECK_HIP(hipMalloc(a, sizeof(float) * D));
    for (float** a : {&S->mu_y, &S->sd_y}) MLS_CHECK_HIP(hipMalloc(a, sizeof(float) * O));
    MLS_CHECK_HIP(hipMalloc(&S->loss, sizeof(float) * 4));
    S->cap = capacity;
    MLS_CHECK_HIP(hipMalloc(&S->ds_th, sizeof(double) * (size_t)capacity * D));
    MLS_CHECK_HIP(hipMalloc(&S->ds_G, sizeof(double) * (size_t)capacity * O));
    MLS_CHECK_HIP(hipMalloc(&S->perm, sizeof(int32_t) * (size_t)capacity));
    // He initialisation from Philox normals; zero biases and moments
    MLS_CHECK_HIP(hipMemsetAsync(S->p, 0, sizeof(float) * S->np, s));
    MLS_CHECK_HIP(hipMemsetAsync(S->m, 0, sizeof(float) * S->np, s));
    MLS_CHECK_HIP(hipMemsetAsync(S->v, 0, sizeof(float) * S->np, s));
    DevBuf z;
    MLS_TRY(z.ensure(sizeof(double) * (size_t)std::max<int64_t>((int64_t)H * std::max(D, H), (int64_t)O * H)));
    struct { float* w; int64_t n; int fan; } L[3] = {{S->W1(), (int64_t)H * D, D}, {S->W2(), (int64_t)H * H, H},
                                                      {S->W3(), (int64_t)O * H, H}};
    for (int q = 0; q < 3; ++q) {
        MLS_TRY(launch_philox(seed, 7, 0, (uint32_t)q, L[q].n, 1, z.as<double>(), s));
        f2f_scaled_kernel<<<(unsigned)((L[q].n + 255) / 256), 256, 0, s>>>(L[q].n, z.as<double>(),
                                                                         std::sqrt(2.0f / L[q].fan), L[q].w);
        MLS_CHECK_HIP(hipGetLastError());
    }
    if (mlp_fits(ctx)) {  // the padding of the copies stays zero
        const int64_t n16 = mlp_dims(S).total();
        MLS_CHECK_HIP(hipMalloc(&S->w16, sizeof(__bf16) * (size_t)n16));
        zero16_kernel<<<(unsigned)((n16 + 255) / 256), 256, 0, s>>>(n16, S->w16);
        MLS_TRY(mlp_copies(S, s));
    }
    MLS_CHECK_HIP(hipStreamSynchronize(s));
    z.release();
    return MLS2MC_OK;
}

int mls2mc_surrogate_n_params(const mls2mc_ctx* ctx)
{
    return (ctx && ctx->sur) ? (int)ctx->sur->np : -1;
}

int mls2mc_surrogate_set_params(mls2mc_ctx* ctx, const float* params, void* stream)
{
    MLS_REQUIRE(ctx && ctx->sur && params, "surrogate_set_params: no surrogate or null pointer");
    MLS_CHECK_HIP(hipMemcpyAsync(ctx->sur->p, params, sizeof(float) * ctx->sur->np, hipMemcpyDeviceToDevice,
                                 (hipStream_t)stream));
    return mlp_copies(ctx->sur, (hipStream_t)stream);
}

int mls2mc_surrogate_get_params(mls2mc_ctx* ctx, float* params, void* stream)
{
    MLS_REQUIRE(ctx && ctx->sur && params, "surrogate_get_params: no surrogate or null pointer");
    MLS_CHECK_HIP(hipMemcpyAsync(params, ctx->sur->p, sizeof(float) * ctx->sur->np, hipMemcpyDeviceToDevice,
                                 (hipStream_t)stream));
    return MLS2MC_OK;
}

int mls2mc_surrogate_add_pairs(mls2mc_ctx* ctx, int64_t n, const double* theta, const double* G, void* stream)
{
    MLS_REQUIRE(ctx && ctx->sur, "surrogate_add_pairs: call mls2mc_surrogate_init first");
    MLS_REQUIRE(n >= 0, "surrogate_add_pairs: n < 0");
    if (n == 0) return MLS2MC_OK;
    MLS_REQUIRE(theta && G, "surrogate_add_pairs: null pointer");
    Surrogate* S = ctx->sur;
    const hipStream_t s = (hipStream_t)stream;
    if (n > S->cap) {  // keep the last cap pairs
        theta += (n - S->cap) * S->D;
        G += (n - S->cap) * S->O;
        n = S->cap;
    }
    int64_t done = 0;
    while (done < n) {
        const int64_t k = std::min(n - done, S->cap - S->head);
        MLS_CHECK_HIP(hipMemcpyAsync(S->ds_th + S->head * S->D, theta + done * S->D, sizeof(double) * k * S->D,
                                     hipMemcpyDeviceToDevice, s));
        MLS_CHECK_HIP(hipMemcpyAsync(S->ds_G + S->head * S->O, G + done * S->O, sizeof(double) * k * S->O,
                                     hipMemcpyDeviceToDevice, s));
        S->head = (S->head + k) % S->cap;
        done += k;
    }
    S->count = std::min(S->cap, S->count + n);
    return MLS2MC_OK;
}

int64_t mls2mc_surrogate_n_pairs(const mls2mc_ctx* ctx) { return (ctx && ctx->sur) ? ctx->sur->count : -1; }

int mls2mc_surrogate_train(mls2mc_ctx* ctx, int epochs, int batch, double lr, uint64_t seed, float* loss_out,
                           void* stream)
{
    MLS_REQUIRE(ctx && ctx->sur, "surrogate_train: call mls2mc_surrogate_init first");
    Surrogate* S = ctx->sur;
    MLS_REQUIRE(epochs >= 0 && batch >= 1 && batch <= 65536 && lr > 0, "surrogate_train: bad epochs/batch/lr");
    MLS_REQUIRE(S->count >= batch, "surrogate_train: fewer pairs than one batch");
    const hipStream_t s = (hipStream_t)stream;
    const bool fused = S->w16 != nullptr;
    if (!fused) MLS_TRY(sur_ensure_batch(S, batch));
    const int64_t n = S->count;
    // standardisation statistics of the current dataset
    col_stats_kernel<<<S->D, 256, 0, s>>>(n, S->D, S->ds_th, S->mu_x, S->sd_x);
    col_stats_kernel<<<S->O, 256, 0, s>>>(n, S->O, S->ds_G, S->mu_y, S->sd_y);
    MLS_CHECK_HIP(hipGetLastError());
    S->standardized = true;
    std::mt19937_64 gen(seed);
    std::vector<int32_t> perm(n);
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const int64_t nb = n / batch;
    for (int ep = 0; ep < epochs; ++ep) {
        std::iota(perm.begin(), perm.end(), 0);
        std::shuffle(perm.begin(), perm.end(), gen);
        MLS_CHECK_HIP(hipMemcpyAsync(S->perm, perm.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, s));
        double ep_loss = 0.0;
        for (int64_t bi = 0; bi < nb; ++bi) {
            const int32_t* idx = S->perm + bi * batch;
            ++S->adam_t;
            const float c1 = 1.f - std::pow(b1, (float)S->adam_t), c2 = 1.f - std::pow(b2, (float)S->adam_t);
            if (fused) {
                MLS_TRY(mlp_step(S, batch, idx, S->ds_th, S->ds_G, true, true, (float)lr, b1, b2, c1, c2, eps, s));
                if (bi == nb - 1 && loss_out) MLS_TRY(mlp_loss(S, batch, s));
            } else {
                standardize_kernel<<<(unsigned)((batch * S->D + 255) / 256), 256, 0, s>>>(batch, S->D, idx, S->ds_th,
                                                                                         S->mu_x, S->sd_x, S->X);
                standardize_kernel<<<(unsigned)((batch * S->O + 255) / 256), 256, 0, s>>>(batch, S->O, idx, S->ds_G,
                                                                                         S->mu_y, S->sd_y, S->T);
                MLS_CHECK_HIP(hipGetLastError());
                MLS_TRY(sur_forward(S, batch, s));
                MLS_TRY(sur_backward(S, batch, s));
                adam_kernel<<<(unsigned)((S->np + 255) / 256), 256, 0, s>>>(S->np, S->p, S->g, S->m, S->v, (float)lr,
                                                                            b1, b2, c1, c2, eps);
                MLS_CHECK_HIP(hipGetLastError());
            }
            if (bi == nb - 1 && loss_out) {
                float l;
                MLS_CHECK_HIP(hipMemcpyAsync(&l, S->loss, sizeof(float), hipMemcpyDeviceToHost, s));
                MLS_CHECK_HIP(hipStreamSynchronize(s));
                ep_loss = l;
            }
        }
        if (loss_out) loss_out[ep] = (float)ep_loss;
    }
    return MLS2MC_OK;
}

int mls2mc_surrogate_predict(mls2mc_ctx* ctx, int64_t N, const double* theta, double* G_out, void* stream)
{
    MLS_REQUIRE(ctx && (ctx->sur || ctx->d_sur_S), "surrogate_predict: call mls2mc_surrogate_init first");
    MLS_REQUIRE(N >= 0, "surrogate_predict: N < 0");
    if (N == 0) return MLS2MC_OK;
    MLS_REQUIRE(theta && G_out, "surrogate_predict: null pointer");
    if (ctx->d_sur_S)  // the linear surrogate
        return launch_linear_map(N, ctx->prob.K, ctx->nobs, ctx->d_sur_S, theta, G_out, (hipStream_t)stream);
    Surrogate* S = ctx->sur;
    const hipStream_t s = (hipStream_t)stream;
    if (S->w16) {
        for (int64_t q0 = 0; q0 < N; q0 += kLaunchParticles) {  // 64 threads a row
            const int64_t B = std::min(kLaunchParticles, N - q0);
            MlpRows P = mlp_rows(S, B);
            P.th = theta + q0 * S->D;
            P.out = G_out + q0 * S->O;
            if (S->standardized) { P.mux = S->mu_x; P.sdx = S->sd_x; P.muy = S->mu_y; P.sdy = S->sd_y; }
            mlp_rows_kernel<false><<<(unsigned)((B + 15) / 16), kRowThreads, mlp_dims(S).lds(), s>>>(P);
            MLS_CHECK_HIP(hipGetLastError());
        }
        return MLS2MC_OK;
    }
    const int64_t chunk = 4096;
    MLS_TRY(sur_ensure_batch(S, std::min(N, chunk)));
    for (int64_t q0 = 0; q0 < N; q0 += chunk) {
        const int64_t B = std::min(chunk, N - q0);
        standardize_kernel<<<(unsigned)((B * S->D + 255) / 256), 256, 0, s>>>(
            B, S->D, nullptr, theta + q0 * S->D, S->standardized ? S->mu_x : nullptr, S->sd_x, S->X);
        MLS_CHECK_HIP(hipGetLastError());
        MLS_TRY(sur_forward(S, B, s));
        if (S->standardized) {
            unstandardize_kernel<<<(unsigned)((B * S->O + 255) / 256), 256, 0, s>>>(B, S->O, S->OUT, S->mu_y,
                                                                                   S->sd_y, G_out + q0 * S->O);
        } else {
            f2d_kernel<<<(unsigned)((B * S->O + 255) / 256), 256, 0, s>>>(B * S->O, S->OUT, G_out + q0 * S->O);
        }
        MLS_CHECK_HIP(hipGetLastError());
    }
    return MLS2MC_OK;
}

// loss and gradient on raw (unstandardised) inputs and targets, for checks
int mls2mc_surrogate_loss_grad(mls2mc_ctx* ctx, int64_t B, const double* x, const double* target, float* loss_out,
                               float* grad_out, void* stream)
{
    MLS_REQUIRE(ctx && ctx->sur, "surrogate_loss_grad: call mls2mc_surrogate_init first");
    MLS_REQUIRE(B >= 1 && B <= 65536, "surrogate_loss_grad: need 1 <= B <= 65536");
    MLS_REQUIRE(x && target && loss_out && grad_out, "surrogate_loss_grad: null pointer");
    Surrogate* S = ctx->sur;
    const hipStream_t s = (hipStream_t)stream;
    if (S->w16) {
        MLS_TRY(mlp_step(S, B, nullptr, x, target, false, false, 0.f, 0.f, 0.f, 1.f, 1.f, 0.f, s));
        MLS_TRY(mlp_loss(S, B, s));
    } else {
        MLS_TRY(sur_ensure_batch(S, B));
        standardize_kernel<<<(unsigned)((B * S->D + 255) / 256), 256, 0, s>>>(B, S->D, nullptr, x, nullptr, nullptr, S->X);
        standardize_kernel<<<(unsigned)((B * S->O + 255) / 256), 256, 0, s>>>(B, S->O, nullptr, target, nullptr, nullptr, S->T);
        MLS_CHECK_HIP(hipGetLastError());
        MLS_TRY(sur_forward(S, B, s));
        MLS_TRY(sur_backward(S, B, s));
    }
    MLS_CHECK_HIP(hipMemcpyAsync(grad_out, S->g, sizeof(float) * S->np, hipMemcpyDeviceToDevice, s));
    MLS_CHECK_HIP(hipMemcpyAsync(loss_out, S->loss, sizeof(float), hipMemcpyDeviceToDevice, s));
    return MLS2MC_OK;
}


int mls2mc_pcn_step_da(mls2mc_ctx* ctx, const mls2mc_stage* st, int64_t N, double* theta, double* G_lo,
                       double* G_hi, double* phi_lo, double* phi_hi, const double* y, const double* xi,
                       const double* u1, const double* u2, uint8_t* accepted_out, uint8_t* stage1_out,
                       int64_t* n_solved_lo, int64_t* n_solved_hi, void* stream)
{
    MLS_REQUIRE(ctx != nullptr && st != nullptr, "pcn_step_da: null argument");
    MLS_REQUIRE(ctx->sur != nullptr || ctx->d_sur_S != nullptr,
                "pcn_step_da: no surrogate (mls2mc_surrogate_init or mls2mc_set_linear_surrogate)");
    MLS_REQUIRE(st->kernel == MLS2MC_KERNEL_PCN, "pcn_step_da: delayed acceptance is built for the pCN kernel");
    MLS_REQUIRE(st->l_lo >= ctx->prob.l_min && st->l_lo <= ctx->prob.l_max, "pcn_step_da: level outside the context");
    const bool bridge = st->l_hi != st->l_lo;
    if (bridge) {
        MLS_REQUIRE(st->l_hi == st->l_lo + 1 && st->l_hi <= ctx->prob.l_max, "pcn_step_da: bridging needs l_hi = l_lo + 1");
        MLS_REQUIRE(st->zeta >= 0.0 && st->zeta <= 1.0, "pcn_step_da: need 0 <= zeta <= 1");
    }
    MLS_REQUIRE(st->s > 0.0 && st->s <= 1.0 && st->beta >= 0.0 && st->beta <= 1.0, "pcn_step_da: bad s or beta");
    MLS_REQUIRE(N >= 0 && N <= (int64_t(1) << 26), "pcn_step_da: need 0 <= N <= 2^26");
    if (N == 0) return MLS2MC_OK;
    MLS_REQUIRE(theta && y && xi && u1 && u2 && accepted_out, "pcn_step_da: null pointer");
    const bool need_lo = !bridge || st->zeta < 1.0, need_hi = bridge;
    MLS_REQUIRE(!need_lo || (G_lo && phi_lo), "pcn_step_da: null coarse-level cache");
    MLS_REQUIRE(!need_hi || (G_hi && phi_hi), "pcn_step_da: null fine-level cache");
    const hipStream_t s = (hipStream_t)stream;
    const int K = ctx->prob.K, nobs = ctx->nobs;
    // scratch layout (doubles, then ints)
    const size_t nd = (size_t)N * (2 * K + 4 * nobs + 4) + 8;
    const size_t bytes = nd * sizeof(double) + (size_t)N * (sizeof(int32_t) * 3 + 2) + 64;
    MLS_TRY(ctx->ws_da.ensure(bytes));
    double* p = ctx->ws_da.as<double>();
    double* thn = p; p += (size_t)N * K;
    double* thc = p; p += (size_t)N * K;
    double* Gs = p; p += (size_t)N * nobs;       // surrogate outputs (old, then new)
    double* Gcl = p; p += (size_t)N * nobs;
    double* Gch = p; p += (size_t)N * nobs;
    double* Gs2 = p; p += (size_t)N * nobs;
    double* ps_old = p; p += N;
    double* ps_new = p; p += N;
    double* pcl = p; p += N;
    double* pch = p; p += N;
    int64_t* count = reinterpret_cast<int64_t*>(p); p += 8;
    int32_t* idx = reinterpret_cast<int32_t*>(p);
    int32_t* itl = idx + N;
    int32_t* ith = itl + N;
    int8_t* stl = reinterpret_cast<int8_t*>(ith + N);
    int8_t* sth = stl + N;
    const double inv_sigma = 1.0 / ctx->prob.sigma_n;
    MLS_TRY(launch_pcn_propose(N, K, st->s, MLS2MC_KERNEL_PCN, theta, xi, thn, s));
    MLS_TRY(mls2mc_surrogate_predict(ctx, N, theta, Gs, stream));
    MLS_TRY(mls2mc_surrogate_predict(ctx, N, thn, Gs2, stream));
    const unsigned gN = (unsigned)((N + 255) / 256);
    da_psis_kernel<<<gN, 256, 0, s>>>(N, nobs, Gs, y, inv_sigma, st->beta, ps_old);
    da_psis_kernel<<<gN, 256, 0, s>>>(N, nobs, Gs2, y, inv_sigma, st->beta, ps_new);
    da_stage1_kernel<<<1, 1024, 0, s>>>(N, u1, ps_old, ps_new, idx, count, accepted_out, stage1_out,
                                        need_lo ? n_solved_lo : nullptr, need_hi ? n_solved_hi : nullptr);
    gather_count_kernel<<<(unsigned)((N * K + 255) / 256), 256, 0, s>>>(N, K, idx, count, thn, thc);
    MLS_CHECK_HIP(hipGetLastError());
    if (need_lo) MLS_TRY(forward_theta(ctx, st->l_lo, N, thc, Gcl, stl, itl, y, pcl, s, count));
    if (need_hi) MLS_TRY(forward_theta(ctx, st->l_hi, N, thc, Gch, sth, ith, y, pch, s, count));
    if (ctx->da_err) {  // the surrogate's error against the finer level's solve
        da_err_kernel<<<1, 256, 0, s>>>(N, count, idx, nobs, Gs2, need_hi ? Gch : Gcl, inv_sigma, ctx->da_err);
        MLS_CHECK_HIP(hipGetLastError());
    }
    const int mode = !bridge ? 0 : (st->zeta < 1.0 ? 1 : 2);
    da_stage2_kernel<<<gN, 256, 0, s>>>(N, count, idx, K, nobs, mode, st->beta, st->zeta, u2, ps_old, ps_new, thn,
                                       Gcl, Gch, pcl, pch, stl, sth, theta, G_lo, G_hi, phi_lo, phi_hi,
                                       accepted_out);
    MLS_CHECK_HIP(hipGetLastError());
    return MLS2MC_OK;
}

}  // extern "C"
