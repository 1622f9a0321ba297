// learned_kernels.hip - kernels of the learned preconditioner.
//
// The preconditioner maps a residual block R to
//   W = D0 .* R + b1 (C E + a)^H E (C E + a) R
//     = (D0 + b1 a^2 E) .* R + 2 a b1 E .* C(E .* R) + b1 E .* C(E .* C(E .* R)),
// a diagonal term plus two spectral-convolution layers (b1 = max(beta1, 0),
// a = beta0, so the layers add a positive semidefinite term and W stays a
// Hermitian positive definite map, as LOBPCG requires), where C = F V F^{-1}
// is the potential block of H~ (the apply's lifted-FFT convolution with the
// kinetic term off) and
//   D0 = M .* (1 + exp(o0[shell(k)])) / 2,  E = M .* exp(o1[shell(k)])
// with M the diagonal of eq:precond and (o0, o1) the two outputs of a small
// MLP (3 hidden layers, GELU) evaluated once per kinetic-energy shell.  D0
// never drops below M/2, so every component of the residual keeps at least
// half of its plain-preconditioned weight.  MLP
// weights are stored in bfloat16; every product accumulates in float32 and the
// optimiser keeps float32 master weights (Adam).  Grid-sized arithmetic is in
// float64 like the rest of the eigensolver's block algebra.

#include <hip/hip_runtime.h>

#include <cstdint>

#include "learned_dev.hpp"

namespace iwfpm {

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));  // inf / nan
    u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest, ties to even
    return (uint16_t)(u >> 16);
}

// GELU(x) = x Phi(x) (exact form) and its derivative Phi(x) + x phi(x)
__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float x) {
    float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
    float pdf = 0.39894228040143268f * expf(-0.5f * x * x);
    return cdf + x * pdf;
}

// ---------------------------------------------------------------------------
// dense layers of the shell MLP on the matrix cores (v_mfma_f32_16x16x16_bf16,
// float32 accumulation).  The weights are bfloat16; an operand held in
// float32 (activations, gradients) is split into three bfloat16 terms
// x = h + m + l (each the round-to-nearest of what the previous ones left),
// which carry its full 24-bit significand, and products of bfloat16 terms are
// exact in float32, so each layer computes what a float32 loop over the
// bf16-rounded weights would, up to the order of the float32 additions.
//
// These products are small (1,024 shells x 256 x 256) and bound by latency: a
// wave that walks K 16 values at a time, element by element, waits for its
// loads again and again (94 us a product).
//
// Forward (k_mlp_fwd): one wave per 16 x 16 tile adds up K in steps of 16
// (v_mfma_f32_16x16x16_bf16: lane l holds A[l%16][4(l/16) .. 4(l/16)+3] and
// B[4(l/16) .. 4(l/16)+3][l%16] and ends with D[4(l/16) + v][l%16], v < 4).
// That order stays as it is: the outputs scale float64 directions, and these
// would follow every change of its rounding.  Only the loads changed: 64
// values of K at a time, the next 64 in flight.
//
// Backward (k_mlp_gemm): a workgroup takes a 32 x 32 tile and its waves split K
// in steps of 32 (v_mfma_f32_16x16x32_bf16: lane l holds k = 8(l/16) ..
// 8(l/16)+7 of row or column l%16, the result as above), each with the next
// step's loads in flight; the waves' tiles are added in LDS in a fixed order,
// where GELU's derivative is applied.  The bias gradient is one more row of
// X^T, of ones.
//
// Loss and gradient of a 65,536-point plan: 2,079 us in all before (the
// products 660, the bias sums 587), 463 now (forward 14 us a product where it
// runs, backward 7 and 15).
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMlpTile = 32;
constexpr int kMlpWaves = 8;

// x = h + m + l in bfloat16 (exact for normal float32 x; round to nearest even
// in hardware, v_cvt_pk_bf16_f32)
__device__ __forceinline__ void split3(float x, short& h, short& m, short& l) {
    const __bf16 a = (__bf16)x;
    const float r1 = x - (float)a;
    const __bf16 b = (__bf16)r1;
    const float r2 = r1 - (float)b;
    h = __builtin_bit_cast(short, a);
    m = __builtin_bit_cast(short, b);
    l = __builtin_bit_cast(short, (__bf16)r2);
}

// eight values k .. k + 7 (zero past K) of row r of an operand stored with k
// contiguous (T: float or bfloat16), or of column r of one stored with k as rows
template <typename T>
__device__ __forceinline__ void mlp_load(const T* __restrict__ p, int ld, bool kcontig, bool vec, int r, int R, int k,
                                         int K, float (&x)[8]) {
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = 0.f;
    if (k >= K) return;
    if (kcontig && vec) {  // K a multiple of 8, rows aligned to 16 bytes
        if (r >= R) return;
        const T* s = p + (size_t)r * ld + k;
        if constexpr (sizeof(T) == 4) {
            const float4 a = reinterpret_cast<const float4*>(s)[0], b = reinterpret_cast<const float4*>(s)[1];
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
            x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        } else {
            const s16x8 v = *reinterpret_cast<const s16x8*>(s);
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = bf2f((uint16_t)v[q]);
        }
        return;
    }
    // loads from the last row or value there is, so that none waits for a branch
    const int rr = min(r, R - 1);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int kk = min(k + q, K - 1);
        const size_t e = kcontig ? (size_t)rr * ld + kk : (size_t)kk * ld + rr;
        float v;
        if constexpr (sizeof(T) == 4) v = p[e];
        else v = bf2f(p[e]);
        x[q] = r < R && k + q < K ? v : 0.f;
    }
}

// C (M x N) = A (M x K, float32, row-major) B (K x N, bfloat16, row-major) +
// bias; Z (optional) receives C, Y = act(C); vec: rows of A start on 16 bytes
// and K is a multiple of 4
__global__ void __launch_bounds__(64) k_mlp_fwd(const float* __restrict__ A, const uint16_t* __restrict__ B,
                                                const float* __restrict__ bias, float* __restrict__ Z,
                                                float* __restrict__ Y, int M, int N, int K, int act, int vec) {
    const int lane = threadIdx.x;
    const int tiles_n = (N + 15) >> 4;
    const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    const int row = tm * 16 + li, col = tn * 16 + li;
    constexpr int U = 4;  // steps of 16 loaded together
    auto fetch = [&](int k0, float4 (&a)[U], uint16_t (&b)[U][4]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + 16 * u + lk;
            a[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (row < M) {
                const float* s = A + (size_t)row * K + k;
                if (vec) {
                    if (k < K) a[u] = *reinterpret_cast<const float4*>(s);
                } else {
                    if (k < K) a[u].x = s[0];
                    if (k + 1 < K) a[u].y = s[1];
                    if (k + 2 < K) a[u].z = s[2];
                    if (k + 3 < K) a[u].w = s[3];
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) b[u][q] = col < N && k + q < K ? B[(size_t)(k + q) * N + col] : (uint16_t)0;
        }
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float4 a[U];
    uint16_t b[U][4];
    fetch(0, a, b);
    for (int k0 = 0; k0 < K; k0 += 16 * U) {
        float4 an[U];
        uint16_t bn[U][4];
        fetch(k0 + 16 * U, an, bn);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k0 + 16 * u >= K) break;
            const float av[4] = {a[u].x, a[u].y, a[u].z, a[u].w};
            bf16x4 ah, am, al, bh;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                short h, m, l;
                split3(av[q], h, m, l);
                ah[q] = h;
                am[q] = m;
                al[q] = l;
                bh[q] = (short)b[u][q];
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(am, bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(al, bh, acc, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a[u] = an[u];
#pragma unroll
            for (int q = 0; q < 4; ++q) b[u][q] = bn[u][q];
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = tm * 16 + lk + v;
        if (r < M && col < N) {
            const float z = acc[v] + bias[col];
            const size_t e = (size_t)r * N + col;
            if (Z) Z[e] = z;
            Y[e] = act ? gelu(z) : z;
        }
    }
}

struct MlpGemm {
    const float* A;      // M x K; a_k: k contiguous (row stride lda), else stored K x M
    const void* B;       // K x N, TB; b_k: k contiguous (stored N x K), else row stride ldb
    float* Y;            // the sums, times GELU'(dact) where that is given
    const float* dact;   // pre-activations (M x N), or null
    float* ones;         // null, or where row M - 1 goes: A's last row is then all ones
    int M, N, K, lda, ldb, a_k, b_k, a_vec, b_vec;
};

template <typename TB>
__global__ void __launch_bounds__(64 * kMlpWaves) k_mlp_gemm(MlpGemm g) {
    __shared__ float red[kMlpWaves][kMlpTile][kMlpTile + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = 8 * (lane >> 4);
    const int tiles_n = (g.N + kMlpTile - 1) / kMlpTile;
    const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
    const int r0 = tm * kMlpTile, c0 = tn * kMlpTile;
    const int Ma = g.ones ? g.M - 1 : g.M;  // rows that A holds
    const TB* B = reinterpret_cast<const TB*>(g.B);
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](int k0, float (&a)[2][8], float (&b)[2][8]) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int r = r0 + 16 * t + li;
            mlp_load<float>(g.A, g.lda, g.a_k, g.a_vec, r, Ma, k0 + lk, g.K, a[t]);
            if (g.ones && r == g.M - 1)
#pragma unroll
                for (int q = 0; q < 8; ++q) a[t][q] = k0 + lk + q < g.K ? 1.f : 0.f;
            mlp_load<TB>(B, g.ldb, g.b_k, g.b_vec, c0 + 16 * t + li, g.N, k0 + lk, g.K, b[t]);
        }
    };
    float a[2][8], b[2][8];
    const int step = 32 * kMlpWaves;
    int k0 = 32 * wave;
    if (k0 < g.K) fetch(k0, a, b);
    for (; k0 < g.K; k0 += step) {
        float an[2][8], bn[2][8];
        if (k0 + step < g.K) fetch(k0 + step, an, bn);
        bf16x8 ah[2], am[2], al[2], bh[2], bm[2], bl[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            s16x8 h, m, l;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                short x, y, z;
                split3(a[t][q], x, y, z);
                h[q] = x;
                m[q] = y;
                l[q] = z;
            }
            ah[t] = __builtin_bit_cast(bf16x8, h);
            am[t] = __builtin_bit_cast(bf16x8, m);
            al[t] = __builtin_bit_cast(bf16x8, l);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                short x, y = 0, z = 0;
                if constexpr (sizeof(TB) == 4) split3(b[t][q], x, y, z);
                else x = (short)(__float_as_uint(b[t][q]) >> 16);
                h[q] = x;
                m[q] = y;
                l[q] = z;
            }
            bh[t] = __builtin_bit_cast(bf16x8, h);
            bm[t] = __builtin_bit_cast(bf16x8, m);
            bl[t] = __builtin_bit_cast(bf16x8, l);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am[i], bh[j], acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
                if constexpr (sizeof(TB) == 4) {
                    // float32 x float32: the six largest of the nine terms
                    // (what is left is below 2^-23 of each product)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bm[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am[i], bm[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
                }
            }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                a[t][q] = an[t][q];
                b[t][q] = bn[t][q];
            }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][16 * i + 4 * (lane >> 4) + v][16 * j + li] = acc[i][j][v];
    __syncthreads();
    const int waves = min(kMlpWaves, (g.K + 31) / 32);  // the others' tiles are zero
    for (int e = threadIdx.x; e < kMlpTile * kMlpTile; e += blockDim.x) {
        const int i = e / kMlpTile, j = e - i * kMlpTile;
        const int r = r0 + i, c = c0 + j;
        if (r >= g.M || c >= g.N) continue;
        float z = red[0][i][j];
        for (int w = 1; w < waves; ++w) z += red[w][i][j];
        if (g.ones && r == g.M - 1) {
            g.ones[c] = z;
            continue;
        }
        const size_t o = (size_t)r * g.N + c;
        g.Y[o] = g.dact ? z * gelu_grad(g.dact[o]) : z;
    }
}

__global__ void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v, const float* __restrict__ g,
                       uint16_t* __restrict__ wbf, int n, float lr, float b1, float b2, float c1, float c2, float eps) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    float gg = g[e];
    float mm = b1 * m[e] + (1.f - b1) * gg;
    float vv = b2 * v[e] + (1.f - b2) * gg * gg;
    m[e] = mm;
    v[e] = vv;
    float nw = w[e] - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    w[e] = nw;
    wbf[e] = f2bf(nw);
}

__global__ void k_to_bf16(const float* __restrict__ w, uint16_t* __restrict__ wbf, int n) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) wbf[e] = f2bf(w[e]);
}

// ---------------------------------------------------------------------------
// grid-sized kernels (HBM-bound elementwise passes and reductions)
// ---------------------------------------------------------------------------

__global__ void k_expand(const double* __restrict__ M, const int* __restrict__ shell, const float* __restrict__ O,
                         double* __restrict__ D0, double* __restrict__ E, long long N) {
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < N; k += (long long)gridDim.x * blockDim.x) {
        int s = shell[k];
        double mk = M[k];
        D0[k] = 0.5 * mk * (1.0 + exp((double)O[2 * s]));
        E[k] = mk * exp((double)O[2 * s + 1]);
    }
}

__global__ void k_scale_cols(ColPtrs R, double2* __restrict__ Y, int m, const double* __restrict__ d, long long N) {
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < N; k += (long long)gridDim.x * blockDim.x) {
        double s = d[k];
        for (int j = 0; j < m; ++j) {
            double2 a = R.p[j][k];
            Y[(size_t)j * N + k] = make_double2(s * a.x, s * a.y);
        }
    }
}

__global__ void k_scale(const double2* __restrict__ A, double2* __restrict__ Y, int m, const double* __restrict__ d,
                        long long N) {
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < N; k += (long long)gridDim.x * blockDim.x) {
        double s = d[k];
#pragma unroll 4
        for (int j = 0; j < m; ++j) {
            double2 a = A[(size_t)j * N + k];
            Y[(size_t)j * N + k] = make_double2(s * a.x, s * a.y);
        }
    }
}

// coefficients of the expanded layers: E A (c0), E Cc (c1) and the extra diagonal E (dl)
struct LayerCoef {
    double a, b1, c0, c1, dl;
};
__device__ __forceinline__ LayerCoef layer_coef(const float* beta) {
    LayerCoef c;
    c.a = beta[0];
    c.b1 = beta[1] > 0.f ? (double)beta[1] : 0.0;
    c.c0 = 2.0 * c.a * c.b1;
    c.c1 = c.b1;
    c.dl = c.b1 * c.a * c.a;
    return c;
}

__global__ void k_combine(ColPtrs R, const double2* __restrict__ A, const double2* __restrict__ C, ColPtrs W, int m,
                          const double* __restrict__ D0, const double* __restrict__ E, const float* __restrict__ beta,
                          long long N) {
    const LayerCoef lc = layer_coef(beta);
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < N; k += (long long)gridDim.x * blockDim.x) {
        double e = E[k], d = D0[k] + lc.dl * e;
        for (int j = 0; j < m; ++j) {
            double2 r = R.p[j][k], a = A[(size_t)j * N + k], c = C[(size_t)j * N + k];
            W.p[j][k] = make_double2(d * r.x + e * (lc.c0 * a.x + lc.c1 * c.x), d * r.y + e * (lc.c0 * a.y + lc.c1 * c.y));
        }
    }
}

// block sum of v over the block's wavefronts (blockDim.x = 256), result valid in thread 0
__device__ __forceinline__ double block_sum(double v, double* sh) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[wv] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
    return t;
}

__device__ __forceinline__ double redot(double2 a, double2 b) { return a.x * b.x + a.y * b.y; }  // Re(conj(a) b)

__global__ void __launch_bounds__(256) k_shell_grad(const double2* __restrict__ G, const double2* __restrict__ R,
                                                    const double2* __restrict__ A, const double2* __restrict__ C,
                                                    const double2* __restrict__ B1, const double2* __restrict__ B2,
                                                    int m, const double* __restrict__ M,
                                                    const double* __restrict__ D0,
                                                    const double* __restrict__ E, const float* __restrict__ beta,
                                                    const int* __restrict__ shell, double* __restrict__ dO,
                                                    double* __restrict__ dbeta, long long N) {
    __shared__ double sh[4];
    const LayerCoef lc = layer_coef(beta);
    double gb0 = 0.0, gb1 = 0.0, gbd = 0.0;
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < N; k += (long long)gridDim.x * blockDim.x) {
        double dd = 0.0, de = 0.0, ga = 0.0, gc = 0.0;
#pragma unroll 4
        for (int j = 0; j < m; ++j) {
            const size_t o = (size_t)j * N + k;
            double2 g = G[o], r = R[o], a = A[o], c = C[o], p1 = B1[o], p2 = B2[o];
            double gr = redot(g, r), gA = redot(g, a), gC = redot(g, c);
            dd += gr;
            de += lc.c0 * (gA + redot(p1, r)) + lc.c1 * (gC + redot(p1, a) + redot(p2, r));
            ga += gA;
            gc += gC;
        }
        const double e = E[k];
        const int s = shell[k];
        atomicAdd(&dO[2 * s], dd * (D0[k] - 0.5 * M[k]));  // dD0/do0 = M exp(o0) / 2
        atomicAdd(&dO[2 * s + 1], (de + lc.dl * dd) * e);
        gb0 += ga * e;
        gb1 += gc * e;
        gbd += dd * e;
    }
    double v = block_sum(gb0, sh);
    if (threadIdx.x == 0) atomicAdd(&dbeta[0], v);
    v = block_sum(gb1, sh);
    if (threadIdx.x == 0) atomicAdd(&dbeta[1], v);
    v = block_sum(gbd, sh);
    if (threadIdx.x == 0) atomicAdd(&dbeta[2], v);
}

// (dL/dc0, dL/dc1, dL/ddl) -> gradient of (beta0, beta1); below zero beta1 passes
// the gradient of its positive side so that the optimiser can switch the layers on
__global__ void k_beta_grad(const double* __restrict__ dbeta, const float* __restrict__ beta, float* __restrict__ g) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const LayerCoef lc = layer_coef(beta);
    const double g0 = dbeta[0], g1 = dbeta[1], gd = dbeta[2];
    g[0] = (float)(2.0 * lc.b1 * g0 + 2.0 * lc.a * lc.b1 * gd);
    g[1] = (float)(2.0 * lc.a * g0 + g1 + lc.a * lc.a * gd);
}

__global__ void k_to_float(const double* __restrict__ a, float* __restrict__ b, int n, double scale) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) b[e] = (float)(a[e] * scale);
}

__global__ void k_nonfinite(const float* __restrict__ a, int n, int* __restrict__ flag) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n && !isfinite(a[e])) atomicOr(flag, 1);
}

__global__ void k_nonfinite_d(const double* __restrict__ a, long long n, int* __restrict__ flag) {
    bool bad = false;
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long long)gridDim.x * blockDim.x)
        bad = bad || !isfinite(a[k]);
    if (bad) atomicOr(flag, 1);
}

// ---------------------------------------------------------------------------
static int blocks_for(long long n, int cap) {
    long long b = (n + 255) / 256;
    return (int)(b < 1 ? 1 : (b > cap ? cap : b));
}
constexpr int kGridCap = 4096;
constexpr int kNoCap = 1 << 30;

static int mlp_blocks(const MlpGemm& g) {
    return ((g.M + kMlpTile - 1) / kMlpTile) * ((g.N + kMlpTile - 1) / kMlpTile);
}
// rows of ld elements of `esz` bytes at p start on 16 bytes and hold whole groups of eight
static int mlp_vec(const void* p, int ld, int K, int esz) {
    return K % 8 == 0 && ld * esz % 16 == 0 && reinterpret_cast<uintptr_t>(p) % 16 == 0;
}

hipError_t lp_dense_fwd(const float* X, const uint16_t* W, const float* b, float* Z, float* Y, int S, int in, int out,
                        int act, hipStream_t st) {
    const int vec = in % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
    k_mlp_fwd<<<((S + 15) / 16) * ((out + 15) / 16), 64, 0, st>>>(X, W, b, Z, Y, S, out, in, act, vec);
    return hipGetLastError();
}
hipError_t lp_dense_bwd(const float* X, const float* dZ, const uint16_t* W, const float* Zin, float* dX, float* dW,
                        float* db, int S, int in, int out, hipStream_t st) {
    if (dX) {
        // dX (S x in) = dZ (S x out) W^T, times GELU'(Zin)
        const MlpGemm g{dZ, W, dX, Zin, nullptr, S, in, out, out, out, 1, 1, mlp_vec(dZ, out, out, 4),
                        mlp_vec(W, out, out, 2)};
        k_mlp_gemm<uint16_t><<<mlp_blocks(g), 64 * kMlpWaves, 0, st>>>(g);
    }
    // [dW; db] (in + 1 rows x out) = [X 1]^T (in + 1 x S) dZ (S x out)
    const MlpGemm g{X, dZ, dW, nullptr, db, in + 1, out, S, in, out, 0, 0, 0, 0};
    k_mlp_gemm<float><<<mlp_blocks(g), 64 * kMlpWaves, 0, st>>>(g);
    return hipGetLastError();
}
hipError_t lp_adam(float* w, float* m, float* v, const float* g, uint16_t* wbf, int n, float lr, float b1, float b2,
                   float c1, float c2, float eps, hipStream_t st) {
    k_adam<<<blocks_for(n, kNoCap), 256, 0, st>>>(w, m, v, g, wbf, n, lr, b1, b2, c1, c2, eps);
    return hipGetLastError();
}
hipError_t lp_to_bf16(const float* w, uint16_t* wbf, int n, hipStream_t st) {
    k_to_bf16<<<blocks_for(n, kNoCap), 256, 0, st>>>(w, wbf, n);
    return hipGetLastError();
}
hipError_t lp_expand(const double* M, const int* shell, const float* O, double* D0, double* E, long long N,
                     hipStream_t st) {
    k_expand<<<blocks_for(N, kGridCap), 256, 0, st>>>(M, shell, O, D0, E, N);
    return hipGetLastError();
}
hipError_t lp_scale_cols(const ColPtrs& R, double2* Y, int m, const double* d, long long N, hipStream_t st) {
    k_scale_cols<<<blocks_for(N, kGridCap), 256, 0, st>>>(R, Y, m, d, N);
    return hipGetLastError();
}
hipError_t lp_scale(const double2* A, double2* Y, int m, const double* d, long long N, hipStream_t st) {
    k_scale<<<blocks_for(N, kGridCap), 256, 0, st>>>(A, Y, m, d, N);
    return hipGetLastError();
}
hipError_t lp_combine(const ColPtrs& R, const double2* A, const double2* C, const ColPtrs& W, int m, const double* D0,
                      const double* E, const float* beta, long long N, hipStream_t st) {
    k_combine<<<blocks_for(N, kGridCap), 256, 0, st>>>(R, A, C, W, m, D0, E, beta, N);
    return hipGetLastError();
}
hipError_t lp_shell_grad(const double2* G, const double2* R, const double2* A, const double2* C, const double2* B1,
                         const double2* B2, int m, const double* M, const double* D0, const double* E,
                         const float* beta, const int* shell, double* dO, double* dbeta, long long N,
                         hipStream_t st) {
    k_shell_grad<<<blocks_for(N, kGridCap), 256, 0, st>>>(G, R, A, C, B1, B2, m, M, D0, E, beta, shell, dO, dbeta,
                                                          N);
    return hipGetLastError();
}
hipError_t lp_beta_grad(const double* dbeta, const float* beta, float* g, hipStream_t st) {
    k_beta_grad<<<1, 64, 0, st>>>(dbeta, beta, g);
    return hipGetLastError();
}
hipError_t lp_to_float(const double* a, float* b, int n, double scale, hipStream_t st) {
    k_to_float<<<blocks_for(n, kNoCap), 256, 0, st>>>(a, b, n, scale);
    return hipGetLastError();
}
hipError_t lp_nonfinite_d(const double* a, long long n, int* flag, hipStream_t st) {
    k_nonfinite_d<<<blocks_for(n, kGridCap), 256, 0, st>>>(a, n, flag);
    return hipGetLastError();
}
hipError_t lp_nonfinite(const float* a, int n, int* flag, hipStream_t st) {
    k_nonfinite<<<blocks_for(n, kNoCap), 256, 0, st>>>(a, n, flag);
    return hipGetLastError();
}

}  // namespace iwfpm
