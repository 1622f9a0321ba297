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
// half of its plain-preconditioned weight.  MLP weights are stored in bfloat16;
// the forward products accumulate in float32, the backward ones in float64, and
// the optimiser keeps float32 master weights (Adam).  Grid-sized arithmetic is
// in float64 like the rest of the eigensolver's block algebra.

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
__device__ __forceinline__ double gelu_grad(double x) {
    const double cdf = 0.5 * (1.0 + erf(x * 0.70710678118654752));
    const double pdf = 0.39894228040143268 * exp(-0.5 * x * x);
    return cdf + x * pdf;
}

// ---------------------------------------------------------------------------
// dense layers of the shell MLP on the matrix cores, weights in bfloat16.
//
// These products are small (1,024 shells x 256 x 256) and bound by latency: a
// wave that walks K 16 values at a time, element by element, waits for its
// loads again and again (94 us a product).
//
// Forward (k_mlp_fwd): float32 accumulation.  The float32 activations are split
// into three bfloat16 terms x = h + m + l (each the round-to-nearest of what the
// previous ones left), which carry the full 24-bit significand, and products of
// bfloat16 terms are exact in float32, so a layer computes what a float32 loop
// over the bf16-rounded weights would, up to the order of the float32 additions.
// One wave per 16 x 16 tile adds up K in steps of 16
// (v_mfma_f32_16x16x16_bf16: lane l holds A[l%16][4(l/16) .. 4(l/16)+3] and
// B[4(l/16) .. 4(l/16)+3][l%16] and ends with D[4(l/16) + v][l%16], v < 4).
// That order stays as it is: the outputs scale float64 directions, and these
// would follow every change of its rounding.  Only the loads changed: 64
// values of K at a time, the next 64 in flight.
//
// Backward (k_mlp_dx, k_mlp_dw): float64 on the matrix cores
// (v_mfma_f64_16x16x4f64: lane l holds A[l%16][l/16] and B[l/16][l%16] and ends
// with D[l/16 + 4v][l%16], v < 4).  The shells' gradients cancel when they are
// summed (at weak coupling sum |dO| is hundreds of times |sum dO|, and more), so
// sums in float32 lose digits that the result needs.  Error of the gradient
// against 64 bits (norms; 37 cases, couplings 0.1 to 10, 2 to 12 columns): 0.29e-6
// to 2.3e-6 with float32 sums over 16 values of K a step, 0.08e-6 to 2.5e-6 over
// 32 a step, 0.03e-6 to 2.2e-6 now and in no case larger than either; what is
// left is the float32 forward pass.  A workgroup takes a 16 x 16 tile and its
// waves split K, each with the next step's loads in flight; their tiles are
// added in LDS in a fixed order, where GELU's derivative is applied.  The bias
// gradient is one more row of X^T, of ones.
//
// Loss and gradient of a 65,536-point plan: 2,079 us with a wave per tile that
// loads K element by element (the products 660, the bias sums 587), 414 now
// (forward 14 us a product where it runs, backward 14 and 11; 436 with the split
// float32 products).
// ---------------------------------------------------------------------------
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

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

constexpr int kMlpWaves = 8;

// the workgroup's tile: every wave's part, added up in wave order; element e of
// the tile (row e / 16, column e % 16) goes to thread e
__device__ __forceinline__ double mlp_tile_sum(const f64x4& acc, double (&red)[kMlpWaves][16][17]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][(lane >> 4) + 4 * v][lane & 15] = acc[v];
    __syncthreads();
    double z = 0.0;
    if (threadIdx.x < 256)
        for (int w = 0; w < kMlpWaves; ++w) z += red[w][threadIdx.x >> 4][threadIdx.x & 15];
    return z;
}

// dX (S x in) = dZ (S x out) W^T .* GELU'(Zin), W (in x out) bfloat16.  A lane's
// four steps of a round take four neighbouring k, the same for both operands;
// vec: out is a multiple of 4 and rows start on 16 (dZ) and 8 bytes (W)
__global__ void __launch_bounds__(64 * kMlpWaves) k_mlp_dx(const double* __restrict__ dZ,
                                                           const uint16_t* __restrict__ W,
                                                           const float* __restrict__ Zin, double* __restrict__ dX,
                                                           int S, int in, int out, int vec) {
    __shared__ double red[kMlpWaves][16][17];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = 4 * (lane >> 4);
    const int tiles_n = (in + 15) >> 4;
    const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
    const int s = tm * 16 + li, i = tn * 16 + li;
    const double* a = dZ + (size_t)min(s, S - 1) * out;
    const uint16_t* b = W + (size_t)min(i, in - 1) * out;
    // loads from the last row or values there are, so that none waits for a branch
    auto fetch = [&](int k0, double (&x)[4], uint16_t (&w)[4]) {
        if (vec) {
            const int k = min(k0 + lk, out - 4);
            const double2 x0 = reinterpret_cast<const double2*>(a + k)[0], x1 = reinterpret_cast<const double2*>(a + k)[1];
            const ushort4 wv = *reinterpret_cast<const ushort4*>(b + k);
            x[0] = x0.x; x[1] = x0.y; x[2] = x1.x; x[3] = x1.y;
            w[0] = wv.x; w[1] = wv.y; w[2] = wv.z; w[3] = wv.w;
            return;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = min(k0 + lk + q, out - 1);
            x[q] = a[k];
            w[q] = b[k];
        }
    };
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    double x[4];
    uint16_t w[4];
    int k0 = 16 * wave;
    if (k0 < out) fetch(k0, x, w);
    for (; k0 < out; k0 += 16 * kMlpWaves) {
        double xn[4];
        uint16_t wn[4];
        fetch(k0 + 16 * kMlpWaves, xn, wn);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool ok = k0 + lk + q < out;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ok && s < S ? x[q] : 0.0,
                                                       ok && i < in ? (double)bf2f(w[q]) : 0.0, acc, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            x[q] = xn[q];
            w[q] = wn[q];
        }
    }
    const double z = mlp_tile_sum(acc, red);
    const int r = tm * 16 + (threadIdx.x >> 4), c = tn * 16 + (threadIdx.x & 15);
    if (threadIdx.x >= 256 || r >= S || c >= in) return;
    const size_t e = (size_t)r * in + c;
    dX[e] = z * gelu_grad((double)Zin[e]);
}

// dW (in x out) = X^T dZ, X (S x in), and db (out) = the column sums of dZ as row
// `in` of the product
__global__ void __launch_bounds__(64 * kMlpWaves) k_mlp_dw(const float* __restrict__ X,
                                                           const double* __restrict__ dZ, float* __restrict__ dW,
                                                           float* __restrict__ db, int S, int in, int out) {
    __shared__ double red[kMlpWaves][16][17];
    constexpr int U = 8;  // steps of 4 loaded together
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int tiles_n = (out + 15) >> 4;
    const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
    const int i = tm * 16 + li, o = tn * 16 + li;
    const float* a = X + min(i, in - 1);
    const double* b = dZ + min(o, out - 1);
    auto fetch = [&](int s0, float (&x)[U], double (&d)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t s = min(s0 + 4 * u + lk, S - 1);
            x[u] = a[s * in];
            d[u] = b[s * out];
        }
    };
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    float x[U];
    double d[U];
    constexpr int step = 4 * U * kMlpWaves;
    int s0 = 4 * U * wave;
    if (s0 < S) fetch(s0, x, d);
    for (; s0 < S; s0 += step) {
        float xn[U];
        double dn[U];
        fetch(s0 + step, xn, dn);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = s0 + 4 * u + lk < S;
            const double av = i < in ? (double)x[u] : (i == in ? 1.0 : 0.0);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ok ? av : 0.0, ok && o < out ? d[u] : 0.0, acc, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = xn[u];
            d[u] = dn[u];
        }
    }
    const double z = mlp_tile_sum(acc, red);
    const int r = tm * 16 + (threadIdx.x >> 4), c = tn * 16 + (threadIdx.x & 15);
    if (threadIdx.x >= 256 || r > in || c >= out) return;
    if (r == in) db[c] = (float)z;
    else dW[(size_t)r * out + c] = (float)z;
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

static int mlp_tiles(int M, int N) { return ((M + 15) / 16) * ((N + 15) / 16); }

hipError_t lp_dense_fwd(const float* X, const uint16_t* W, const float* b, float* Z, float* Y, int S, int in, int out,
                        int act, hipStream_t st) {
    const int vec = in % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
    k_mlp_fwd<<<mlp_tiles(S, out), 64, 0, st>>>(X, W, b, Z, Y, S, out, in, act, vec);
    return hipGetLastError();
}
hipError_t lp_dense_bwd(const float* X, const double* dZ, const uint16_t* W, const float* Zin, double* dX, float* dW,
                        float* db, int S, int in, int out, hipStream_t st) {
    if (dX) {
        const int vec = out % 4 == 0 && reinterpret_cast<uintptr_t>(dZ) % 16 == 0 && reinterpret_cast<uintptr_t>(W) % 8 == 0;
        k_mlp_dx<<<mlp_tiles(S, in), 64 * kMlpWaves, 0, st>>>(dZ, W, Zin, dX, S, in, out, vec);
    }
    k_mlp_dw<<<mlp_tiles(in + 1, out), 64 * kMlpWaves, 0, st>>>(X, dZ, dW, db, S, in, out);
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
hipError_t lp_nonfinite_d(const double* a, long long n, int* flag, hipStream_t st) {
    k_nonfinite_d<<<blocks_for(n, kGridCap), 256, 0, st>>>(a, n, flag);
    return hipGetLastError();
}
hipError_t lp_nonfinite(const float* a, int n, int* flag, hipStream_t st) {
    k_nonfinite<<<blocks_for(n, kNoCap), 256, 0, st>>>(a, n, flag);
    return hipGetLastError();
}

}  // namespace iwfpm
