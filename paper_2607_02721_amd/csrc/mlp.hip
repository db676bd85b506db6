// Learned sampling proposal: an MLP 64 -> 256 -> 256 -> 256 -> 1 with SiLU
// that predicts log-sensitivity from per-Gaussian features.  The products run
// on the BF16 matrix cores of gfx950 (v_mfma_f32_16x16x32_bf16, FP32
// accumulation); activations are rounded to BF16 between layers and kept in
// FP32 (pre-activation) for the backward pass; parameters and Adam moments are
// FP32.  Training and inference each run the whole network in one kernel per
// block of rows; a second training form computes everything in FP32 (a
// precision mode for gradient checks).
//
// Parameter vector (FP32, PyTorch Linear layout [out][in]):
//   W1[256][64] b1[256] W2[256][256] b2[256] W3[256][256] b3[256] w4[256] b4
#include "gs_internal.hpp"

#include <math.h>

#include <cmath>

#include <algorithm>

namespace gs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// SiLU and its derivative with the hardware reciprocal (v_rcp_f32, 1 ulp)
// instead of an IEEE division: the same form in training and inference.
__device__ __forceinline__ float sigmoid_fast(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigmoid_fast(z); }
__device__ __forceinline__ float silu_grad(float z) {
    const float s = sigmoid_fast(z);
    return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------------------
// FP32 training step: v_mfma_f32_16x16x4_f32, one kernel per product.
//
// acc += A-fragment x B-fragment over one k step of 32 (8 consecutive k per
// lane): the instruction sums over the four 16-lane groups, so call e of 8
// multiplies the k = 8 g + e of every group g; the eight cover the 32 k.
struct Frag8 {
    float4 lo, hi;
    __device__ __forceinline__ void load(const float *p) {
        lo = *reinterpret_cast<const float4 *>(p);
        hi = *reinterpret_cast<const float4 *>(p + 4);
    }
};

__device__ __forceinline__ void mma32(const Frag8 &a, const Frag8 &b, f32x4 &acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.lo.x, b.lo.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.lo.y, b.lo.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.lo.z, b.lo.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.lo.w, b.lo.w, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.hi.x, b.hi.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.hi.y, b.hi.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.hi.z, b.hi.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.hi.w, b.hi.w, acc, 0, 0, 0);
}

// C[M][N] = A[M][K] * B[N][K]^T (row-major, K contiguous), FP32 accumulate.
// Block = 4 waves computing a 64x64 tile (each wave 32x32 = 2x2 MFMA tiles of
// 16x16, K in steps of 32).  Fragment layout of the 16x16 MFMAs: lane l
// holds row (l % 16) of A and column (l % 16) of B^T for the 8 consecutive k
// at 8 (l / 16); the 16x16 result gives lane l the 4 rows 4 (l / 16) + r of
// column l % 16.
// Split K: block z multiplies k in [z kchunk, min(K, (z + 1) kchunk)) and
// stores its partial product at C + z czstride (epilogue 0 only).
// Epilogues: 0 = store C; 1 = Z = C + bias -> store Z and SiLU(Z).
// Requires M, N multiples of 64 and K, kchunk multiples of 32 (checked by the host).
template <int kEpi>
__global__ __launch_bounds__(256) void k_gemm_nt(const float *__restrict__ A, int lda, const float *__restrict__ B, int ldb,
                                                 int K, int kchunk, float *__restrict__ C, int ldc, int64_t czstride,
                                                 const float *__restrict__ bias, float *__restrict__ H, int ldh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int row0 = blockIdx.x * 64 + (w & 1) * 32;
    const int col0 = blockIdx.y * 64 + (w >> 1) * 32;
    const int fr = lane & 15, fk = (lane >> 4) * 8;
    const int kb = blockIdx.z * kchunk, ke = min(K, kb + kchunk);
    C += (int64_t)blockIdx.z * czstride;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float *a0 = A + (int64_t)(row0 + fr) * lda + fk;
    const float *a1 = A + (int64_t)(row0 + 16 + fr) * lda + fk;
    const float *b0 = B + (int64_t)(col0 + fr) * ldb + fk;
    const float *b1 = B + (int64_t)(col0 + 16 + fr) * ldb + fk;
    for (int k0 = kb; k0 < ke; k0 += 32) {
        Frag8 fa0, fa1, fb0, fb1;
        fa0.load(a0 + k0);
        fa1.load(a1 + k0);
        fb0.load(b0 + k0);
        fb1.load(b1 + k0);
        mma32(fa0, fb0, acc[0][0]);
        mma32(fa0, fb1, acc[0][1]);
        mma32(fa1, fb0, acc[1][0]);
        mma32(fa1, fb1, acc[1][1]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = row0 + i * 16 + (lane >> 4) * 4 + r;
                const int col = col0 + j * 16 + fr;
                float v = acc[i][j][r];
                if (kEpi == 0) {
                    C[(int64_t)row * ldc + col] = v;
                } else {
                    v += bias[col];
                    C[(int64_t)row * ldc + col] = v;
                    H[(int64_t)row * ldh + col] = silu(v);
                }
            }
}

static void gemm_nt(int epi, const float *A, int lda, const float *B, int ldb, int M, int N, int K, float *C, int ldc,
                    const float *bias, float *H, int ldh, hipStream_t st) {
    dim3 grid(M / 64, N / 64);
    if (epi == 0)
        hipLaunchKernelGGL((k_gemm_nt<0>), grid, dim3(256), 0, st, A, lda, B, ldb, K, K, C, ldc, (int64_t)0, bias,
                           H, ldh);
    else
        hipLaunchKernelGGL((k_gemm_nt<1>), grid, dim3(256), 0, st, A, lda, B, ldb, K, K, C, ldc, (int64_t)0, bias,
                           H, ldh);
}

// Weight gradients are M x N = 256 x {256, 64} products over K = the batch
// rows: a 4 x 4 (or 4 x 1) grid of tiles would leave most of the 256 CUs
// idle, so K is split into up to kMaxSplits ranges of at least 512 rows, each
// tile of each range is one block, and a second kernel sums the partial
// products in range order (fixed, so the result is deterministic).
constexpr int kMaxSplits = 32;
static int split_count(int64_t K) { return (int)std::max<int64_t>(1, std::min<int64_t>(kMaxSplits, K / 512)); }

__global__ void k_sum_splits(const float *__restrict__ part, int splits, int64_t count, float *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    float s = part[i];
    for (int z = 1; z < splits; ++z) s += part[(int64_t)z * count + i];
    out[i] = s;
}

static void gemm_nt_splitk(const float *A, int lda, const float *B, int ldb, int M, int N, int K, float *part, float *C,
                           hipStream_t st) {
    const int S = split_count(K);
    const int kchunk = (int)(((int64_t)K + S - 1) / S + 31) / 32 * 32;
    const int used = (K + kchunk - 1) / kchunk;
    dim3 grid(M / 64, N / 64, used);
    hipLaunchKernelGGL((k_gemm_nt<0>), grid, dim3(256), 0, st, A, lda, B, ldb, K, kchunk, part, N,
                       (int64_t)M * N, (const float *)nullptr, (float *)nullptr, 0);
    const int64_t count = (int64_t)M * N;
    hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, part, used, count, C);
}

// Copies of the weights in T: Wk[out][in] and, if kTransposed, the transposes
// W2^T and W3^T ([in][out]) that the backward products read.  One block per
// 64x64 tile (W2, W3, then W1), transposed through LDS so that both copies are
// written in order.
constexpr int kCastBlocks = 36;
template <typename T, bool kTransposed>
__global__ __launch_bounds__(256) void k_weights_cast(const float *__restrict__ P, T *__restrict__ W1,
                                                      T *__restrict__ W2, T *__restrict__ W3, T *__restrict__ W2t,
                                                      T *__restrict__ W3t) {
    __shared__ float tile[64][65];
    const int b = blockIdx.x, layer = b < 16 ? 1 : (b < 32 ? 2 : 0);
    const int in = layer ? kMlpH : kMlpIn;
    const int o0 = layer ? ((b >> 2) & 3) * 64 : (b - 32) * 64, c0 = layer ? (b & 3) * 64 : 0;
    const float *src = P + (layer == 1 ? kOffW2 : (layer == 2 ? kOffW3 : kOffW1));
    T *dst = layer == 1 ? W2 : (layer == 2 ? W3 : W1), *dstt = layer == 1 ? W2t : W3t;
    const int col = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int row = k * 4 + (threadIdx.x >> 6);
        const float v = src[(int64_t)(o0 + row) * in + c0 + col];
        dst[(int64_t)(o0 + row) * in + c0 + col] = static_cast<T>(v);
        if (kTransposed) tile[row][col] = v;
    }
    if (kTransposed && layer) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int row = k * 4 + (threadIdx.x >> 6);
            dstt[(int64_t)(c0 + row) * kMlpH + o0 + col] = static_cast<T>(tile[col][row]);
        }
    }
}

// ---------------------------------------------------------------------------
// Elementwise and small kernels of the FP32 step.

// X0[r][c] = (feat[r][c] - mean[c]) * inv_std[c]; rows >= n are zero.
__global__ void k_standardize(const float *__restrict__ feat, const float *__restrict__ norm, int64_t n,
                              int64_t rows, float *__restrict__ X0) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * kMlpIn) return;
    const int64_t r = i / kMlpIn;
    const int c = (int)(i % kMlpIn);
    const float v = r < n ? (feat[i] - norm[c]) * norm[kMlpIn + c] : 0.0f;
    X0[i] = v;
}

// y[r] = H3[r] . w4 + b4, one wave per row.
__global__ __launch_bounds__(256) void k_head(const float *__restrict__ H3, const float *__restrict__ P, int64_t n,
                                              float *__restrict__ y) {
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= n) return;
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < kMlpH / 64; ++k) {
        const int c = k * 64 + lane;
        acc += H3[r * kMlpH + c] * P[kOffW4 + c];
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) y[r] = acc + P[kOffB4];
}

// Loss and head backward.  dy = 2 (yhat - y) / n; per row r < n:
//   dZ3[r][c] = dy w4[c] silu'(Z3[r][c])  (also transposed into dZ3t).
// Block b (64 rows) writes its sums over those rows to part[b][0..257]:
// grad(w4)[c] (c < 256), grad(b4) (256) and the loss (257); k_head_sums adds
// the blocks in order (no float atomics: the result is deterministic).
constexpr int kHeadCols = kMlpH + 2;
__global__ __launch_bounds__(256) void k_head_backward(const float *__restrict__ yhat, const float *__restrict__ y,
                                                       int64_t n, int64_t rows, const float *__restrict__ Z3,
                                                       const float *__restrict__ H3, const float *__restrict__ P,
                                                       float *__restrict__ dZ3, float *__restrict__ dZ3t,
                                                       float *__restrict__ part) {
    // one block per 64 rows; thread c handles column c of those rows
    const int c = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const float w4 = P[kOffW4 + c];
    float gw = 0.0f, gb = 0.0f, ls = 0.0f;
    for (int k = 0; k < 64; ++k) {
        const int64_t r = r0 + k;
        float dz = 0.0f;
        if (r < n) {
            const float e = yhat[r] - y[r];
            const float dy = 2.0f * e / (float)n;
            dz = dy * w4 * silu_grad(Z3[r * kMlpH + c]);
            gw += dy * H3[r * kMlpH + c];
            if (c == 0) {
                gb += dy;
                ls += e * e / (float)n;
            }
        }
        const float b = dz;
        dZ3[r * kMlpH + c] = b;
        dZ3t[(int64_t)c * rows + r] = b;
    }
    float *out = part + (int64_t)blockIdx.x * kHeadCols;
    out[c] = gw;
    if (c == 0) {
        out[kMlpH] = gb;
        out[kMlpH + 1] = ls;
    }
}

// G[kOffW4 + c] (c <= 256: w4 then b4) and the loss from the per-block
// partials, summed over blocks in order.
// 64 columns per block; the four waves sum the blocks b = q, q + 4, ... in
// order (eight loads in flight), and their sums are added in wave order.
__global__ __launch_bounds__(256) void k_head_sums(const float *__restrict__ part, int nblocks,
                                                   float *__restrict__ G, float *__restrict__ loss) {
    __shared__ float sh[4][64];
    const int l = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int c = blockIdx.x * 64 + l;
    float s = 0.0f;
    if (c < kHeadCols) {
        int b = q;
        for (; b + 28 < nblocks; b += 32) {
            float x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = part[(int64_t)(b + 4 * k) * kHeadCols + c];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += x[k];
        }
        for (; b < nblocks; b += 4) s += part[(int64_t)b * kHeadCols + c];
    }
    sh[q][l] = s;
    __syncthreads();
    if (q == 0 && c < kHeadCols) {
        const float t = ((sh[0][l] + sh[1][l]) + sh[2][l]) + sh[3][l];
        if (c < kMlpH + 1)
            G[kOffW4 + c] = t;
        else
            *loss = t;
    }
}

// dZ = dH * silu'(Z) for a hidden layer; writes dZ and its transpose.
__global__ void k_act_backward(const float *__restrict__ dH, const float *__restrict__ Z, int64_t n, int64_t rows,
                               float *__restrict__ dZ, float *__restrict__ dZt) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * kMlpH) return;
    const int64_t r = i / kMlpH;
    const int c = (int)(i % kMlpH);
    const float v = r < n ? dH[i] * silu_grad(Z[i]) : 0.0f;
    const float b = v;
    dZ[i] = b;
    dZt[(int64_t)c * rows + r] = b;
}

// out[c][r] = in[r][c] for a rows x cols matrix.
__global__ void k_transpose(const float *__restrict__ in, int64_t rows, int cols, float *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * cols) return;
    const int64_t r = i / cols;
    const int c = (int)(i % cols);
    out[(int64_t)c * rows + r] = in[i];
}

// grad(b)[c] = sum_r dZt[c][r]: one block per output c, fixed order.
__global__ __launch_bounds__(256) void k_bias_grad(const float *__restrict__ dZt, int64_t rows, float *__restrict__ g) {
    __shared__ float sh[256];
    const int c = blockIdx.x;
    float s = 0.0f;
    for (int64_t r = threadIdx.x; r < rows; r += 256) s += dZt[(int64_t)c * rows + r];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) g[c] = sh[0];
}

// Adam (Kingma & Ba) with bias correction; m and v follow P in `adam`.
// omb1 = 1 - beta1 and omb2 = 1 - beta2 come from the host rounded once from
// double (1.0f - 0.999f in float32 would be 5e-5 off 0.001).
struct AdamStep {
    float lr, b1, b2, omb1, omb2, eps, c1, c2;
};
static AdamStep adam_step(float lr, int64_t step) {
    const double b1 = 0.9, b2 = 0.999;
    return {lr,   (float)b1, (float)b2, (float)(1.0 - b1), (float)(1.0 - b2), 1e-8f, (float)(1.0 - std::pow(b1, (double)step)),
            (float)(1.0 - std::pow(b2, (double)step))};
}

__device__ __forceinline__ void adam_update(float *__restrict__ P, float *__restrict__ adam, int64_t i, float g,
                                            const AdamStep &a) {
    const float m = a.b1 * adam[i] + a.omb1 * g;
    const float v = a.b2 * adam[kMlpParams + i] + a.omb2 * (g * g);
    adam[i] = m;
    adam[kMlpParams + i] = v;
    P[i] -= a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
}

__global__ void k_adam(float *__restrict__ P, float *__restrict__ adam, const float *__restrict__ G, AdamStep a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMlpParams) adam_update(P, adam, i, G[i], a);
}

// Deterministic initialisation: uniform(-a, a) with a = sqrt(6 / (fan_in + fan_out))
// for weights (24 bits of a 64-bit finaliser of seed and parameter index:
// MurmurHash3's fmix64), zero biases.
__device__ __forceinline__ uint32_t mix32(uint64_t x) {
    x ^= x >> 33;
    x *= 0xff51afd7ed558ccdull;
    x ^= x >> 33;
    x *= 0xc4ceb9fe1a85ec53ull;
    x ^= x >> 33;
    return (uint32_t)x;
}
__global__ void k_mlp_init(float *__restrict__ P, uint64_t seed) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kMlpParams) return;
    float fan_in = 0, fan_out = 0;
    bool weight = true;
    if (i < kOffB1) { fan_in = kMlpIn; fan_out = kMlpH; }
    else if (i < kOffW2) weight = false;
    else if (i < kOffB2) { fan_in = kMlpH; fan_out = kMlpH; }
    else if (i < kOffW3) weight = false;
    else if (i < kOffB3) { fan_in = kMlpH; fan_out = kMlpH; }
    else if (i < kOffW4) weight = false;
    else if (i < kOffB4) { fan_in = kMlpH; fan_out = 1; }
    else weight = false;
    if (!weight) {
        P[i] = 0.0f;
        return;
    }
    const float a = sqrtf(6.0f / (fan_in + fan_out));
    const float u = (float)(mix32(seed * 0x9E3779B97F4A7C15ull + (uint64_t)i) >> 8) * (1.0f / 16777216.0f);
    P[i] = (2.0f * u - 1.0f) * a;
}

// ---------------------------------------------------------------------------
// Training scratch for `rows` rows: the FP32 step's arrays, which the BF16 step
// and inference need less than (split_count ranges of gradients take at most
// what kMaxSplits ranges of one layer and three FP32 pre-activations do).
size_t mlp_scratch_bytes(int64_t rows) {
    const size_t h = (size_t)rows * kMlpH;
    size_t b = 0;
    b += 2 * (size_t)kMlpH * kMlpIn + 4 * (size_t)kMlpH * kMlpH;   // weights and transposes
    b += (size_t)rows * kMlpIn * 2;                                // X0, X0t
    b += 3 * h;                                                    // Z1..Z3
    b += 4 * h;                                                    // H1..H3, transposed H
    b += (size_t)rows;                                             // yhat
    b += 3 * h;                                                    // dZ, dZt, dH
    b += (size_t)kMlpParams;                                       // gradient buffer
    b += (size_t)kMaxSplits * kMlpH * kMlpH;                       // split-K partial products
    b += (size_t)(rows / 64 + 1) * kHeadCols;                      // head partials per block
    return b * 4 + 64 * 256;
}

struct Carver {
    char *p;
    size_t off = 0;
    template <typename T>
    T *take(size_t count) {
        off = (off + 255) & ~(size_t)255;
        T *r = (T *)(p + off);
        off += count * sizeof(T);
        return r;
    }
};

struct MlpBufs {
    float *W1, *W2, *W3, *W2t, *W3t, *X0, *X0t, *H1, *H2, *H3, *Ht, *dZ, *dZt;
    float *Z1, *Z2, *Z3, *yhat, *dH, *G, *Gpart, *Hpart;
};

static MlpBufs carve_mlp(void *base, int64_t rows) {
    Carver c{(char *)base};
    const size_t h = (size_t)rows * kMlpH;
    MlpBufs m;
    m.W1 = c.take<float>((size_t)kMlpH * kMlpIn);
    m.W2 = c.take<float>((size_t)kMlpH * kMlpH);
    m.W3 = c.take<float>((size_t)kMlpH * kMlpH);
    m.W2t = c.take<float>((size_t)kMlpH * kMlpH);
    m.W3t = c.take<float>((size_t)kMlpH * kMlpH);
    m.X0 = c.take<float>((size_t)rows * kMlpIn);
    m.X0t = c.take<float>((size_t)rows * kMlpIn);
    m.Z1 = c.take<float>(h);
    m.Z2 = c.take<float>(h);
    m.Z3 = c.take<float>(h);
    m.H1 = c.take<float>(h);
    m.H2 = c.take<float>(h);
    m.H3 = c.take<float>(h);
    m.Ht = c.take<float>(h);
    m.yhat = c.take<float>((size_t)rows);
    m.dZ = c.take<float>(h);
    m.dZt = c.take<float>(h);
    m.dH = c.take<float>(h);
    m.G = c.take<float>((size_t)kMlpParams);
    m.Gpart = c.take<float>((size_t)kMaxSplits * kMlpH * kMlpH);
    m.Hpart = c.take<float>((size_t)(rows / 64 + 1) * kHeadCols);
    return m;
}

static inline unsigned blocks_for(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

static void mlp_forward_rows(const float *P, const MlpBufs &m, int64_t rows, hipStream_t st) {
    const int H = kMlpH;
    gemm_nt(1, m.X0, kMlpIn, m.W1, kMlpIn, rows, H, kMlpIn, m.Z1, H, P + kOffB1, m.H1, H, st);
    gemm_nt(1, m.H1, H, m.W2, H, rows, H, H, m.Z2, H, P + kOffB2, m.H2, H, st);
    gemm_nt(1, m.H2, H, m.W3, H, rows, H, H, m.Z3, H, P + kOffB3, m.H3, H, st);
}

// ---------------------------------------------------------------------------
// BF16 network, all layers of a block of rows in one kernel.
//
// The activations of the block's rows stay in LDS as one row-major bf16 buffer
// (padded row stride, so the 16 rows a fragment load reads fall on different
// banks) that holds the input, then each layer's output in place: a layer's
// products are finished in registers, the block meets at a barrier, and only
// then are they written over its input.  The bf16 weights are read straight
// from global memory (L2); wave w computes output columns [32 w, 32 w + 32).
//
// The products are taken transposed (the weights as the first operand of
// v_mfma_f32_16x16x32_bf16, the activations as the second): lane l gives 8
// consecutive k, from 8 (l / 16), of row l % 16 of either operand, and of a
// 16x16 output tile it holds four consecutive output columns 4 (l / 16) .. + 3
// of row l % 16, which go to LDS as one 8-byte store and are the layout the
// next layer reads.
constexpr int kFuseWaves = 8, kFuseThreads = 64 * kFuseWaves;
constexpr int kFuseCols = kMlpH / kFuseWaves / 16;   // 16-column tiles per wave
constexpr int kFusePitch = kMlpH + 8;                // bf16 per LDS row

// The wave's weights of a layer: fragments of 32 k by 16 columns.
template <int kK>
__device__ __forceinline__ void fused_weights(const __bf16 *__restrict__ W, int w, int lane,
                                              bf16x8 (&b)[kMlpH / 32][kFuseCols]) {
#pragma unroll
    for (int k = 0; k < kK / 32; ++k)
#pragma unroll
        for (int j = 0; j < kFuseCols; ++j)
            b[k][j] = *reinterpret_cast<const bf16x8 *>(W + (int64_t)(16 * (kFuseCols * w + j) + (lane & 15)) * kK +
                                                        32 * k + (lane >> 4) * 8);
}

// The lane's four values of a 1-D array of kMlpH columns, per column tile.
__device__ __forceinline__ void fused_columns(const float *__restrict__ x, int w, int lane,
                                              float (&v)[kFuseCols][4]) {
#pragma unroll
    for (int j = 0; j < kFuseCols; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[j][r] = x[16 * kFuseCols * w + 16 * j + (lane >> 4) * 4 + r];
}

// Writes the block's new activations over the old ones, bracketed by barriers.
template <int kTiles, typename F>
__device__ __forceinline__ void fused_store(__bf16 (*Out)[kFusePitch], int w, int lane, F &&value) {
    const int fr = lane & 15, g4 = (lane >> 4) * 4;
    __syncthreads();            // every wave has read the layer's input
#pragma unroll
    for (int i = 0; i < kTiles; ++i)
#pragma unroll
        for (int j = 0; j < kFuseCols; ++j) {
            const bf16x4 v = {(__bf16)value(i, j, 0), (__bf16)value(i, j, 1), (__bf16)value(i, j, 2),
                              (__bf16)value(i, j, 3)};
            *reinterpret_cast<bf16x4 *>(&Out[16 * i + fr][16 * kFuseCols * w + 16 * j + g4]) = v;
        }
    __syncthreads();
}

// Inference.  A million rows take at least 0.20 ms of matrix instructions and
// about 0.25 ms of vector instructions (SiLU's exponential alone takes 1.9 issue
// slots, measured), so the two have to overlap: a wave holds a layer's weights for
// its 32 columns in registers (the next layer's are on their way) and goes through
// the 128 rows 16 at a time, with the SiLU of one 16-row tile beside the products of
// the next.  Layers alternate between two LDS buffers,
// so one barrier per layer is enough; 136 KB make one block per CU, which goes
// through row blocks in turn with the next block's features already loading.
// With the products of all rows first, one buffer and 2 blocks of 4 waves per
// CU, a million rows took 620 us; this takes 440.
constexpr int kFuseTiles = 8;                 // 16-row fragment tiles per block
constexpr int kFuseRows = 16 * kFuseTiles;
constexpr int kFuseBlocks = 256;
constexpr int kFuseIn = kFuseRows * kMlpIn / kFuseThreads;   // input values per thread

// out(i, x): x[j][r] = SiLU of the wave's outputs of row tile i.
template <int kK, typename F>
__device__ __forceinline__ void fused_layer(const __bf16 (*In)[kFusePitch], const bf16x8 (&b)[kMlpH / 32][kFuseCols],
                                            const float *__restrict__ bias, int w, int lane, F &&out) {
    float bj[kFuseCols][4];
    fused_columns(bias, w, lane, bj);
    f32x4 prev[kFuseCols], acc[kFuseCols];
#pragma unroll
    for (int i = 0; i <= kFuseTiles; ++i) {
        if (i < kFuseTiles) {
#pragma unroll
            for (int j = 0; j < kFuseCols; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < kK / 32; ++k) {
                const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&In[16 * i + (lane & 15)][32 * k + (lane >> 4) * 8]);
#pragma unroll
                for (int j = 0; j < kFuseCols; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[k][j], a, acc[j], 0, 0, 0);
            }
        }
        if (i > 0) {
#pragma unroll
            for (int j = 0; j < kFuseCols; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) prev[j][r] = silu(prev[j][r] + bj[j][r]);
            out(i - 1, prev);
        }
#pragma unroll
        for (int j = 0; j < kFuseCols; ++j) prev[j] = acc[j];
    }
}

__global__ __launch_bounds__(kFuseThreads, 2) void k_mlp_fused(const float *__restrict__ feat,
                                                               const float *__restrict__ norm, int64_t n,
                                                               const __bf16 *__restrict__ W1,
                                                               const __bf16 *__restrict__ W2,
                                                               const __bf16 *__restrict__ W3,
                                                               const float *__restrict__ P, float *__restrict__ y) {
    static_assert(kMlpIn == 64, "a lane per input column");
    __shared__ __attribute__((aligned(16))) __bf16 buf[2][kFuseRows][kFusePitch];
    __shared__ float ypart[kFuseWaves][kFuseRows];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, fr = lane & 15, g4 = (lane >> 4) * 4;
    const int64_t step = (int64_t)gridDim.x * kFuseRows;
    const float mean = norm[lane], inv_std = norm[kMlpIn + lane];
    float x[kFuseIn];           // row w + 8 q, column lane of a block; rows past n are zero
    auto load_x = [&](int64_t r0) {
#pragma unroll
        for (int q = 0; q < kFuseIn; ++q) {
            const int64_t row = r0 + w + kFuseWaves * q;
            x[q] = row < n ? feat[row * kMlpIn + lane] : mean;
        }
    };
    auto put_x = [&](__bf16 (*H)[kFusePitch]) {
#pragma unroll
        for (int q = 0; q < kFuseIn; ++q) H[w + kFuseWaves * q][lane] = (__bf16)((x[q] - mean) * inv_std);
    };
    bf16x8 ba[kMlpH / 32][kFuseCols], bb[kMlpH / 32][kFuseCols];
    load_x((int64_t)blockIdx.x * kFuseRows);
    fused_weights<kMlpIn>(W1, w, lane, ba);
    put_x(buf[0]);
    __syncthreads();
    int in = 0;
    for (int64_t r0 = (int64_t)blockIdx.x * kFuseRows; r0 < n; r0 += step, in ^= 1) {
        __bf16(*A)[kFusePitch] = buf[in], (*B)[kFusePitch] = buf[in ^ 1];
        auto store = [&](__bf16 (*H)[kFusePitch], int i, const f32x4 (&v)[kFuseCols]) {
#pragma unroll
            for (int j = 0; j < kFuseCols; ++j) {
                const bf16x4 h = {(__bf16)v[j][0], (__bf16)v[j][1], (__bf16)v[j][2], (__bf16)v[j][3]};
                *reinterpret_cast<bf16x4 *>(&H[16 * i + fr][16 * (kFuseCols * w + j) + g4]) = h;
            }
        };
        fused_weights<kMlpH>(W2, w, lane, bb);
        fused_layer<kMlpIn>(A, ba, P + kOffB1, w, lane, [&](int i, const f32x4 (&v)[kFuseCols]) { store(B, i, v); });
        __syncthreads();
        fused_weights<kMlpH>(W3, w, lane, ba);
        load_x(r0 + step);
        fused_layer<kMlpH>(B, bb, P + kOffB2, w, lane, [&](int i, const f32x4 (&v)[kFuseCols]) { store(A, i, v); });
        __syncthreads();
        put_x(B);
        // head: this wave's columns of each row, then over the four lanes of the
        // row, then over the waves
        float w4[kFuseCols][4];
        fused_columns(P + kOffW4, w, lane, w4);
#pragma unroll
        for (int j = 0; j < kFuseCols; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) w4[j][r] = (float)(__bf16)w4[j][r];
        fused_layer<kMlpH>(A, ba, P + kOffB3, w, lane, [&](int i, const f32x4 (&v)[kFuseCols]) {
            float s = 0.0f;
#pragma unroll
            for (int j = 0; j < kFuseCols; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) s += (float)(__bf16)v[j][r] * w4[j][r];
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (lane < 16) ypart[w][16 * i + lane] = s;
        });
        fused_weights<kMlpIn>(W1, w, lane, ba);
        __syncthreads();
        if (threadIdx.x < kFuseRows && r0 + threadIdx.x < n) {
            const int t = threadIdx.x;
            y[r0 + t] = (((ypart[0][t] + ypart[1][t]) + (ypart[2][t] + ypart[3][t])) +
                         ((ypart[4][t] + ypart[5][t]) + (ypart[6][t] + ypart[7][t]))) +
                        P[kOffB4];
        }
    }
}

// Training: forward, loss and backward of 64 rows per block, so a batch of
// 16 384 rows is one block on each CU.  The pre-activations of the three layers
// stay in registers (32 per layer and lane) until their SiLU derivative is
// taken; what the weight gradients need (standardised inputs, H1, H2 and the
// three dZ, in BF16) is written in groups of eight rows, [row / 8][column][8],
// which is what their products read (8 consecutive rows of a column per lane).
// One product, transpose or activation per kernel went through FP32 Z and dH in
// memory and transposed with 2-byte stores a batch apart: 27 launches,
// 380 us for 16 384 rows; the four launches here take 70 (this kernel 42, the
// products 16), 65 536 rows 1480 -> 220.
//
// With dy = 2 (yhat - y) / n:  dZ3[r][c] = dy w4[c] silu'(Z3[r][c]),
// dZk = (dZ(k+1) W(k+1)) silu'(Zk); rows from n on have dZ = 0.
// Each half of 32 rows writes its sums to part[2 block + half][...]: the bias
// gradients b1, b2, b3 and grad(w4) (kMlpH each), grad(b4), and the loss (no
// float atomics: fixed order, so the result is deterministic).
constexpr int kTrainTiles = 4, kTrainRows = 16 * kTrainTiles;
constexpr int kPartCols = 4 * kMlpH + 2;

struct TrainBufs {
    __bf16 *W1, *W2, *W3, *W2t, *W3t;          // weights and transposes
    __bf16 *X0, *H1, *H2, *dZ1, *dZ2, *dZ3;    // groups of eight rows
    float *part;                               // [2 rows / 64][kPartCols]
    float *grad;                               // [splits][kMlpParams + 1]: gradient and loss of a range of rows
};

static TrainBufs carve_train(void *base, int64_t rows, int splits) {
    Carver c{(char *)base};
    const size_t h = (size_t)rows * kMlpH;
    TrainBufs m;
    m.W1 = c.take<__bf16>((size_t)kMlpH * kMlpIn);
    m.W2 = c.take<__bf16>((size_t)kMlpH * kMlpH);
    m.W3 = c.take<__bf16>((size_t)kMlpH * kMlpH);
    m.W2t = c.take<__bf16>((size_t)kMlpH * kMlpH);
    m.W3t = c.take<__bf16>((size_t)kMlpH * kMlpH);
    m.X0 = c.take<__bf16>((size_t)rows * kMlpIn);
    m.H1 = c.take<__bf16>(h);
    m.H2 = c.take<__bf16>(h);
    m.dZ1 = c.take<__bf16>(h);
    m.dZ2 = c.take<__bf16>(h);
    m.dZ3 = c.take<__bf16>(h);
    m.part = c.take<float>((size_t)(rows / kTrainRows) * 2 * kPartCols);
    m.grad = c.take<float>((size_t)splits * (kMlpParams + 1));
    return m;
}

// The weights are loaded a k step ahead rather than a layer ahead: a layer's 64
// registers beside the three layers' pre-activations spill (48 us against 42).
template <int kK>
__device__ __forceinline__ void train_product(const __bf16 (*In)[kFusePitch], const __bf16 *__restrict__ W, int w,
                                              int lane, f32x4 (&acc)[kTrainTiles][kFuseCols]) {
    const int fr = lane & 15, fk = (lane >> 4) * 8;
#pragma unroll
    for (int i = 0; i < kTrainTiles; ++i)
#pragma unroll
        for (int j = 0; j < kFuseCols; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const __bf16 *wrow = W + (int64_t)(16 * kFuseCols * w + fr) * kK + fk;
    bf16x8 b[kFuseCols], bn[kFuseCols];
#pragma unroll
    for (int j = 0; j < kFuseCols; ++j) b[j] = *reinterpret_cast<const bf16x8 *>(wrow + 16 * j * kK);
    for (int k0 = 0; k0 < kK; k0 += 32) {
        if (k0 + 32 < kK) {
#pragma unroll
            for (int j = 0; j < kFuseCols; ++j) bn[j] = *reinterpret_cast<const bf16x8 *>(wrow + 16 * j * kK + k0 + 32);
        }
#pragma unroll
        for (int i = 0; i < kTrainTiles; ++i) {
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&In[16 * i + fr][k0 + fk]);
#pragma unroll
            for (int j = 0; j < kFuseCols; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a, acc[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < kFuseCols; ++j) b[j] = bn[j];
    }
}

// Copies the block's activations to `dst` in groups of eight rows; thread t
// takes column t % 256 of the half t / 256 of the rows.  Returns the sum of
// what it copied.
__device__ __forceinline__ float fused_copy_out(const __bf16 (*H)[kFusePitch], __bf16 *__restrict__ dst,
                                                int64_t r0) {
    const int c = threadIdx.x & (kMlpH - 1), half = threadIdx.x / kMlpH;
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < kTrainRows / 16; ++q) {
        const int g = half * (kTrainRows / 16) + q;
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[e] = H[8 * g + e][c];
            s += (float)v[e];
        }
        *reinterpret_cast<bf16x8 *>(dst + ((r0 / 8 + g) * kMlpH + c) * 8) = v;
    }
    return s;
}

__global__ __launch_bounds__(kFuseThreads, 2) void k_mlp_train(const float *__restrict__ feat,
                                                               const float *__restrict__ norm,
                                                               const float *__restrict__ y, int64_t n,
                                                               const float *__restrict__ P, TrainBufs m) {
    static_assert(kFuseThreads == 2 * kMlpH && kTrainRows == 64 && kMlpIn == 64, "thread maps of this kernel");
    __shared__ __attribute__((aligned(16))) __bf16 H[kTrainRows][kFusePitch];
    __shared__ float err[kTrainRows], dy[kTrainRows];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, fr = lane & 15;
    const int c = threadIdx.x & (kMlpH - 1), half = threadIdx.x / kMlpH;
    const int64_t r0 = (int64_t)blockIdx.x * kTrainRows;
    float *part = m.part + ((int64_t)blockIdx.x * 2 + half) * kPartCols;
    {   // standardised inputs: wave w takes rows 8 w .. 8 w + 7, a lane per column
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t row = r0 + 8 * w + e;
            const float x = row < n ? (feat[row * kMlpIn + lane] - norm[lane]) * norm[kMlpIn + lane] : 0.0f;
            v[e] = (__bf16)x;
            H[8 * w + e][lane] = v[e];
        }
        *reinterpret_cast<bf16x8 *>(m.X0 + ((r0 / 8 + w) * kMlpIn + lane) * 8) = v;
    }
    __syncthreads();
    f32x4 z1[kTrainTiles][kFuseCols], z2[kTrainTiles][kFuseCols], z3[kTrainTiles][kFuseCols];
    auto add_bias = [&](f32x4 (&z)[kTrainTiles][kFuseCols], const float *bias) {
        float bj[kFuseCols][4];
        fused_columns(bias, w, lane, bj);
#pragma unroll
        for (int i = 0; i < kTrainTiles; ++i)
#pragma unroll
            for (int j = 0; j < kFuseCols; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) z[i][j][r] += bj[j][r];
    };
    train_product<kMlpIn>(H, m.W1, w, lane, z1);
    add_bias(z1, P + kOffB1);
    fused_store<kTrainTiles>(H, w, lane, [&](int i, int j, int r) { return silu(z1[i][j][r]); });
    fused_copy_out(H, m.H1, r0);
    train_product<kMlpH>(H, m.W2, w, lane, z2);
    add_bias(z2, P + kOffB2);
    fused_store<kTrainTiles>(H, w, lane, [&](int i, int j, int r) { return silu(z2[i][j][r]); });
    fused_copy_out(H, m.H2, r0);
    train_product<kMlpH>(H, m.W3, w, lane, z3);
    add_bias(z3, P + kOffB3);
    fused_store<kTrainTiles>(H, w, lane, [&](int i, int j, int r) { return silu(z3[i][j][r]); });
    // head: wave w takes rows 8 w .. 8 w + 7
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int r = 8 * w + e;
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < kMlpH / 64; ++k)
            acc += (float)H[r][k * 64 + lane] * (float)(__bf16)P[kOffW4 + k * 64 + lane];
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
        if (lane == 0) {
            const float d = r0 + r < n ? acc + P[kOffB4] - y[r0 + r] : 0.0f;
            err[r] = d;
            dy[r] = r0 + r < n ? 2.0f * d / (float)n : 0.0f;
        }
    }
    __syncthreads();
    {
        float gw = 0.0f;
        for (int k = 0; k < kTrainRows / 2; ++k) {
            const int r = half * (kTrainRows / 2) + k;
            if (r0 + r < n) gw += dy[r] * (float)H[r][c];
        }
        part[3 * kMlpH + c] = gw;
        if ((w & 3) == 0) {     // one wave of each half: its 32 rows
            const int r = half * (kTrainRows / 2) + (lane & 31);
            float gb = dy[r], ls = err[r] * err[r] / (float)n;
            for (int off = 16; off > 0; off >>= 1) {
                gb += __shfl_xor(gb, off);
                ls += __shfl_xor(ls, off);
            }
            if (lane == 0) {
                part[4 * kMlpH] = gb;
                part[4 * kMlpH + 1] = ls;
            }
        }
    }
    float w4[kFuseCols][4];
    fused_columns(P + kOffW4, w, lane, w4);
    fused_store<kTrainTiles>(H, w, lane, [&](int i, int j, int r) {
        const int row = 16 * i + fr;
        return r0 + row < n ? dy[row] * (float)(__bf16)w4[j][r] * silu_grad(z3[i][j][r]) : 0.0f;
    });
    part[2 * kMlpH + c] = fused_copy_out(H, m.dZ3, r0);
    train_product<kMlpH>(H, m.W3t, w, lane, z3);
    fused_store<kTrainTiles>(H, w, lane, [&](int i, int j, int r) {
        return r0 + 16 * i + fr < n ? z3[i][j][r] * silu_grad(z2[i][j][r]) : 0.0f;
    });
    part[kMlpH + c] = fused_copy_out(H, m.dZ2, r0);
    train_product<kMlpH>(H, m.W2t, w, lane, z3);
    fused_store<kTrainTiles>(H, w, lane, [&](int i, int j, int r) {
        return r0 + 16 * i + fr < n ? z3[i][j][r] * silu_grad(z1[i][j][r]) : 0.0f;
    });
    part[c] = fused_copy_out(H, m.dZ1, r0);
}

// Weight gradients dZ^T H of the three layers, 64x64 tiles over a range of
// rows: block (z, t) takes tile t of W2 (16), W3 (16) and W1 (4) over the rows
// [z kchunk, (z + 1) kchunk), and t = kGradTiles sums the per-block partials of
// those rows, so grad[z] is the whole gradient (and loss) of range z.  One
// launch of 37 blocks per range keeps the chip filled, and the ranges, which
// the index deals over the XCDs, are read by all their tiles through one L2.
constexpr int kGradTiles = 36;
__global__ __launch_bounds__(256) void k_mlp_grad(TrainBufs m, int64_t rows, int64_t kchunk) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, t = blockIdx.y;
    const int64_t kb = (int64_t)blockIdx.x * kchunk, ke = min(rows, kb + kchunk);
    float *out = m.grad + (int64_t)blockIdx.x * (kMlpParams + 1);
    if (t == kGradTiles) {
        const int p0 = (int)(kb / (kTrainRows / 2)), p1 = (int)(ke / (kTrainRows / 2));
        for (int c = threadIdx.x; c < kPartCols; c += 256) {
            float s = 0.0f;
#pragma unroll 8
            for (int p = p0; p < p1; ++p) s += m.part[(int64_t)p * kPartCols + c];
            const int which = c / kMlpH, k = c % kMlpH;
            out[which == 0 ? kOffB1 + k : which == 1 ? kOffB2 + k : which == 2 ? kOffB3 + k : kOffW4 + (c - 3 * kMlpH)] =
                s;
        }
        return;
    }
    static_assert(kOffB4 == kOffW4 + kMlpH && kMlpParams == kOffB4 + 1, "w4, b4 and the loss follow each other");
    const __bf16 *A = t < 16 ? m.dZ2 : (t < 32 ? m.dZ3 : m.dZ1), *B = t < 16 ? m.H1 : (t < 32 ? m.H2 : m.X0);
    const int nb = t < 32 ? kMlpH : kMlpIn;
    const int row0 = (t < 32 ? (t >> 2) & 3 : t - 32) * 64 + (w & 1) * 32;
    const int col0 = (t < 32 ? t & 3 : 0) * 64 + (w >> 1) * 32;
    out += t < 16 ? kOffW2 : (t < 32 ? kOffW3 : kOffW1);
    const int fr = lane & 15, fg = lane >> 4;
    const __bf16 *a = A + ((kb / 8 + fg) * kMlpH + row0 + fr) * 8;
    const __bf16 *b = B + ((kb / 8 + fg) * nb + col0 + fr) * 8;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // 64 rows at a time, the next 64 loading
    bf16x8 fa[2][2], fb[2][2], na[2][2], nb8[2][2];
    auto load = [&](bf16x8 (&xa)[2][2], bf16x8 (&xb)[2][2]) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                xa[k][i] = *reinterpret_cast<const bf16x8 *>(a + (4 * k * kMlpH + 16 * i) * 8);
                xb[k][i] = *reinterpret_cast<const bf16x8 *>(b + (4 * k * nb + 16 * i) * 8);
            }
    };
    const int blocks = (int)((ke - kb) / kTrainRows);
    load(fa, fb);
    for (int q = 0; q < blocks; ++q) {
        a += 8 * kMlpH * 8;
        b += 8 * nb * 8;
        if (q + 1 < blocks) load(na, nb8);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[k][i], fb[k][j], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                fa[k][i] = na[k][i];
                fb[k][i] = nb8[k][i];
            }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                out[(int64_t)(row0 + 16 * i + fg * 4 + r) * nb + col0 + 16 * j + fr] = acc[i][j][r];
}

// Sums the ranges in order: the gradient (to grad_out, and one Adam step, where
// wanted) and the loss.
__global__ __launch_bounds__(256) void k_mlp_finish(const float *__restrict__ grad, int splits, float *__restrict__ P,
                                                    float *__restrict__ adam, AdamStep a,
                                                    float *__restrict__ grad_out, float *__restrict__ loss) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i > kMlpParams) return;
    float g = 0.0f;
#pragma unroll 8
    for (int z = 0; z < splits; ++z) g += grad[(int64_t)z * (kMlpParams + 1) + i];
    if (i == kMlpParams) {
        *loss = g;
        return;
    }
    if (grad_out) grad_out[i] = g;
    if (adam) adam_update(P, adam, i, g, a);
}

void mlp_init(float *params, uint64_t seed, hipStream_t st) {
    hipLaunchKernelGGL(k_mlp_init, dim3(blocks_for(kMlpParams)), dim3(256), 0, st, params, seed);
}

// Predictions for n rows of raw features: the bf16 weights, then one fused
// launch over every row (the scratch holds only the weights).
void mlp_forward(const float *P, const float *feat, const float *norm, int64_t n, float *y, void *scratch,
                 int64_t rows, hipStream_t st) {
    const TrainBufs m = carve_train(scratch, rows, 1);
    hipLaunchKernelGGL((k_weights_cast<__bf16, false>), dim3(kCastBlocks), dim3(256), 0, st, P, m.W1, m.W2, m.W3,
                       m.W2t, m.W3t);
    const unsigned blocks = (unsigned)std::min<int64_t>(kFuseBlocks, (n + kFuseRows - 1) / kFuseRows);
    hipLaunchKernelGGL(k_mlp_fused, dim3(blocks), dim3(kFuseThreads), 0, st, feat, norm, n, m.W1, m.W2, m.W3, P, y);
}

// Loss and gradient on one batch of n <= rows rows in FP32, and one Adam step
// (step >= 1) if adam != nullptr.  grad_out (optional) receives the gradient.
// Every sum has a fixed order, so two calls on the same inputs give the same
// bits.
static void train_step_fp32(float *P, float *adam, int64_t step, float lr, const float *feat, const float *norm,
                            const float *y, int64_t n, float *loss, float *grad_out, void *scratch, int64_t rows,
                            hipStream_t st) {
    const MlpBufs m = carve_mlp(scratch, rows);
    const int H = kMlpH;
    const int64_t R = (n + 63) / 64 * 64;
    hipLaunchKernelGGL((k_weights_cast<float, true>), dim3(kCastBlocks), dim3(256), 0, st, P, m.W1, m.W2, m.W3, m.W2t,
                       m.W3t);
    hipLaunchKernelGGL(k_standardize, dim3(blocks_for(R * kMlpIn)), dim3(256), 0, st, feat, norm, n, R, m.X0);
    mlp_forward_rows(P, m, R, st);
    hipLaunchKernelGGL(k_head, dim3((unsigned)((R + 3) / 4)), dim3(256), 0, st, m.H3, P, R, m.yhat);
    hipLaunchKernelGGL(k_head_backward, dim3((unsigned)(R / 64)), dim3(256), 0, st, m.yhat, y, n, R, m.Z3, m.H3, P,
                       m.dZ, m.dZt, m.Hpart);
    hipLaunchKernelGGL(k_head_sums, dim3((kHeadCols + 63) / 64), dim3(256), 0, st, m.Hpart, (int)(R / 64), m.G, loss);
    // layer 3: grad W3 = dZ3^T H2, grad b3, dH2 = dZ3 W3
    hipLaunchKernelGGL(k_transpose, dim3(blocks_for(R * H)), dim3(256), 0, st, m.H2, R, H, m.Ht);
    gemm_nt_splitk(m.dZt, (int)R, m.Ht, (int)R, H, H, (int)R, m.Gpart, m.G + kOffW3, st);
    hipLaunchKernelGGL(k_bias_grad, dim3(H), dim3(256), 0, st, m.dZt, R, m.G + kOffB3);
    gemm_nt(0, m.dZ, H, m.W3t, H, R, H, H, m.dH, H, nullptr, nullptr, 0, st);
    hipLaunchKernelGGL(k_act_backward, dim3(blocks_for(R * H)), dim3(256), 0, st, m.dH, m.Z2, n, R, m.dZ, m.dZt);
    // layer 2
    hipLaunchKernelGGL(k_transpose, dim3(blocks_for(R * H)), dim3(256), 0, st, m.H1, R, H, m.Ht);
    gemm_nt_splitk(m.dZt, (int)R, m.Ht, (int)R, H, H, (int)R, m.Gpart, m.G + kOffW2, st);
    hipLaunchKernelGGL(k_bias_grad, dim3(H), dim3(256), 0, st, m.dZt, R, m.G + kOffB2);
    gemm_nt(0, m.dZ, H, m.W2t, H, R, H, H, m.dH, H, nullptr, nullptr, 0, st);
    hipLaunchKernelGGL(k_act_backward, dim3(blocks_for(R * H)), dim3(256), 0, st, m.dH, m.Z1, n, R, m.dZ, m.dZt);
    // layer 1: grad W1 = dZ1^T X0
    hipLaunchKernelGGL(k_transpose, dim3(blocks_for(R * kMlpIn)), dim3(256), 0, st, m.X0, R, kMlpIn, m.X0t);
    gemm_nt_splitk(m.dZt, (int)R, m.X0t, (int)R, H, kMlpIn, (int)R, m.Gpart, m.G + kOffW1, st);
    hipLaunchKernelGGL(k_bias_grad, dim3(H), dim3(256), 0, st, m.dZt, R, m.G + kOffB1);
    if (grad_out) hipMemcpyAsync(grad_out, m.G, sizeof(float) * kMlpParams, hipMemcpyDeviceToDevice, st);
    if (adam)
        hipLaunchKernelGGL(k_adam, dim3(blocks_for(kMlpParams)), dim3(256), 0, st, P, adam, m.G, adam_step(lr, step));
}

void mlp_train_step(float *P, float *adam, int64_t step, float lr, const float *feat, const float *norm,
                    const float *y, int64_t n, float *loss, float *grad_out, void *scratch, int64_t rows,
                    hipStream_t st, bool fp32) {
    if (fp32) return train_step_fp32(P, adam, step, lr, feat, norm, y, n, loss, grad_out, scratch, rows, st);
    const int64_t R = (n + kTrainRows - 1) / kTrainRows * kTrainRows;
    const int S = split_count(R);
    const int64_t kchunk = ((R + S - 1) / S + kTrainRows - 1) / kTrainRows * kTrainRows;
    const int used = (int)((R + kchunk - 1) / kchunk);
    const TrainBufs m = carve_train(scratch, R, used);
    hipLaunchKernelGGL((k_weights_cast<__bf16, true>), dim3(kCastBlocks), dim3(256), 0, st, P, m.W1, m.W2, m.W3, m.W2t,
                       m.W3t);
    hipLaunchKernelGGL(k_mlp_train, dim3((unsigned)(R / kTrainRows)), dim3(kFuseThreads), 0, st, feat, norm, y, n, P,
                       m);
    hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)used, kGradTiles + 1), dim3(256), 0, st, m, R, kchunk);
    hipLaunchKernelGGL(k_mlp_finish, dim3(blocks_for(kMlpParams + 1)), dim3(256), 0, st, m.grad, used, P, adam,
                       adam_step(lr, adam ? step : 1), grad_out, loss);
}

}  // namespace gs

namespace gs {

// ---------------------------------------------------------------------------
// Proposal mixture and training targets.
//
// p_i = (1 - f) e_i / sum_j e_j + f / n with e_i = exp(y_i - max_j y_j): the
// network's predicted ln s normalised into a distribution and mixed with a
// uniform floor f, so every Gaussian keeps p_i >= f / n (sensitivity sampling
// stays unbiased for any such proposal, proof of Theorem 2).  The maximum is
// an order-free integer atomic on ordered float bits and the sum is a
// fixed-order FP64 reduction, so the result is deterministic.

__device__ __forceinline__ uint32_t ordered_bits(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ordered(uint32_t o) {
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}

// Device-wide atomics on one address serialise (about 10 ns each): with one
// per wave of 3907 blocks the maximum over 10^6 values took 179 us, almost all
// of it waiting on them.  A fixed grid strides over the values, each block
// folds its waves in LDS and adds one atomic (prediction and mixture of 10^6
// rows: 849 -> 675 us).
constexpr int kMaxBlocks = 256;
__global__ __launch_bounds__(256) void k_max_ordered(const float *__restrict__ y, int64_t n,
                                                     uint32_t *__restrict__ out) {
    __shared__ uint32_t sh[4];
    uint32_t m = 0u;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        m = max(m, ordered_bits(y[i]));
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(out, max(max(sh[0], sh[1]), max(sh[2], sh[3])));
}

__global__ __launch_bounds__(256) void k_exp_shift(const float *__restrict__ y, int64_t n,
                                                   const uint32_t *__restrict__ ymax, float *__restrict__ e) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) e[i] = (float)exp((double)y[i] - (double)from_ordered(*ymax));
}

__global__ __launch_bounds__(256) void k_mix(float *__restrict__ p, int64_t n, const double *__restrict__ esum,
                                             float floor) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = (float)((1.0 - (double)floor) * (double)p[i] / *esum + (double)floor / (double)n);
}

// ln(max(s, floor)): regression targets from exact sensitivities.
__global__ __launch_bounds__(256) void k_log_floor(const float *__restrict__ s, int64_t n, float floor,
                                                   float *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = (float)log((double)fmaxf(s[i], floor));
}

size_t mixture_scratch_bytes(int64_t n) { return sizeof(double) * ((size_t)(n + 4095) / 4096 + 2) + 256; }

void proposal_mixture(const float *y, int64_t n, float floor, float *p, void *scratch, hipStream_t st) {
    uint32_t *ymax = (uint32_t *)scratch;
    double *esum = (double *)((char *)scratch + 64);
    double *tmp = esum + 1;
    launch_fill_u32(ymax, 0u, 1, st);
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, kMaxBlocks);
    hipLaunchKernelGGL(k_max_ordered, dim3(blocks), dim3(256), 0, st, y, n, ymax);
    const unsigned g = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_exp_shift, dim3(g), dim3(256), 0, st, y, n, ymax, p);
    launch_sum_f32_to_f64(p, n, esum, tmp, st);
    hipLaunchKernelGGL(k_mix, dim3(g), dim3(256), 0, st, p, n, esum, floor);
}

void log_targets(const float *s, int64_t n, float floor, float *out, hipStream_t st) {
    hipLaunchKernelGGL(k_log_floor, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, s, n, floor, out);
}

}  // namespace gs
