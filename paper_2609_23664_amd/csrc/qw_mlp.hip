// Learned planner cost model: a 3-layer perceptron (12 -> 64 -> 64 -> 2,
// ReLU) trained on the GPU with these kernels.
//
// Layout: FP32 master parameters in one array (qw.h, QW_MLP_*):
//   W1[12][64], b1[64], W2[64][64], b2[64], W3[64][2], b3[2]  (row-major,
//   W[k][j] multiplies input k into output j).
// Every GEMM rounds its two inputs to BF16 (round to nearest even) and
// accumulates in FP32 on the matrix cores (v_mfma_f32_16x16x16_bf16);
// biases, ReLU, the loss gradient and Adam are FP32.
//
// MFMA 16x16x16 BF16 operand layout (wave of 64 lanes, lane l, item i<4):
//   A[m][k]: m = l % 16, k = 4 (l / 16) + i
//   B[k][n]: n = l % 16, k = 4 (l / 16) + i
//   D[m][n]: n = l % 16, m = 4 (l / 16) + i
// Reductions over the batch (weight gradients) run in a fixed order, so
// results are deterministic.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "qw_kernels.h"

namespace qw {
namespace {

constexpr int IN = 12, W = 64, OUT = 2;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + IN * W, OFF_W2 = OFF_B1 + W, OFF_B2 = OFF_W2 + W * W,
              OFF_W3 = OFF_B2 + W, OFF_B3 = OFF_W3 + W * OUT, N_PARAMS = OFF_B3 + OUT;
static_assert(N_PARAMS == 5122, "parameter count");

// Workspace per batch row (floats): Z1[64], Z2[64], Y[2], dY[2], dZ2[64], dZ1[64]
constexpr int WS_Z1 = 0, WS_Z2 = 64, WS_Y = 128, WS_DY = 130, WS_DZ2 = 132, WS_DZ1 = 196,
              WS_ROW = 260;

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 -> BF16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ short bf16_rne(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}

// Batch row b reads row src_row(rows, b) of the inputs and targets: rows[b]
// when a row list is given (a gathered mini-batch), else b.
__device__ __forceinline__ size_t src_row(const uint32_t *__restrict__ rows, int b) {
    return rows ? (size_t)rows[b] : (size_t)b;
}

__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Four FP32 values as one MFMA operand.
__device__ __forceinline__ bf16x4 operand(const float (&v)[4]) {
    bf16x4 o;
    #pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = bf16_rne(v[i]);
    return o;
}

// A layer's activations of 16 rows in BF16 between two products; rows padded
// to 68 entries so that the 16 rows' operand reads spread over the banks.
struct alignas(8) Act {
    short v[16][W + 4];
    // operand A (m = lane % 16, k = k0 + 4 (lane / 16) + i)
    __device__ __forceinline__ bf16x4 read(int r, int k) const {
        return *reinterpret_cast<const bf16x4 *>(&v[r][k]);
    }
};

// Forward pass, and with BWD the backward pass through the rows for L =
// (1 / 2B) sum (y - t)^2: dY = (Y - T) / B, dZ2 = (dY W3^T) * [Z2 > 0],
// dZ1 = (dZ2 W2^T) * [Z1 > 0]. A workgroup takes 16 rows; wave t of its four
// computes columns 16 t .. 16 t + 15 of every layer, activations pass through
// LDS, and pre-activations stay in registers for the ReLU masks (the outputs
// of all layers share one layout). Bound by latency, not by its 3 to 7
// products: so all weight operands are requested before the first product.
// One wave per 16 rows with each layer through the workspace in memory took
// 27 us for the forward pass of 256 rows and 11 us more for the rows'
// backward pass; this form takes 7.0 us for both.
template <bool BWD>
__global__ __launch_bounds__(256) void mlp_rows_kernel(const float *__restrict__ p,
                                                       const float *__restrict__ x,
                                                       const uint32_t *__restrict__ rows,
                                                       const float *__restrict__ tgt, uint32_t B,
                                                       float *__restrict__ ws, float *__restrict__ y) {
    __shared__ Act h1, h2;
    __shared__ float dy[16][OUT];
    const int lane = threadIdx.x & 63, t = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4, col = 16 * t + r;
    const int row0 = blockIdx.x * 16;
    const bool a_ok = row0 + r < (int)B;
    const size_t a_row = a_ok ? src_row(rows, row0 + r) : 0;
    // operands: inputs, then every layer's weights
    float xa[4], w1[4], w2[4][4], w3[4][4];
    #pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 4 * g + i;
        xa[i] = a_ok && k < IN ? x[a_row * IN + k] : 0.f;
        w1[i] = k < IN ? p[OFF_W1 + k * W + col] : 0.f;
        #pragma unroll
        for (int s = 0; s < 4; ++s) {
            w2[s][i] = p[OFF_W2 + (16 * s + k) * W + col];
            w3[s][i] = r < OUT ? p[OFF_W3 + (16 * s + k) * OUT + r] : 0.f;
        }
    }
    const float b1 = p[OFF_B1 + col], b2 = p[OFF_B2 + col], b3 = r < OUT ? p[OFF_B3 + r] : 0.f;
    float w3t[4], w2t[4][4], tg[4];
    if constexpr (BWD) {
        #pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 4 * g + i;
            w3t[i] = k < OUT ? p[OFF_W3 + col * OUT + k] : 0.f;
            #pragma unroll
            for (int s = 0; s < 4; ++s) w2t[s][i] = p[OFF_W2 + col * W + 16 * s + k];
            const int m = 4 * g + i;
            tg[i] = t == 0 && r < OUT && row0 + m < (int)B ? tgt[src_row(rows, row0 + m) * OUT + r] : 0.f;
        }
    }
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    // layer 1: Z1 = X W1 + b1
    f32x4 z1 = mfma(operand(xa), operand(w1), zero);
    #pragma unroll
    for (int i = 0; i < 4; ++i) {
        z1[i] += b1;
        h1.v[4 * g + i][col] = bf16_rne(fmaxf(z1[i], 0.f));
    }
    __syncthreads();
    // layer 2: Z2 = relu(Z1) W2 + b2
    f32x4 z2 = zero;
    #pragma unroll
    for (int s = 0; s < 4; ++s) z2 = mfma(h1.read(r, 16 * s + 4 * g), operand(w2[s]), z2);
    #pragma unroll
    for (int i = 0; i < 4; ++i) {
        z2[i] += b2;
        h2.v[4 * g + i][col] = bf16_rne(fmaxf(z2[i], 0.f));
    }
    __syncthreads();
    // layer 3: Y = relu(Z2) W3 + b3 (one tile: wave 0)
    if (t == 0) {
        f32x4 yv = zero;
        #pragma unroll
        for (int s = 0; s < 4; ++s) yv = mfma(h2.read(r, 16 * s + 4 * g), operand(w3[s]), yv);
        #pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = 4 * g + i;
            const bool ok = row0 + m < (int)B;
            const float v = yv[i] + b3;
            if (ok && r < OUT) {
                float *wr = ws + (size_t)(row0 + m) * WS_ROW;
                wr[WS_Y + r] = v;
                if (y) y[(size_t)(row0 + m) * OUT + r] = v;
                if constexpr (BWD) wr[WS_DY + r] = (v - tg[i]) * (1.0f / (float)B);
            }
            if constexpr (BWD)
                if (r < OUT) dy[m][r] = ok ? (v - tg[i]) * (1.0f / (float)B) : 0.f;
        }
    }
    if constexpr (BWD) {
        __syncthreads();
        float da[4];
        #pragma unroll
        for (int i = 0; i < 4; ++i) da[i] = 4 * g + i < OUT ? dy[r][4 * g + i] : 0.f;
        const f32x4 q2 = mfma(operand(da), operand(w3t), zero);
        float d2[4];
        #pragma unroll
        for (int i = 0; i < 4; ++i) {
            d2[i] = z2[i] > 0.f ? q2[i] : 0.f;
            h1.v[4 * g + i][col] = bf16_rne(d2[i]);
        }
        __syncthreads();
        f32x4 q1 = zero;
        #pragma unroll
        for (int s = 0; s < 4; ++s) q1 = mfma(h1.read(r, 16 * s + 4 * g), operand(w2t[s]), q1);
        #pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (row0 + 4 * g + i >= (int)B) continue;
            float *wr = ws + (size_t)(row0 + 4 * g + i) * WS_ROW;
            wr[WS_Z1 + col] = z1[i];
            wr[WS_Z2 + col] = z2[i];
            wr[WS_DZ2 + col] = d2[i];
            wr[WS_DZ1 + col] = z1[i] > 0.f ? q1[i] : 0.f;
        }
    }
}

// Weight gradients: one workgroup per 16x16 tile of dW1, dW2 or dW3 (tiles:
// dW1 1x4, 12 rows padded to 16; dW2 4x4; dW3 4x1, 2 columns padded). Its
// waves take the batch's groups of 16 rows in turn (wave w groups w, w +
// waves, ...), each with its own FP32 accumulator, and the waves' tiles are
// added in wave order; the first tile of a column block also sums its
// operand's columns in FP32 for the bias gradient. The order depends on the
// batch size alone. Bound by the latency of the workspace reads: one wave a
// tile with a serial column sum took 48 us at 256 rows, this 5.2 us.
constexpr int kWeightWaves = 16;

__global__ __launch_bounds__(64 * kWeightWaves) void mlp_weights_kernel(
    const float *__restrict__ x, const uint32_t *__restrict__ rows, uint32_t B,
    const float *__restrict__ ws, float *__restrict__ grad) {
    __shared__ float red[kWeightWaves][256];
    __shared__ float redb[kWeightWaves][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int Bi = (int)B, groups = (Bi + 15) / 16;
    // tile (layer, tm, tn): A column block tm, B column block tn
    const int layer = blockIdx.x < 4 ? 1 : (blockIdx.x < 20 ? 2 : 3);
    const int tm = layer == 1 ? 0 : (layer == 2 ? ((int)blockIdx.x - 4) / 4 : (int)blockIdx.x - 20);
    const int tn = layer == 1 ? (int)blockIdx.x : (layer == 2 ? ((int)blockIdx.x - 4) % 4 : 0);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float col = 0.f;
    #pragma unroll 2
    for (int s = wave; s < groups; s += waves) {
        float av[4], bv[4];
        #pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 16 * s + 4 * g + i;
            const float *wr = ws + (size_t)k * WS_ROW;
            av[i] = bv[i] = 0.f;
            if (k < Bi) {
                if (layer == 1) {   // dW1 = X^T dZ1
                    if (r < IN) av[i] = x[src_row(rows, k) * IN + r];
                    bv[i] = wr[WS_DZ1 + 16 * tn + r];
                } else if (layer == 2) {   // dW2 = relu(Z1)^T dZ2
                    av[i] = fmaxf(wr[WS_Z1 + 16 * tm + r], 0.f);
                    bv[i] = wr[WS_DZ2 + 16 * tn + r];
                } else {   // dW3 = relu(Z2)^T dY
                    av[i] = fmaxf(wr[WS_Z2 + 16 * tm + r], 0.f);
                    if (r < OUT) bv[i] = wr[WS_DY + r];
                }
            }
        }
        acc = mfma(operand(av), operand(bv), acc);
        col += (bv[0] + bv[1]) + (bv[2] + bv[3]);
    }
    *reinterpret_cast<f32x4 *>(&red[wave][4 * lane]) = acc;
    col += __shfl_xor(col, 16, 64);
    col += __shfl_xor(col, 32, 64);
    if (lane < 16) redb[wave][lane] = col;
    __syncthreads();
    for (int e = threadIdx.x; e < 256; e += blockDim.x) {
        float v = red[0][e];
        for (int w = 1; w < waves; ++w) v += red[w][e];
        // element i of lane l: row m = 4 (l / 16) + i, column l % 16
        const int l = e >> 2, m = 4 * (l >> 4) + (e & 3), n = l & 15;
        if (layer == 1) {
            if (m < IN) grad[OFF_W1 + m * W + 16 * tn + n] = v;
        } else if (layer == 2) {
            grad[OFF_W2 + (16 * tm + m) * W + 16 * tn + n] = v;
        } else if (n < OUT) {
            grad[OFF_W3 + (16 * tm + m) * OUT + n] = v;
        }
    }
    if (tm == 0 && (int)threadIdx.x < (layer == 3 ? OUT : 16)) {
        float v = redb[0][threadIdx.x];
        for (int w = 1; w < waves; ++w) v += redb[w][threadIdx.x];
        const int off = layer == 1 ? OFF_B1 : (layer == 2 ? OFF_B2 : OFF_B3);
        grad[off + 16 * tn + threadIdx.x] = v;
    }
}

// Adam (FP32): m = b1 m + (1 - b1) g; v = b2 v + (1 - b2) g^2;
// p -= lr * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps).
__global__ __launch_bounds__(256) void mlp_adam_kernel(float *__restrict__ p,
                                                       const float *__restrict__ g,
                                                       float *__restrict__ m, float *__restrict__ v,
                                                       uint32_t n, float lr, float b1, float b2,
                                                       float eps, float c1, float c2) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = fmaf(b1, m[i], (1.0f - b1) * gi);
    const float vi = fmaf(b2, v[i], (1.0f - b2) * gi * gi);
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Loss 1/(2B) sum_b sum_j (Y[b][j] - T[b][j])^2 from the forward pass's Y in
// the workspace, in FP64, by one wave: lane l sums rows l, l + 64, ... in
// order, then the 64 lane sums are added pairwise in a fixed tree.
__global__ __launch_bounds__(64) void mlp_loss_kernel(const float *__restrict__ tgt,
                                                      const uint32_t *__restrict__ rows,
                                                      uint32_t B, const float *__restrict__ ws,
                                                      double *__restrict__ out) {
    __shared__ double part[64];
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    for (int b = lane; b < (int)B; b += 64) {
        for (int j = 0; j < OUT; ++j) {
            const double d = (double)ws[(size_t)b * WS_ROW + WS_Y + j] - (double)tgt[src_row(rows, b) * OUT + j];
            s = fma(d, d, s);
        }
    }
    part[lane] = s;
    __syncthreads();
    for (int h = 32; h > 0; h >>= 1) {
        if (lane < h) part[lane] += part[lane + h];
        __syncthreads();
    }
    if (lane == 0) out[0] = part[0] / (2.0 * (double)B);
}

}  // namespace

size_t mlp_workspace_floats(uint32_t batch) { return (size_t)batch * WS_ROW; }

hipError_t launch_mlp_forward(hipStream_t st, const float *p, const float *x, const uint32_t *rows,
                              uint32_t B, float *ws, float *y) {
    if (B == 0) return hipSuccess;
    hipLaunchKernelGGL(mlp_rows_kernel<false>, dim3((B + 15) / 16), dim3(256), 0, st, p, x, rows,
                       (const float *)nullptr, B, ws, y);
    return hipGetLastError();
}

hipError_t launch_mlp_backward(hipStream_t st, const float *p, const float *x, const float *t,
                               const uint32_t *rows, uint32_t B, float *ws, float *grad) {
    if (B == 0) return hipSuccess;
    hipLaunchKernelGGL(mlp_rows_kernel<true>, dim3((B + 15) / 16), dim3(256), 0, st, p, x, rows, t, B, ws,
                       (float *)nullptr);
    // one wave per 16 rows of the batch up to kWeightWaves
    const uint32_t waves = (B + 15) / 16 < (uint32_t)kWeightWaves ? (B + 15) / 16 : (uint32_t)kWeightWaves;
    hipLaunchKernelGGL(mlp_weights_kernel, dim3(24), dim3(64 * waves), 0, st, x, rows, B,
                       (const float *)ws, grad);
    return hipGetLastError();
}

hipError_t launch_mlp_loss(hipStream_t st, const float *p, const float *x, const float *t,
                           const uint32_t *rows, uint32_t B, float *ws, double *out) {
    if (B == 0) return hipSuccess;
    hipLaunchKernelGGL(mlp_rows_kernel<false>, dim3((B + 15) / 16), dim3(256), 0, st, p, x, rows,
                       (const float *)nullptr, B, ws, (float *)nullptr);
    hipLaunchKernelGGL(mlp_loss_kernel, dim3(1), dim3(64), 0, st, t, rows, B, (const float *)ws, out);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(hipStream_t st, float *p, const float *g, float *m, float *v,
                           uint32_t step, float lr, float b1, float b2, float eps) {
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(mlp_adam_kernel, dim3((N_PARAMS + 255) / 256), dim3(256), 0, st, p, g, m, v,
                       (uint32_t)N_PARAMS, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace qw
