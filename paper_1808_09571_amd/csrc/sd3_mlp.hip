// Training kernels of the tile-pair ranker MLP (10 -> 64 -> 64 -> 64 -> 1, ReLU,
// FP32): forward pass, mean-squared-error loss, backward pass (data and weight
// gradients) and the Adam update.
//
// One launch takes every layer of both passes (k_mlp): a block keeps the
// weights in LDS and walks batches of 16 samples, whose activations never
// leave it, and each layer is a chain of FP32 v_mfma_f32_16x16x4_f32 (FP32
// products and sums, as the dot products before).  The weight gradients stay
// in the accumulators over all of a block's samples and leave as one partial
// per block; k_mlp_reduce adds the partials in block order, so a result does
// not depend on scheduling.  A minibatch is latency-bound (4096 samples are
// 0.22 GFLOP, 2 us of the FP32 matrix rate): the chain of eight small
// contractions and the block's load of 36 KB of weights.  Loss, gradient and
// Adam step of 4096 samples: 383 us as 15 launches with one dot product per
// thread (266 us of them in the weight gradients' serial sums), 21 us now: 13.5 us
// here, 4.2 in the reduction, 2.2 in Adam.
#include <algorithm>

#include "sd3_mlp.h"

namespace sd3 {

using mfx4 = float __attribute__((ext_vector_type(4)));

constexpr int MT = 16;    // samples per batch
// row strides in LDS: a wave's operand reads (16 rows x 4 columns, or 4 rows x
// 16 columns) start 4 banks apart per row
constexpr int WS = 68;    // 64-wide rows
constexpr int XS = 20;    // inputs, padded with zeros
static_assert(MLP_H * XS == 5 * 256 && MLP_H * MLP_H == 16 * 256, "weights staged by 256 threads");

struct MlpLds {
    float w1[MLP_H * XS], w2[MLP_H * WS], w3[MLP_H * WS];  // [out][in]
    float b[3][MLP_H], w4[MLP_H], b4;
    float x[MT * XS];
    float h[3][MT * WS];  // activations of the hidden layers
    float d[3][MT * WS];  // gradients with respect to their pre-activations
    float dy[MT], e[MT];
};

// acc += A B over `steps` groups of four: lane l takes A[l % 16][4 s + l / 16]
// = a[(l % 16) ar + (4 s + l / 16) ak] and B[4 s + l / 16][l % 16] likewise;
// it ends with D[4 (l / 16) + r][l % 16] in acc[r].
template <int STEPS>
__device__ __forceinline__ mfx4 mm16(const float *a, int ar, int ak, const float *b, int bk, int bc, mfx4 acc) {
    const int lane = lane_id(), m = lane & 15, q = lane >> 4;
#pragma unroll
    for (int s = 0; s < STEPS; s++) {
        const int k = 4 * s + q;
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m * ar + k * ak], b[k * bk + m * bc], acc, 0, 0, 0);
    }
    return acc;
}

// GRAD: partials of the gradient (MLP_NPARAM floats) and of the loss (one
// more) per block; else the outputs y.
template <bool GRAD>
__global__ __launch_bounds__(256) void k_mlp(const float *P, const float *X, const float *T, int64_t n, float *y,
                                             float *part) {
    __shared__ MlpLds L;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const int m = lane & 15, q = lane >> 4;
    // (every load of the weights first: one memory latency)
    {
        float v2[16], v3[16], v1[5];
#pragma unroll
        for (int j = 0; j < 16; j++) {
            v2[j] = P[MLP_W2 + 256 * j + tid];
            v3[j] = P[MLP_W3 + 256 * j + tid];
        }
#pragma unroll
        for (int j = 0; j < 5; j++) {
            const int i = 256 * j + tid, o = i / XS, k = i % XS;
            v1[j] = k < MLP_IN ? P[MLP_W1 + o * MLP_IN + k] : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < 16; j++) {
            const int at = (4 * j + w) * WS + lane;
            L.w2[at] = v2[j];
            L.w3[at] = v3[j];
        }
#pragma unroll
        for (int j = 0; j < 5; j++) L.w1[256 * j + tid] = v1[j];
    }
    if (tid < MLP_H) {
        L.b[0][tid] = P[MLP_B1 + tid];
        L.b[1][tid] = P[MLP_B2 + tid];
        L.b[2][tid] = P[MLP_B3 + tid];
        L.w4[tid] = P[MLP_W4 + tid];
    }
    if (tid == 0) L.b4 = P[MLP_B4];
    // wave w's share of the gradients: rows 16 w .. 16 w + 15 (outputs) of
    // every weight matrix, and one vector (w: b3, b2, b1, w4)
    mfx4 g1 = {0.0f, 0.0f, 0.0f, 0.0f}, g2[4], g3[4];
    for (int j = 0; j < 4; j++) g2[j] = g3[j] = g1;
    float gv = 0.0f, gb4 = 0.0f, loss = 0.0f;
    const int64_t nb = (n + MT - 1) / MT;
    for (int64_t t = blockIdx.x; t < nb; t += gridDim.x) {
        const int64_t i0 = t * MT;
        const int have = (int)min((int64_t)MT, n - i0);
        __syncthreads();  // the previous batch is done with x, h and d
        for (int i = tid; i < MT * XS; i += 256) {
            const int r = i / XS, k = i % XS;
            L.x[i] = r < have && k < MLP_IN ? X[(i0 + r) * MLP_IN + k] : 0.0f;
        }
        __syncthreads();
        // hidden layers: wave w forms outputs 16 w .. 16 w + 15 (rows past
        // the batch are kept at 0)
        auto layer = [&](int l, mfx4 acc) __attribute__((always_inline)) {
            const int o = 16 * w + m;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int i = 4 * q + r;
                L.h[l][i * WS + o] = i < have ? fmaxf(acc[r] + L.b[l][o], 0.0f) : 0.0f;
            }
            __syncthreads();
        };
        const mfx4 z = {0.0f, 0.0f, 0.0f, 0.0f};
        layer(0, mm16<3>(L.x, XS, 1, L.w1 + 16 * w * XS, 1, XS, z));
        layer(1, mm16<16>(L.h[0], WS, 1, L.w2 + 16 * w * WS, 1, WS, z));
        layer(2, mm16<16>(L.h[1], WS, 1, L.w3 + 16 * w * WS, 1, WS, z));
        // output: 16 lanes per sample, each four units
        {
            const int i = 4 * w + q;
            const float *h = L.h[2] + i * WS;
            float s = 0.0f;
#pragma unroll
            for (int r = 0; r < 4; r++) s += h[m + 16 * r] * L.w4[m + 16 * r];
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o);
            s += L.b4;
            if (!GRAD) {
                if (m == 0 && i < have) y[i0 + i] = s;
                continue;
            }
            const float err = i < have ? s - T[i0 + i] : 0.0f;
            const float dy = 2.0f * err / (float)n;
            if (m == 0) {
                L.dy[i] = dy;
                L.e[i] = err * err / (float)n;
            }
#pragma unroll
            for (int r = 0; r < 4; r++)
                L.d[2][i * WS + m + 16 * r] = h[m + 16 * r] > 0.0f ? dy * L.w4[m + 16 * r] : 0.0f;
        }
        __syncthreads();
        // backward through layers 3 and 2: wave w forms the inputs' gradients
        // 16 w .. 16 w + 15 and adds its rows of the weight gradients
        auto back = [&](int l, const float *W, mfx4(&g)[4]) __attribute__((always_inline)) {
            const mfx4 acc = mm16<16>(L.d[l], WS, 1, W + 16 * w, WS, 1, z);
            const int k = 16 * w + m;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int at = (4 * q + r) * WS + k;
                L.d[l - 1][at] = L.h[l - 1][at] > 0.0f ? acc[r] : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < 4; j++)
                g[j] = mm16<4>(L.d[l] + 16 * w, 1, WS, L.h[l - 1] + 16 * j, WS, 1, g[j]);
            __syncthreads();
        };
        back(2, L.w3, g3);
        back(1, L.w2, g2);
        g1 = mm16<4>(L.d[0] + 16 * w, 1, WS, L.x, XS, 1, g1);
        // vectors: b3, b2, b1 from the gradients, w4 from dy h3
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < MT; i++)
            s += w < 3 ? L.d[2 - w][i * WS + lane] : L.dy[i] * L.h[2][i * WS + lane];
        gv += s;
        if (tid == 0) {
            float sb = 0.0f, sl = 0.0f;
            for (int i = 0; i < MT; i++) {
                sb += L.dy[i];
                sl += L.e[i];
            }
            gb4 += sb;
            loss += sl;
        }
    }
    if (!GRAD) return;
    float *o = part + (int64_t)blockIdx.x * (MLP_NPARAM + 1);
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const int row = 16 * w + 4 * q + r;
        if (m < MLP_IN) o[MLP_W1 + row * MLP_IN + m] = g1[r];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            o[MLP_W2 + row * MLP_H + 16 * j + m] = g2[j][r];
            o[MLP_W3 + row * MLP_H + 16 * j + m] = g3[j][r];
        }
    }
    o[(w == 0 ? MLP_B3 : w == 1 ? MLP_B2 : w == 2 ? MLP_B1 : MLP_W4) + lane] = gv;
    if (tid == 0) {
        o[MLP_B4] = gb4;
        o[MLP_NPARAM] = loss;
    }
}

// The gradient and the loss: the sums of nb blocks' partials, 64 parameters a
// block, 16 threads each taking every sixteenth partial.
__global__ __launch_bounds__(1024) void k_mlp_reduce(const float *part, int nb, float *G, float *loss) {
    __shared__ float red[16][64];
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + l;
    float s = 0.0f;
    if (p <= MLP_NPARAM) {
#pragma unroll 8
        for (int b = w; b < nb; b += 16) s += part[(int64_t)b * (MLP_NPARAM + 1) + p];
    }
    red[w][l] = s;
    __syncthreads();
    if (w == 0 && p <= MLP_NPARAM) {
        for (int k = 1; k < 16; k++) s += red[k][l];
        if (p < MLP_NPARAM) G[p] = s;
        else *loss = s;
    }
}

// Adam (Kingma & Ba 2015) with bias-corrected moments.
__global__ void k_adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    float gi = g[i];
    float mi = b1 * m[i] + (1.0f - b1) * gi;
    float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

static unsigned g256(int64_t n) { return (unsigned)((n + 255) / 256 > 0 ? (n + 255) / 256 : 1); }

// One batch of 16 samples a block up to 512 blocks (two a CU by their LDS),
// which then walk on: more blocks would only add partials to sum.
int mlp_blocks(int64_t n) { return (int)std::min<int64_t>((n + MT - 1) / MT, 512); }

void mlp_forward(const float *P, const float *X, int64_t n, float *y, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_mlp<false>, dim3(mlp_blocks(n)), dim3(256), 0, st, P, X, nullptr, n, y, nullptr);
}

void mlp_loss_grad(const float *P, const float *X, const float *T, int64_t n, float *part, float *loss, float *G,
                   hipStream_t st) {
    const int nb = mlp_blocks(n);
    if (nb > 0)
        hipLaunchKernelGGL(k_mlp<true>, dim3(nb), dim3(256), 0, st, P, X, T, n, nullptr, part);
    hipLaunchKernelGGL(k_mlp_reduce, dim3(MLP_NPARAM / 64 + 1), dim3(1024), 0, st, part, nb, G, loss);
}

void adam_step(float *p, const float *g, float *m, float *v, int64_t n, int step, float lr,
               float b1, float b2, float eps, hipStream_t st) {
    if (n <= 0) return;
    float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(g256(n)), dim3(256), 0, st, p, g, m, v, n, lr, b1, b2, eps, c1,
                       c2);
}

}  // namespace sd3
