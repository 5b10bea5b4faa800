// kf_mlp.hip -- training and inference kernels of the learned cost model: a
// d -> H -> H -> H -> 1 multilayer perceptron with ReLU, mean-squared error on
// log run time and Adam. The layer products are dense contractions and run on
// the matrix cores (v_mfma_f32_16x16x4f32, FP32 in and out); the rest is
// element-wise. All reductions are in fixed order, so training is
// bit-reproducible.
//
// The network is tiny, so a step is bound by launches and by the latency of its
// chain of layers, not by bytes or operations. A step is three launches: the
// layers of a block of 16 samples, forward and backward, in one workgroup with
// the activations in LDS (mlp_rows_kernel); the gradients of every layer's
// weights and biases, one 16 x 16 tile per workgroup (mlp_wgrad_kernel); Adam.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "device/kf_blocks.h"

namespace kf {

typedef float f4v __attribute__((ext_vector_type(4)));

// C(i,j) = sum_k A(i,k) B(k,j) [+ bias(j)] [relu] [* (mask(i,j) > 0)], with
// element strides so that either operand can be read transposed:
// A(i,k) = A[i*sai + k*sak], B(k,j) = B[k*sbk + j*sbj], C(i,j) = C[i*ldc + j].
// Lane layout of the 16x16x4 FP32 MFMA on a 64-lane wave: lane l supplies
// A(l%16, l/16) and B(l/16, l%16) of the 16x4 / 4x16 slices and receives
// C(4*(l/16) + r, l%16) in accumulator register r.
__global__ void __launch_bounds__(64) mlp_gemm_kernel(int M, int N, int K, const float* __restrict__ A,
                                                      long sai, long sak, const float* __restrict__ B, long sbk,
                                                      long sbj, float* __restrict__ C, long ldc,
                                                      const float* __restrict__ bias, int relu,
                                                      const float* __restrict__ mask, long ldm) {
    const int lane = threadIdx.x;
    const int i0 = blockIdx.y * 16, j0 = blockIdx.x * 16;
    const int ia = i0 + (lane & 15), jb = j0 + (lane & 15), kk = lane >> 4;
    f4v acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += 4) {
        const int k = k0 + kk;
        const float a = (ia < M && k < K) ? A[ia * sai + k * sak] : 0.f;
        const float b = (jb < N && k < K) ? B[k * sbk + jb * sbj] : 0.f;
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
    }
    const int j = j0 + (lane & 15);
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + 4 * (lane >> 4) + r;
        if (i < M && j < N) {
            float v = acc[r];
            if (bias) v += bias[j];
            if (relu) v = v > 0.f ? v : 0.f;
            if (mask) v = mask[i * ldm + j] > 0.f ? v : 0.f;
            C[i * ldc + j] = v;
        }
    }
}

// loss = mean((p - y)^2); dp = 2 (p - y) / n (dp may be null). One workgroup of 256 threads.
__device__ __forceinline__ void mlp_mse_block(int n, const float* __restrict__ p, const float* __restrict__ y,
                                              float* __restrict__ dp, float* __restrict__ loss) {
    __shared__ float part[256];
    const int t = threadIdx.x;
    float s = 0.f;
    for (int i = t; i < n; i += 256) {
        const float d = p[i] - y[i];
        s += d * d;
        if (dp) dp[i] = 2.f * d / (float)n;
    }
    part[t] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) part[t] += part[t + w];
        __syncthreads();
    }
    if (t == 0 && loss) *loss = part[0] / (float)n;
}
__global__ void __launch_bounds__(256) mlp_mse_kernel(int n, const float* __restrict__ p, const float* __restrict__ y,
                                                      float* __restrict__ dp, float* __restrict__ loss) {
    mlp_mse_block(n, p, y, dp, loss);
}

// ---- a block of 16 samples through every layer ------------------------------
// Parameters of layer l: (rows + 1) x cols floats, the bias is the last row.
__device__ __forceinline__ long mlp_w_off(int l, int d, int h) {
    return l == 0 ? 0 : (long)(d + 1) * h + (long)(l - 1) * (h + 1) * h;
}

// Workgroup b owns samples 16 b .. 16 b + 15; wave w computes column tiles w,
// w + W, ... of each layer. Forward sums run over k = 0, 1, ... four at a time,
// as in mlp_gemm_kernel. Backward (BWD) the gradient of a layer's input is its
// output gradient times the transposed weights, so a lane reads four
// consecutive k of one weight row (16 bytes) and k runs in the order
// 16 s + t, + 4, + 8, + 12. H and dZ receive each hidden layer's activations and
// pre-activation gradients (n x h each) for the weight gradients. LDS rows are
// zero past d and h up to the next multiple of 32.
typedef f4v f4v_any __attribute__((aligned(4)));

struct mlp_net {
    int n, d, h, L, hs;   // hs: row pitch of the LDS tiles
    const float* P;
    const float* X;
    const float* y;
    float* H;
    float* dZ;
    float* pred;
    float* dpred;
};

// The block's inputs into `cur`, zero past n and d.
template <int NT>
__device__ __forceinline__ void mlp_load_x(const mlp_net& m, long r0, float* cur) {
    const int dpad = (m.d + 31) / 32 * 32;
    for (int i = threadIdx.x; i < 16 * dpad; i += NT) {
        const int r = i / dpad, c = i - r * dpad;
        cur[r * m.hs + c] = (r0 + r < m.n && c < m.d) ? m.X[(r0 + r) * m.d + c] : 0.f;
    }
}
// Output layer (one column) from the activations in `cur`, by wave 0; the
// output gradients 2 (p - y) / n of the block go to dp.
template <bool BWD>
__device__ __forceinline__ void mlp_output(const mlp_net& m, const float* __restrict__ WL, long r0, const float* cur, float* dp) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const float bias = WL[m.h];
    f4v acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < m.h; k0 += 128) {
        float a[32], b[32];
#pragma unroll
        for (int s = 0; s < 32; ++s) {
            const int k = k0 + 4 * s + lk;
            const float v = WL[min(k, m.h - 1)];
            b[s] = (lr == 0 && k < m.h) ? v : 0.f;
            a[s] = cur[lr * m.hs + min(k, m.hs - 1)];
        }
#pragma unroll
        for (int s = 0; s < 32; ++s)
            if (k0 + 4 * s < m.h) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], acc, 0, 0, 0);
    }
    if (lr == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * lk + r;
            const bool in = r0 + i < m.n;
            const float p = acc[r] + bias;
            if (in) m.pred[r0 + i] = p;
            if constexpr (BWD) {
                const float g = in ? 2.f * (p - m.y[r0 + i]) / (float)m.n : 0.f;
                dp[i] = g;
                if (in) m.dpred[r0 + i] = g;
            }
        }
    }
}
// Gradient of the last hidden layer's pre-activations: dp w^T where the
// activation is positive.
template <int NT>
__device__ __forceinline__ void mlp_last_grad(const mlp_net& m, const float* __restrict__ WL, long r0, const float* cur,
                                              const float* dp, float* nxt) {
    const int cols = (m.h + 31) / 32 * 32;
    float* dZl = m.dZ + (long)(m.L - 1) * m.n * m.h;
    for (int e = threadIdx.x; e < 16 * cols; e += NT) {
        const int i = e / cols, j = e - i * cols;
        const float w = WL[min(j, m.h - 1)];
        const float v = (j < m.h && cur[i * m.hs + j] > 0.f) ? dp[i] * w : 0.f;
        nxt[i * m.hs + j] = v;
        if (j < m.h && r0 + i < m.n) dZl[(r0 + i) * m.h + j] = v;
    }
}

// Any widths that fit the LDS tiles.
constexpr int MLP_NT = 512, MLP_NW = MLP_NT / 64;
template <bool BWD>
__global__ void __launch_bounds__(MLP_NT) mlp_rows_kernel(mlp_net m) {
    extern __shared__ float mlp_lds[];   // two 16 x hs tiles, then 16 output gradients
    const int n = m.n, h = m.h, L = m.L, hs = m.hs;
    float* cur = mlp_lds;
    float* nxt = mlp_lds + 16 * hs;
    float* dp = mlp_lds + 32 * hs;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
    const long r0 = (long)blockIdx.x * 16;
    const int ht = (h + 31) / 32 * 2;   // tiles of 16 columns
    mlp_load_x<MLP_NT>(m, r0, cur);
    __syncthreads();
    for (int l = 0; l < L; ++l) {
        const int K = l == 0 ? m.d : h;
        const float* __restrict__ W = m.P + mlp_w_off(l, m.d, h);
        for (int t = wave; t < ht; t += MLP_NW) {
            const int j = t * 16 + lr, jc = min(j, h - 1);
            const float bias = W[(long)K * h + jc];
            f4v acc = {0.f, 0.f, 0.f, 0.f};
            for (int k0 = 0; k0 < K; k0 += 64) {   // 16 weight loads in flight per lane
                float b[16];
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    const int k = k0 + 4 * s + lk;
                    const float v = W[(unsigned)(min(k, K - 1) * h + jc)];
                    b[s] = (j < h && k < K) ? v : 0.f;
                }
#pragma unroll
                for (int s = 0; s < 16; ++s)
                    if (k0 + 4 * s < K) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[lr * hs + k0 + 4 * s + lk], b[s], acc, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * lk + r;
                float v = acc[r] + bias;
                v = (j < h && v > 0.f) ? v : 0.f;
                nxt[i * hs + j] = v;
                if (BWD && j < h && r0 + i < n) m.H[((long)l * n + r0 + i) * h + j] = v;
            }
        }
        __syncthreads();
        float* s = cur; cur = nxt; nxt = s;
    }
    const float* __restrict__ WL = m.P + mlp_w_off(L, m.d, h);
    if (wave == 0) mlp_output<BWD>(m, WL, r0, cur, dp);
    if constexpr (BWD) {
        __syncthreads();
        mlp_last_grad<MLP_NT>(m, WL, r0, cur, dp, nxt);
        __syncthreads();
        float* g = nxt;
        float* o = cur;
        for (int l = L - 1; l > 0; --l) {
            const float* __restrict__ W = m.P + mlp_w_off(l, m.d, h);
            for (int t = wave; t < ht; t += MLP_NW) {
                const int j = t * 16 + lr, jc = min(j, h - 1);
                float act[4];   // this lane's own activations of the layer below
#pragma unroll
                for (int r = 0; r < 4; ++r) act[r] = m.H[((long)(l - 1) * n + min(r0 + 4 * lk + r, (long)n - 1)) * h + jc];
                f4v acc = {0.f, 0.f, 0.f, 0.f};
                for (int k0 = 0; k0 < h; k0 += 64) {
                    float b[16];
#pragma unroll
                    for (int s = 0; s < 16; ++s) {
                        const int k = k0 + 16 * (s / 4) + 4 * lk + s % 4;
                        const float v = W[(unsigned)(jc * h + min(k, h - 1))];
                        b[s] = (j < h && k < h) ? v : 0.f;
                    }
#pragma unroll
                    for (int s = 0; s < 16; ++s)
                        if (k0 + 16 * (s / 4) < h)
                            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(g[lr * hs + k0 + 16 * (s / 4) + 4 * lk + s % 4], b[s], acc, 0, 0, 0);
                }
                float* dZo = m.dZ + (long)(l - 1) * n * h;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = 4 * lk + r;
                    const bool in = j < h && r0 + i < n;
                    const float v = (in && act[r] > 0.f) ? acc[r] : 0.f;
                    o[i * hs + j] = v;
                    if (in) dZo[(r0 + i) * h + j] = v;
                }
            }
            __syncthreads();
            float* s = g; g = o; o = s;
        }
    }
}

// h = 32 C for C = 1, 2, 4 (32, 64 and 128, the widths of the cost models; 96 goes the
// general way, for no other reason), and d a multiple of 32: one tile per wave, no masks. Every
// layer waits for the one before, so what counts is the latency of its weights:
// the slices a wave multiplies (hidden layers 1 .. L - 1 forward, then L - 1 .. 1
// backward) are loaded two layers ahead, and what the output layer reads at the
// start. A step of 256 samples through 32 -> 128 (x 3) -> 1 spends 14 us here;
// with each load at its use it took 32 us.
template <int C>
struct mlp_slice {
    float w[8 * C], bias;
};
template <bool BWD, int C>
__device__ __forceinline__ void mlp_load_slice(const mlp_net& m, int q, int j, int lk, mlp_slice<C>& o) {
    constexpr int h = 32 * C;
    if (q < m.L - 1) {
        const float* __restrict__ W = m.P + mlp_w_off(q + 1, m.d, h);
        const unsigned at = (unsigned)(lk * h + j);   // one lane offset for all rows
        o.bias = W[h * h + j];
#pragma unroll
        for (int s = 0; s < 8 * C; ++s) o.w[s] = (W + 4 * s * h)[at];
    } else if (BWD && q < 2 * (m.L - 1)) {
        const float* __restrict__ W = m.P + mlp_w_off(2 * (m.L - 1) - q, m.d, h);
        const unsigned at = (unsigned)(j * h + 4 * lk);
#pragma unroll
        for (int s = 0; s < 2 * C; ++s) {
            const f4v v = *reinterpret_cast<const f4v_any*>(W + 16 * s + at);
            o.w[4 * s] = v.x; o.w[4 * s + 1] = v.y; o.w[4 * s + 2] = v.z; o.w[4 * s + 3] = v.w;
        }
    }
}
template <bool BWD, int C>
__global__ void __launch_bounds__(128 * C) __attribute__((amdgpu_waves_per_eu(1, 2))) mlp_rows32_kernel(mlp_net m) {
    constexpr int h = 32 * C, NT = 128 * C, KS = 8 * C;
    extern __shared__ float mlp_lds[];
    const int n = m.n, L = m.L, hs = m.hs;
    float* cur = mlp_lds;
    float* nxt = mlp_lds + 16 * hs;
    float* dp = mlp_lds + 32 * hs;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
    const long r0 = (long)blockIdx.x * 16;
    const int j = wave * 16 + lr;
    const bool whole = r0 + 16 <= n;
    const float* __restrict__ WL = m.P + mlp_w_off(L, m.d, h);
    float w0[8], a[KS], act[4];
    mlp_slice<C> b, bn, bnn;
    const unsigned at0 = (unsigned)(lk * h + j);
#pragma unroll
    for (int s = 0; s < 8; ++s) w0[s] = (m.P + 4 * s * h)[at0];
    const float bias0 = m.P[m.d * h + j];
    mlp_load_x<NT>(m, r0, cur);
    mlp_load_slice<BWD, C>(m, 0, j, lk, b);
    float wo[KS], yv[4] = {0.f, 0.f, 0.f, 0.f};   // output layer: wave 0
    const float wj = WL[j], biasL = WL[h];
    if (wave == 0) {
#pragma unroll
        for (int s = 0; s < KS; ++s) wo[s] = WL[4 * s + lk];
        if (BWD) {
#pragma unroll
            for (int r = 0; r < 4; ++r) yv[r] = m.y[min(r0 + 4 * lk + r, (long)n - 1)];
        }
    }
    mlp_load_slice<BWD, C>(m, 1, j, lk, bn);
    __syncthreads();
    {   // layer 0: d in steps of 32
        f4v acc = {0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < m.d; k0 += 32) {
            if (k0 > 0) {
#pragma unroll
                for (int s = 0; s < 8; ++s) w0[s] = (m.P + (k0 + 4 * s) * h)[at0];
            }
#pragma unroll
            for (int s = 0; s < 8; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[lr * hs + k0 + 4 * s + lk], w0[s], acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * lk + r;
            const float v = acc[r] + bias0;
            act[r] = v > 0.f ? v : 0.f;
            nxt[i * hs + j] = act[r];
            if (BWD && (whole || r0 + i < n)) m.H[(r0 + i) * h + j] = act[r];
        }
        __syncthreads();
        float* s = cur; cur = nxt; nxt = s;
    }
    for (int l = 1; l < L; ++l) {
#pragma unroll
        for (int s = 0; s < KS; ++s) a[s] = cur[lr * hs + 4 * s + lk];
        mlp_load_slice<BWD, C>(m, l + 1, j, lk, bnn);
        f4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b.w[s], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * lk + r;
            const float v = acc[r] + b.bias;
            act[r] = v > 0.f ? v : 0.f;
            nxt[i * hs + j] = act[r];
            if (BWD && (whole || r0 + i < n)) m.H[((long)l * n + r0 + i) * h + j] = act[r];
        }
        b = bn;
        bn = bnn;
        __syncthreads();
        float* s = cur; cur = nxt; nxt = s;
    }
    if (wave == 0) {   // output layer: one column
        f4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) a[s] = cur[lr * hs + 4 * s + lk];
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], lr == 0 ? wo[s] : 0.f, acc, 0, 0, 0);
        if (lr == 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * lk + r;
                const bool in = whole || r0 + i < n;
                const float p = acc[r] + biasL;
                if (in) m.pred[r0 + i] = p;
                if constexpr (BWD) {
                    const float g = in ? 2.f * (p - yv[r]) / (float)n : 0.f;
                    dp[i] = g;
                    if (in) m.dpred[r0 + i] = g;
                }
            }
        }
    }
    if constexpr (BWD) {
        __syncthreads();
        // each lane holds its activations of the last hidden layer; with several
        // hidden layers its gradients go to the tile that no wave reads any more
        float* g = nxt;
        float* o = cur;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * lk + r;
            const float v = act[r] > 0.f ? dp[i] * wj : 0.f;
            g[i * hs + j] = v;
            if (whole || r0 + i < n) m.dZ[((long)(L - 1) * n + r0 + i) * h + j] = v;
        }
        __syncthreads();
        for (int l = L - 1; l > 0; --l) {
#pragma unroll
            for (int r = 0; r < 4; ++r) act[r] = m.H[((long)(l - 1) * n + min(r0 + 4 * lk + r, (long)n - 1)) * h + j];
#pragma unroll
            for (int s = 0; s < 2 * C; ++s) {
                const f4v v = *reinterpret_cast<const f4v*>(g + lr * hs + 16 * s + 4 * lk);
                a[4 * s] = v.x; a[4 * s + 1] = v.y; a[4 * s + 2] = v.z; a[4 * s + 3] = v.w;
            }
            mlp_load_slice<BWD, C>(m, 2 * (L - 1) - l + 2, j, lk, bnn);
            f4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b.w[s], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * lk + r;
                const bool in = whole || r0 + i < n;
                const float v = (in && act[r] > 0.f) ? acc[r] : 0.f;
                o[i * hs + j] = v;
                if (in) m.dZ[((long)(l - 1) * n + r0 + i) * h + j] = v;
            }
            b = bn;
            bn = bnn;
            __syncthreads();
            float* s = g; g = o; o = s;
        }
    }
}

// ---- gradients of weights and biases ------------------------------------------
// G(i, j) = sum_r A(r, i) D(r, j) for i < in, and G(in, j) = sum_r D(r, j): the
// weight gradient of a layer with input A (n x in) and output gradient D
// (n x out), with the bias gradient as one more row (an input of ones). One
// 16 x 16 tile per workgroup; its four waves take consecutive quarters of the
// samples and are merged in wave order, compensated.
struct mlp_wgrad_layer {
    const float* A;
    const float* D;
    float* G;
    int in, out, tile0;   // first workgroup of the layer
};
constexpr int MLP_MAX_LAYERS = 17;
struct mlp_wgrad_args {
    mlp_wgrad_layer l[MLP_MAX_LAYERS];
    int count;
};

__global__ void __launch_bounds__(256) mlp_wgrad_kernel(int n, mlp_wgrad_args args, int tiles, const float* __restrict__ pred,
                                                        const float* __restrict__ y, float* __restrict__ loss) {
    __shared__ f4v part[4][64];
    if ((int)blockIdx.x == tiles) {   // the loss has a workgroup of its own
        mlp_mse_block(n, pred, y, nullptr, loss);
        return;
    }
    int li = 0;
    while (li + 1 < args.count && (int)blockIdx.x >= args.l[li + 1].tile0) ++li;
    const mlp_wgrad_layer T = args.l[li];
    const int jt = (T.out + 15) / 16, t = (int)blockIdx.x - T.tile0;
    const int i0 = t / jt * 16, j0 = t % jt * 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = i0 + (lane & 15), j = j0 + (lane & 15), lk = lane >> 4;
    const int per = ((n + 3) / 4 + 3) / 4 * 4;   // samples per wave
    const int k1 = min(n, (wave + 1) * per);
    f4v acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = wave * per; k0 < k1; k0 += 64) {
        float a[16], b[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int k = k0 + 4 * s + lk;
            a[s] = (k < k1 && i <= T.in) ? (i < T.in ? T.A[(long)k * T.in + i] : 1.f) : 0.f;
            b[s] = (k < k1 && j < T.out) ? T.D[(long)k * T.out + j] : 0.f;
        }
#pragma unroll
        for (int s = 0; s < 16; ++s)
            if (k0 + 4 * s < k1) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], acc, 0, 0, 0);
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            kf_cs v = kf_cs_init(part[0][lane][r]);
            for (int w = 1; w < 4; ++w) v = kf_cs_add(v, part[w][lane][r]);
            const int gi = i0 + 4 * lk + r;
            if (gi <= T.in && j < T.out) T.G[(long)gi * T.out + j] = kf_cs_value(v);
        }
    }
}

// Adam (Kingma and Ba): m = b1 m + (1 - b1) g; v = b2 v + (1 - b2) g^2;
// p -= lr * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps).
__global__ void mlp_adam_kernel(long n, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                                float* __restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Per-column mean and standard deviation (population, floored at `floor`) of
// an n x d row-major matrix, for the standardisation of features and targets.
// One workgroup per column; thread t adds rows t, t + 256, ... with
// compensated sums, then the 256 pairs are merged by a fixed halving tree.
// Two passes: the mean, then the squared deviations from it.
__device__ __forceinline__ float mlp_block_total(kf_cs v, kf_cs* part) {
    const int t = threadIdx.x;
    part[t] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) part[t] = kf_cs_merge(part[t], part[t + w]);
        __syncthreads();
    }
    const float r = kf_cs_value(part[0]);
    __syncthreads();
    return r;
}

__global__ void __launch_bounds__(256) mlp_col_stats_kernel(long n, int d, const float* __restrict__ X,
                                                            float floor, float* __restrict__ mu,
                                                            float* __restrict__ sd) {
    __shared__ kf_cs part[256];
    const int j = blockIdx.x;
    kf_cs a = kf_cs_init(0.f);
    for (long i = threadIdx.x; i < n; i += 256) a = kf_cs_add(a, X[i * d + j]);
    const float mean = mlp_block_total(a, part) / (float)n;
    kf_cs q = kf_cs_init(0.f);
    for (long i = threadIdx.x; i < n; i += 256) {
        const float e = X[i * d + j] - mean;
        q = kf_cs_add(q, e * e);
    }
    const float var = mlp_block_total(q, part) / (float)n;
    if (threadIdx.x == 0) {
        mu[j] = mean;
        sd[j] = fmaxf(sqrtf(var), floor);
    }
}

// out(r, j) = (X(src, j) - mu(j)) / sd(j) for r < rows, with src = idx[r]
// (a minibatch in shuffled order) or row0 + r when idx is null.
__global__ void mlp_gather_std_kernel(int rows, int d, const float* __restrict__ X, const int* __restrict__ idx,
                                      long row0, const float* __restrict__ mu, const float* __restrict__ sd,
                                      float* __restrict__ out) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long)rows * d) return;
    const int r = (int)(i / d), j = (int)(i % d);
    const long src = idx ? (long)idx[r] : row0 + r;
    out[i] = (X[src * d + j] - mu[j]) / sd[j];
}

// out(i) = p(i) sd + mu: a standardised prediction back to log microseconds.
__global__ void mlp_unstd_kernel(int n, const float* __restrict__ p, const float* __restrict__ mu,
                                 const float* __restrict__ sd, float* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = __builtin_fmaf(p[i], *sd, *mu);
}

hipError_t mlp_col_stats(long n, int d, const float* X, float floor, float* mu, float* sd, hipStream_t st) {
    if (n <= 0 || d <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(mlp_col_stats_kernel, dim3(d), dim3(256), 0, st, n, d, X, floor, mu, sd);
    return hipGetLastError();
}

hipError_t mlp_gather_std(int rows, int d, const float* X, const int* idx, long row0, const float* mu,
                          const float* sd, float* out, hipStream_t st) {
    const long total = (long)rows * d;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(mlp_gather_std_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, rows, d, X,
                       idx, row0, mu, sd, out);
    return hipGetLastError();
}

hipError_t mlp_unstd(int n, const float* p, const float* mu, const float* sd, float* out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(mlp_unstd_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, p, mu, sd, out);
    return hipGetLastError();
}

hipError_t mlp_gemm(int M, int N, int K, const float* A, long sai, long sak, const float* B, long sbk, long sbj,
                    float* C, long ldc, const float* bias, int relu, const float* mask, long ldm, hipStream_t st) {
    if (M <= 0 || N <= 0) return hipSuccess;
    dim3 grid((N + 15) / 16, (M + 15) / 16);
    hipLaunchKernelGGL(mlp_gemm_kernel, grid, dim3(64), 0, st, M, N, K, A, sai, sak, B, sbk, sbj, C, ldc, bias,
                       relu, mask, ldm);
    return hipGetLastError();
}

// Whether a network takes the block kernel: the widths whose two 16-row tiles fit 64
// KiB of LDS, where it is the faster route. A workgroup walks all layers of its 16
// samples, so few samples leave a wide network to few workgroups, whose every layer is
// bound by the latency of its weights; one launch a layer spreads the layer over the
// chip. us of a gradient (of predictions), block against layer by layer, at d = 32:
//  - three layers of 128: n = 16 16 (6.5) against 62 (26), n = 32768 0.25 (0.3) times;
//  - three layers of 480: n = 16 509 (249) against 167 (105), n = 1024 2.2 (1.6) times,
//    n = 4096 0.9 (0.7) times; eight layers n = 4096 0.94 (1.4) times, n = 32768 0.8 both;
//  - three layers of 16, n = 32768: predictions 1.6 times, gradients 0.3 times; and
//    predictions of 480 inputs 1.06 times already at n = 16.
bool mlp_rows_pay(int d, int h, int L, long n, bool grad) {
    if (d > 480 || h > 480) return false;
    if (grad) return h <= 128 || n >= 4096;
    if (h > 128) return n >= (L <= 4 ? 4096 : 16384);
    const bool tiled = d % 32 == 0 && (h == 32 || h == 64 || h == 128);
    return n <= 4096 ? d <= 128 || h >= 32 : h >= 64 || (tiled && d <= 128);
}

hipError_t mlp_rows(int n, int d, int h, int L, const float* P, const float* X, const float* y, float* H, float* dZ,
                    float* pred, float* dpred, hipStream_t st) {
    // row pitch of the LDS tiles: 32 columns a step, plus 4 so that a fragment's
    // 16 rows fall on different banks
    const int hs = ((d > h ? d : h) + 31) / 32 * 32 + 4;
    const size_t lds = (size_t)(32 * hs + 16) * sizeof(float);
    const dim3 grid((unsigned)((n + 15) / 16));
    const mlp_net m = {n, d, h, L, hs, P, X, y, H, dZ, pred, dpred};
    void (*kern)(mlp_net) = y ? mlp_rows_kernel<true> : mlp_rows_kernel<false>;
    int nt = MLP_NT;
    if (d % 32 == 0 && (h == 32 || h == 64 || h == 128)) {
        nt = 4 * h;
        kern = h == 32 ? (y ? mlp_rows32_kernel<true, 1> : mlp_rows32_kernel<false, 1>)
             : h == 64 ? (y ? mlp_rows32_kernel<true, 2> : mlp_rows32_kernel<false, 2>)
                       : (y ? mlp_rows32_kernel<true, 4> : mlp_rows32_kernel<false, 4>);
    }
    hipLaunchKernelGGL(kern, grid, dim3(nt), lds, st, m);
    return hipGetLastError();
}

// Weight and bias gradients of `count` layers, and the loss (pred may be null:
// no loss) in one launch.
hipError_t mlp_wgrad(int n, int count, const float* const* A, const float* const* D, float* const* G, const int* in,
                     const int* out, const float* pred, const float* y, float* loss, hipStream_t st) {
    if (count < 1 || count > MLP_MAX_LAYERS) return hipErrorInvalidValue;
    mlp_wgrad_args args;
    args.count = count;
    int tiles = 0;
    for (int l = 0; l < count; ++l) {
        args.l[l] = {A[l], D[l], G[l], in[l], out[l], tiles};
        tiles += ((in[l] + 1 + 15) / 16) * ((out[l] + 15) / 16);
    }
    hipLaunchKernelGGL(mlp_wgrad_kernel, dim3((unsigned)(tiles + (pred && loss ? 1 : 0))), dim3(256), 0, st, n, args, tiles,
                       pred, y, loss);
    return hipGetLastError();
}

hipError_t mlp_mse(int n, const float* p, const float* y, float* dp, float* loss, hipStream_t st) {
    hipLaunchKernelGGL(mlp_mse_kernel, dim3(1), dim3(256), 0, st, n, p, y, dp, loss);
    return hipGetLastError();
}

hipError_t mlp_adam(long n, float* p, const float* g, float* m, float* v, float lr, float b1, float b2, float eps,
                    float c1, float c2, hipStream_t st) {
    hipLaunchKernelGGL(mlp_adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, p, g, m, v, lr, b1,
                       b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace kf
