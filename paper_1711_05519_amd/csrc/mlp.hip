// The threshold network of the learned schedule (not part of the paper):
// o = w3 . relu(W2 relu(W1 phi + b1) + b2) + b3 with phi in R^4, 32 hidden
// units per layer; the loop uses it as a multiplicative correction of
// Algorithm 1's threshold, zeta = beta (sigma_{r+1} + gamma^{k+1} sigma_1)
// exp(clip(o, -5, 5)) (the tail of the gather). Parameters are one
// FP32 vector of MLP_PARAMS values: W1 (32 x 4, row-major), b1, W2 (32 x 32),
// b2, w3, b3. These kernels train it: a batched forward pass, the gradient
// of sum_b g_b o_b summed over the batch in a fixed order, and Adam.

#include "launch.hpp"

namespace rpca {
namespace {

constexpr int OFF_W1 = 0, OFF_B1 = MLP_H * MLP_IN, OFF_W2 = OFF_B1 + MLP_H, OFF_B2 = OFF_W2 + MLP_H * MLP_H,
              OFF_W3 = OFF_B2 + MLP_H, OFF_B3 = OFF_W3 + MLP_H;
static_assert(OFF_B3 + 1 == MLP_PARAMS, "parameter layout");

__device__ inline void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One wave per sample, lane j < 32 owns hidden unit j. Its rows of both layers'
// weights are loaded whole before the first use (16-byte loads, element
// aligned), so a sample costs one memory latency.
__global__ __launch_bounds__(WAVE) void k_mlp_forward(const float* __restrict__ th, const float* __restrict__ phi,
                                                     float* __restrict__ o, int B) {
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    const int b = blockIdx.x;
    if (b >= B) return;
    __shared__ float h1[MLP_H];
    const int lane = threadIdx.x, unit = lane & (MLP_H - 1);
    const f4 x = *reinterpret_cast<const f4*>(phi + (size_t)b * MLP_IN);
    const f4 w1 = *reinterpret_cast<const f4*>(th + OFF_W1 + unit * MLP_IN);
    f4 w2[MLP_H / 4];
#pragma unroll
    for (int q = 0; q < MLP_H / 4; ++q) w2[q] = *reinterpret_cast<const f4*>(th + OFF_W2 + unit * MLP_H + 4 * q);
    const float b2 = th[OFF_B2 + unit], w3 = th[OFF_W3 + unit], b3 = th[OFF_B3];
    float v = th[OFF_B1 + unit];
#pragma unroll
    for (int i = 0; i < MLP_IN; ++i) v = fmaf(w1[i], x[i], v);
    if (lane < MLP_H) h1[lane] = fmaxf(v, 0.f);
    wave_fence();
    float c = b2;
#pragma unroll
    for (int i = 0; i < MLP_H; ++i) c = fmaf(w2[i / 4][i % 4], h1[i], c);
    c = lane < MLP_H ? w3 * fmaxf(c, 0.f) : 0.f;
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, WAVE);
    if (lane == 0) o[b] = c + b3;
}

// grad = sum over b (in order) of g_b d o_b / d theta, by one workgroup.
//
// Bound by latency (1249 parameters, a few samples). One wave per sample
// recomputes the activations and both layers' derivatives of MLP_CHUNK samples at
// once, with the second layer's weights in LDS (row pitch 33: rows and columns
// are both read without bank conflicts); then thread t adds the chunk's samples,
// in order, to its second-layer weight t and, the first 225 threads, to one of
// the other parameters. One sample after another with five barriers each took
// 17.6 us for 14 samples; now 5.1 us.
constexpr int MLP_CHUNK = 16;
constexpr int MLP_BWD_THREADS = MLP_CHUNK * WAVE;
static_assert(MLP_BWD_THREADS == MLP_H * MLP_H, "one second-layer weight per thread");

__global__ __launch_bounds__(MLP_BWD_THREADS) void k_mlp_backward(const float* __restrict__ th,
                                                                 const float* __restrict__ phi,
                                                                 const float* __restrict__ g, int B,
                                                                 float* __restrict__ grad) {
    __shared__ float w2[MLP_H][MLP_H + 1];
    __shared__ float ph[MLP_CHUNK][MLP_IN], gs[MLP_CHUNK];
    __shared__ float h1[MLP_CHUNK][MLP_H], h2[MLP_CHUNK][MLP_H], ga1[MLP_CHUNK][MLP_H], ga2[MLP_CHUNK][MLP_H];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int unit = lane & (MLP_H - 1);
    // the wave's layer inputs: loaded once, for every chunk
    float w1[MLP_IN];
#pragma unroll
    for (int i = 0; i < MLP_IN; ++i) w1[i] = th[OFF_W1 + unit * MLP_IN + i];
    const float b1 = th[OFF_B1 + unit], b2 = th[OFF_B2 + unit], w3 = th[OFF_W3 + unit];
    w2[tid / MLP_H][tid % MLP_H] = th[OFF_W2 + tid];
    // the other parameter of this thread: b1, W1, b2, w3, b3 in turn
    const int other = tid < OFF_W2 ? tid : OFF_B2 + (tid - OFF_W2);
    const bool has_other = other < MLP_PARAMS;
    float acc2 = 0.f, acc = 0.f;
    __syncthreads();
    for (int b0 = 0; b0 < B; b0 += MLP_CHUNK) {
        const int b = b0 + wave;
        const int cnt = min(MLP_CHUNK, B - b0);
        if (b < B) {   // the same for the whole wave
            float x[MLP_IN];
#pragma unroll
            for (int i = 0; i < MLP_IN; ++i) x[i] = phi[(size_t)b * MLP_IN + i];
            const float gb = g[b];
            float v1 = b1;
#pragma unroll
            for (int i = 0; i < MLP_IN; ++i) v1 = fmaf(w1[i], x[i], v1);
            if (lane < MLP_H) h1[wave][lane] = fmaxf(v1, 0.f);
            if (lane < MLP_IN) ph[wave][lane] = lane == 0 ? x[0] : lane == 1 ? x[1] : lane == 2 ? x[2] : x[3];
            if (lane == 0) gs[wave] = gb;
            wave_fence();
            float v2 = b2;
#pragma unroll
            for (int i = 0; i < MLP_H; ++i) v2 = fmaf(w2[unit][i], h1[wave][i], v2);
            if (lane < MLP_H) {
                h2[wave][lane] = fmaxf(v2, 0.f);
                ga2[wave][lane] = v2 > 0.f ? gb * w3 : 0.f;   // d / d a2
            }
            wave_fence();
            float d1 = 0.f;
#pragma unroll
            for (int j = 0; j < MLP_H; ++j) d1 = fmaf(w2[j][unit], ga2[wave][j], d1);
            if (lane < MLP_H) ga1[wave][lane] = v1 > 0.f ? d1 : 0.f;   // d / d a1
        }
        __syncthreads();
        for (int s = 0; s < cnt; ++s) {
            acc2 += ga2[s][tid / MLP_H] * h1[s][tid % MLP_H];
            if (has_other) {
                float d;
                if (other < OFF_B1) d = ga1[s][other / MLP_IN] * ph[s][other % MLP_IN];
                else if (other < OFF_W2) d = ga1[s][other - OFF_B1];
                else if (other < OFF_W3) d = ga2[s][other - OFF_B2];
                else if (other < OFF_B3) d = gs[s] * h2[s][other - OFF_W3];
                else d = gs[s];
                acc += d;
            }
        }
        __syncthreads();
    }
    grad[OFF_W2 + tid] = acc2;
    if (has_other) grad[other] = acc;
}

// Adam (Kingma and Ba, Algorithm 1), step t >= 1, elementwise
__global__ __launch_bounds__(256) void k_mlp_adam(float* __restrict__ th, float* __restrict__ m, float* __restrict__ v,
                                                 const float* __restrict__ g, int n, int t, float lr, float b1,
                                                 float b2, float eps) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float mi = b1 * m[i] + (1.f - b1) * g[i];
    const float vi = b2 * v[i] + (1.f - b2) * g[i] * g[i];
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / (1.f - powf(b1, (float)t));
    const float vh = vi / (1.f - powf(b2, (float)t));
    th[i] -= lr * mh / (sqrtf(vh) + eps);
}

}  // namespace

hipError_t launch_mlp_forward(const float* th, const float* phi, float* o, int B, hipStream_t s) {
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_forward, dim3(B), dim3(WAVE), 0, s, th, phi, o, B);
    return hipGetLastError();
}

hipError_t launch_mlp_backward(const float* th, const float* phi, const float* g, int B, float* grad, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_backward, dim3(1), dim3(MLP_BWD_THREADS), 0, s, th, phi, g, B, grad);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float* th, float* m, float* v, const float* g, int t, float lr, float b1, float b2,
                           float eps, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_adam, dim3((MLP_PARAMS + 255) / 256), dim3(256), 0, s, th, m, v, g, MLP_PARAMS, t, lr,
                       b1, b2, eps);
    return hipGetLastError();
}

}  // namespace rpca
