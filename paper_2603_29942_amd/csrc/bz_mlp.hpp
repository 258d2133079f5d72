// bz_mlp.hpp -- the work predictor: a 4 -> 64 -> 64 -> 1 multilayer
// perceptron in FP32 with ReLU hidden layers, its forward pass, the gradient
// of the mean squared error and an Adam step, as HIP kernels.
//
// Parameter vector (BZ_MLP_PARAMS floats, row-major weight matrices):
//   W1[64][4], b1[64], W2[64][64], b2[64], w3[64], b3
// The network maps features of a code (field, length, dimension, rank
// deficit of the last information set) to log10 of the combinations the
// method evaluates on it; it only orders work, it never changes a result.
//
// Every sum runs in a fixed order (no atomics), so a training run is
// reproducible bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace bz {

constexpr int MLP_IN = 4, MLP_H = 64;

// The network's inputs for a code: field, length, dimension and the rank
// deficit k - k_m of its last information set, normalised as in training.
__host__ __device__ inline void mlp_features(int p, int n, int k, int deficit, float *f) {
    f[0] = ((float)p - 5.0f) / 2.0f;
    f[1] = ((float)n - 60.0f) / 30.0f;
    f[2] = ((float)k - 25.0f) / 15.0f;
    f[3] = (float)deficit / 8.0f;
}
constexpr int MLP_W1 = 0, MLP_B1 = MLP_W1 + MLP_H * MLP_IN, MLP_W2 = MLP_B1 + MLP_H, MLP_B2 = MLP_W2 + MLP_H * MLP_H,
              MLP_W3 = MLP_B2 + MLP_H, MLP_B3 = MLP_W3 + MLP_H, MLP_NPARAM = MLP_B3 + 1;

// Forward pass: 64 samples per workgroup, one per lane, and 16 units of the
// second layer per wavefront (each wavefront computes the short first layer
// itself).  A wavefront's weights are uniform, so they come through scalar
// loads as operands of the products, without LDS.  The activations meet in
// LDS: the output sums them in the order of the units, and the cache is
// written in whole rows.  The chains of 64 dependent products bound it, which
// is why the units are spread: 8000 samples, one per thread on 32 workgroups,
// took 33 us; 19 us on 125.
// cache (optional): per sample the post-activation h1[64] and h2[64].
constexpr int MLP_FWD_SAMPLES = 64;
__global__ __launch_bounds__(256) void mlp_forward_kernel(const float *__restrict__ prm, const float *__restrict__ x,
                                                          int n, float *__restrict__ y, float *__restrict__ cache) {
    constexpr int LD = 2 * MLP_H + 1;  // odd: the lanes' rows start in different banks
    __shared__ float act[MLP_FWD_SAMPLES * LD];
    const int lane = threadIdx.x & 63;
    const int part = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int s0 = blockIdx.x * MLP_FWD_SAMPLES, s = s0 + lane;
    float in[MLP_IN];
#pragma unroll
    for (int j = 0; j < MLP_IN; j++) in[j] = s < n ? x[(size_t)s * MLP_IN + j] : 0.0f;
    float h1[MLP_H];
#pragma unroll
    for (int i = 0; i < MLP_H; i++) {
        float a = prm[MLP_B1 + i];
#pragma unroll
        for (int j = 0; j < MLP_IN; j++) a = fmaf(prm[MLP_W1 + i * MLP_IN + j], in[j], a);
        h1[i] = fmaxf(a, 0.0f);
        if (cache && i / 16 == part) act[lane * LD + i] = h1[i];
    }
    for (int u = 0; u < MLP_H / 4; u += 4) {
        const float *w = prm + MLP_W2 + (part * (MLP_H / 4) + u) * MLP_H;
        float a[4];
#pragma unroll
        for (int q = 0; q < 4; q++) a[q] = prm[MLP_B2 + part * (MLP_H / 4) + u + q];
#pragma unroll
        for (int j = 0; j < MLP_H; j++)
#pragma unroll
            for (int q = 0; q < 4; q++) a[q] = fmaf(w[q * MLP_H + j], h1[j], a[q]);
#pragma unroll
        for (int q = 0; q < 4; q++) act[lane * LD + MLP_H + part * (MLP_H / 4) + u + q] = fmaxf(a[q], 0.0f);
    }
    __syncthreads();
    if (part == 0 && s < n) {
        float out = prm[MLP_B3];
#pragma unroll 16
        for (int i = 0; i < MLP_H; i++) out = fmaf(prm[MLP_W3 + i], act[lane * LD + MLP_H + i], out);
        y[s] = out;
    }
    if (cache) {
        const int rows = n - s0 < MLP_FWD_SAMPLES ? n - s0 : MLP_FWD_SAMPLES;
        for (int i = threadIdx.x; i < rows * 2 * MLP_H; i += 256)
            cache[(size_t)s0 * 2 * MLP_H + i] = act[(i / (2 * MLP_H)) * LD + i % (2 * MLP_H)];
    }
}

// Gradient of L = mean (y - t)^2 over the samples, in chunks: workgroup c
// takes samples [n c / chunks, n (c + 1) / chunks), 40 at a time.  Their
// activations go to LDS; dL/dy = 2 (y - t) / n and the pre-activation
// gradients of both hidden layers (ReLU passes the gradient where the unit is
// positive) are formed there and never leave it; every parameter's products
// are summed in registers, W2 in 4 x 4 blocks per thread.  The chunk's sums go
// to its row of `part` (the gradient itself when there is one chunk), and
// mlp_sum_kernel adds the rows.  One thread per parameter that ran through all
// samples took 1972 us for 8000 of them, on 18 workgroups waiting for one load
// after the other, and the loss in one thread 453 us; the two kernels now take
// 24 us.  The sums of 40 and of the chunks are also shorter, and no less
// exact, than one of n.
constexpr int MLP_SUB = 40;                    // samples in LDS at a time
constexpr int MLP_NSUM = MLP_NPARAM + 1;       // a row of sums: the gradient and the squared errors
constexpr int MLP_CHUNKS = 256;                // at most: one per compute unit
// chunks for n samples; their rows fit the scratch of n x (2 MLP_H + 1) floats
inline int mlp_chunks(int n) {
    const int c = n / MLP_SUB;
    return c < 1 ? 1 : c > MLP_CHUNKS ? MLP_CHUNKS : c;
}
static_assert(MLP_NSUM <= MLP_SUB * (2 * MLP_H + 1), "a chunk's row of sums fits the scratch of its samples");
__global__ __launch_bounds__(256) void mlp_grad_kernel(const float *__restrict__ prm, const float *__restrict__ x,
                                                       const float *__restrict__ t, int n,
                                                       const float *__restrict__ y, const float *__restrict__ cache,
                                                       float *__restrict__ part, float *__restrict__ grad,
                                                       float *__restrict__ loss) {
    constexpr int LD = MLP_H + 4;  // rows of 16-byte words, shifted by four banks
    __shared__ __align__(16) float w2[MLP_H * LD], h1[MLP_SUB * LD], h2[MLP_SUB * LD], d1[MLP_SUB * LD], d2[MLP_SUB * LD];
    __shared__ float w3[MLP_H], in[MLP_SUB * MLP_IN], dy[MLP_SUB], er[MLP_SUB];
    const int tid = threadIdx.x, chunks = gridDim.x;
    const int first = (int)((long long)n * blockIdx.x / chunks), end = (int)((long long)n * (blockIdx.x + 1) / chunks);
    for (int i = tid; i < MLP_H * MLP_H; i += 256) w2[(i / MLP_H) * LD + i % MLP_H] = prm[MLP_W2 + i];
    if (tid < MLP_H) w3[tid] = prm[MLP_W3 + tid];
    const int a4 = (tid >> 4) * 4, b4 = (tid & 15) * 4;  // the thread's block of W2
    float g2[4][4] = {}, g1 = 0.0f, gb = 0.0f;
    for (int s0 = first; s0 < end; s0 += MLP_SUB) {
        const int ns = end - s0 < MLP_SUB ? end - s0 : MLP_SUB;
        __syncthreads();  // the last round's reads
        for (int i = tid; i < ns * 2 * MLP_H; i += 256) {
            const int s = i / (2 * MLP_H), u = i % (2 * MLP_H);
            const float v = cache[(size_t)s0 * 2 * MLP_H + i];
            if (u < MLP_H) h1[s * LD + u] = v;
            else h2[s * LD + u - MLP_H] = v;
        }
        if (tid < ns * MLP_IN) in[tid] = x[(size_t)s0 * MLP_IN + tid];
        if (tid < ns) {
            const float e = y[s0 + tid] - t[s0 + tid];
            er[tid] = e;
            dy[tid] = 2.0f * e / (float)n;
        }
        __syncthreads();
        for (int i = tid; i < ns * MLP_H; i += 256) {
            const int s = i / MLP_H, u = i % MLP_H;
            d2[s * LD + u] = h2[s * LD + u] > 0.0f ? dy[s] * w3[u] : 0.0f;
        }
        __syncthreads();
        // d1[s][j], four units j of the samples tid / 16 + 16 r per thread
        {
            constexpr int R = (MLP_SUB + 15) / 16;
            float a[R][4] = {};
            const int sr = tid >> 4;
#pragma unroll 2
            for (int i = 0; i < MLP_H; i += 4) {
                float4 w[4], d[R];
#pragma unroll
                for (int q = 0; q < 4; q++) w[q] = *reinterpret_cast<const float4 *>(&w2[(i + q) * LD + b4]);
#pragma unroll
                for (int r = 0; r < R; r++) {
                    const int s = sr + 16 * r < ns ? sr + 16 * r : ns - 1;
                    d[r] = *reinterpret_cast<const float4 *>(&d2[s * LD + i]);
                }
#pragma unroll
                for (int r = 0; r < R; r++) {
                    const float dv[4] = {d[r].x, d[r].y, d[r].z, d[r].w};
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        a[r][0] = fmaf(w[q].x, dv[q], a[r][0]);
                        a[r][1] = fmaf(w[q].y, dv[q], a[r][1]);
                        a[r][2] = fmaf(w[q].z, dv[q], a[r][2]);
                        a[r][3] = fmaf(w[q].w, dv[q], a[r][3]);
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < R; r++) {
                const int s = sr + 16 * r;
                if (s < ns) {
#pragma unroll
                    for (int q = 0; q < 4; q++) d1[s * LD + b4 + q] = h1[s * LD + b4 + q] > 0.0f ? a[r][q] : 0.0f;
                }
            }
        }
        __syncthreads();
        // W2[i][j]: d2_i h1_j
#pragma unroll 2
        for (int s = 0; s < ns; s++) {
            const float4 d = *reinterpret_cast<const float4 *>(&d2[s * LD + a4]);
            const float4 h = *reinterpret_cast<const float4 *>(&h1[s * LD + b4]);
            const float dv[4] = {d.x, d.y, d.z, d.w}, hv[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
            for (int p = 0; p < 4; p++)
#pragma unroll
                for (int q = 0; q < 4; q++) g2[p][q] = fmaf(dv[p], hv[q], g2[p][q]);
        }
        // W1[i][j]: d1_i x_j; one of the vectors per thread of the first four wavefronts
        for (int s = 0; s < ns; s++) g1 = fmaf(d1[s * LD + tid / MLP_IN], in[s * MLP_IN + tid % MLP_IN], g1);
        const int u = tid & 63;
        if (tid < 64) {
            for (int s = 0; s < ns; s++) gb += d1[s * LD + u];
        } else if (tid < 128) {
            for (int s = 0; s < ns; s++) gb += d2[s * LD + u];
        } else if (tid < 192) {
            for (int s = 0; s < ns; s++) gb = fmaf(dy[s], h2[s * LD + u], gb);
        } else if (tid == 192) {
            for (int s = 0; s < ns; s++) gb += dy[s];
        } else if (tid == 193) {
            for (int s = 0; s < ns; s++) gb = fmaf(er[s], er[s], gb);
        }
    }
    static_assert(MLP_H * MLP_IN == 256 && MLP_H == 64, "one W1 parameter and one 4 x 4 block of W2 per thread");
    float *const o = chunks == 1 ? grad : part + (size_t)blockIdx.x * MLP_NSUM;
    o[MLP_W1 + tid] = g1;
#pragma unroll
    for (int p = 0; p < 4; p++)
#pragma unroll
        for (int q = 0; q < 4; q++) o[MLP_W2 + (a4 + p) * MLP_H + b4 + q] = g2[p][q];
    if (tid < 64) o[MLP_B1 + tid] = gb;
    else if (tid < 128) o[MLP_B2 + tid - 64] = gb;
    else if (tid < 192) o[MLP_W3 + tid - 128] = gb;
    else if (tid == 192) o[MLP_B3] = gb;
    else if (tid == 193) {
        if (chunks > 1) o[MLP_NPARAM] = gb;
        else if (loss) *loss = gb / (float)n;
    }
}

// The chunks' sums added up: 64 columns per workgroup, a quarter of the rows
// per wavefront, each in order, then the four in order.
__global__ __launch_bounds__(256) void mlp_sum_kernel(const float *__restrict__ part, int chunks, int n,
                                                      float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ float sums[4][64];
    const int lane = threadIdx.x & 63, seg = threadIdx.x >> 6, q = blockIdx.x * 64 + lane;
    const int lo = chunks * seg / 4, hi = chunks * (seg + 1) / 4;
    float a = 0.0f;
    if (q < MLP_NSUM) {
#pragma unroll 16
        for (int c = lo; c < hi; c++) a += part[(size_t)c * MLP_NSUM + q];
    }
    sums[seg][lane] = a;
    __syncthreads();
    if (seg != 0 || q >= MLP_NSUM) return;
    a = ((sums[0][lane] + sums[1][lane]) + sums[2][lane]) + sums[3][lane];
    if (q < MLP_NPARAM) grad[q] = a;
    else if (loss) *loss = a / (float)n;
}

// Adam (Kingma and Ba) with bias correction; step counts from 1.
__global__ void mlp_adam_kernel(float *__restrict__ prm, const float *__restrict__ grad, float *__restrict__ m,
                                float *__restrict__ v, int step, float lr, float b1, float b2, float eps) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= MLP_NPARAM) return;
    const float g = grad[q];
    const float mq = b1 * m[q] + (1.0f - b1) * g;
    const float vq = b2 * v[q] + (1.0f - b2) * g * g;
    m[q] = mq;
    v[q] = vq;
    const float mh = mq / (1.0f - powf(b1, (float)step));
    const float vh = vq / (1.0f - powf(b2, (float)step));
    prm[q] -= lr * mh / (sqrtf(vh) + eps);
}

}  // namespace bz
