// mlp.hpp -- kernels of the surrogate network: a fully connected
// 5 -> 128 -> 128 -> 128 -> 16 network with tanh hidden activations, FP32.
//
// A call of the network is a chain of small dependent products (128 rows take
// 27 MFLOP forward and backward), so what bounds it is the number of launches
// and the latency of each link, not arithmetic.  One block of eight waves
// therefore takes 16 rows through the whole network: the weights of its
// output columns sit in each wave's registers (loaded once, while the rows are
// normalised), the activations in LDS.  Inference is one launch (six before:
// 27 -> 7 us a call), a training step two: mlp_kernel for the rows' forward
// and backward passes and every block's share of the gradient, adam_kernel
// for the sum of the shares and the update (20 before, 230 -> 22 us a step of
// 128 rows).
//
// Every matrix product runs on the matrix cores: one wave computes a 16x16
// output tile with v_mfma_f32_16x16x4_f32, walking the contraction four at a
// time.  Operand layout of that instruction (per lane l of the wave):
//   A (16x4): A[l % 16][l / 16]   B (4x16): B[l / 16][l % 16]
//   D (16x16): four values, D[4 (l / 16) + r][l % 16], r = 0..3.
// Every sum has a fixed order, so training is bitwise reproducible.
#pragma once

#include "device_common.hpp"

namespace odk {

constexpr int kMlpIn = 5, kMlpHid = 128, kMlpOut = 16, kMlpLayers = 4;
constexpr int kMlpParams = kMlpIn * kMlpHid + kMlpHid + 2 * (kMlpHid * kMlpHid + kMlpHid) +
                           kMlpHid * kMlpOut + kMlpOut;   // 35,856

// Offsets of the layers' weights W_l [in][out] and biases b_l [out] in the
// flat parameter vector.
constexpr int kW1 = 0, kB1 = kW1 + kMlpIn * kMlpHid, kW2 = kB1 + kMlpHid, kB2 = kW2 + kMlpHid * kMlpHid,
              kW3 = kB2 + kMlpHid, kB3 = kW3 + kMlpHid * kMlpHid, kW4 = kB3 + kMlpHid, kB4 = kW4 + kMlpHid * kMlpOut;
static_assert(kB4 + kMlpOut == kMlpParams, "parameter layout");

constexpr int kMlpTile = 16;              // rows per pass of a block
constexpr int kMlpThreads = 512;          // eight waves, one per 16 hidden columns
constexpr int kMlpStride = kMlpHid + 4;   // LDS row stride: a wave's A operands fall into 64 banks
constexpr int kMlpParts = 32;             // most blocks of a training step (gradient shares)

typedef float mlp4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ mlp4 mlp_mfma(float a, float b, mlp4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// A contraction over 128 in two chains: one would wait for the matrix core's
// latency 32 times over.
__device__ __forceinline__ mlp4 mlp_dot(const float* a, const float* b)
{
    mlp4 even = {0.0f, 0.0f, 0.0f, 0.0f}, odd = even;
#pragma unroll
    for (int k = 0; k < 32; k += 2) {
        even = mlp_mfma(a[4 * k], b[k], even);
        odd = mlp_mfma(a[4 * k + 4], b[k + 1], odd);
    }
    return even + odd;
}

// What a block computes for its rows.
struct MlpJob {
    const float* X;      // [n][5]
    const float* T;      // [n][16] standardised targets, or null
    const int* idx;      // rows to take (null: 0 .. n - 1)
    int n;               // rows of the call
    int raw;             // 1: X in raw units, normalised here; 0: already normalised
    const float* norm;   // in_lo[5], in_hi[5], out_mean[16], out_std[16]
    const float* p;      // parameters
    const float* pt;     // the same with W2 .. W4 transposed ([out][in]), for the backward pass
    float* Y;            // [n][16] outputs in target units, or null
    int* inside;         // [n] 1 where every raw input lies in the box, or null
    float* part;         // [blocks][kMlpParams] gradient shares, or null
    float* err;          // [n] squared error per row
};

// Forward pass (and, with TRAIN, the backward pass) of 16-row tiles blockIdx.x,
// blockIdx.x + gridDim.x, ...
template <bool TRAIN>
__global__ __launch_bounds__(kMlpThreads) void mlp_kernel(MlpJob j)
{
    __shared__ float xn[kMlpTile][8];
    __shared__ float h[3][kMlpTile][kMlpStride];
    __shared__ float y[kMlpTile][kMlpOut + 1];
    __shared__ float tt[TRAIN ? kMlpTile : 1][kMlpOut];
    __shared__ float dz[TRAIN ? 3 : 1][TRAIN ? kMlpTile : 1][kMlpStride];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = lane & 15, q = lane >> 4, n0 = 16 * wv;     // operand column / row, contraction quarter, wave's columns
    // lane offsets of the weight loads (the rest of their addresses is uniform)
    unsigned fwd = q * kMlpHid + n0 + c, out = q * kMlpOut + c;
    const float b1 = j.p[kB1 + n0 + c], b2 = j.p[kB2 + n0 + c], b3 = j.p[kB3 + n0 + c], b4 = j.p[kB4 + c];
    // gradient shares: columns n0.. of W1 and W4's rows n0..; rows n0.. of W2 and W3
    const mlp4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    mlp4 g1 = zero, g4 = zero, g2[TRAIN ? 8 : 1], g3[TRAIN ? 8 : 1];
    float gb = 0.0f;      // bias of layer threadIdx.x / 128 + 1 (threads 384..399: layer 4), column threadIdx.x % 128
    if (TRAIN)
#pragma unroll
        for (int t = 0; t < 8; ++t) g2[t] = g3[t] = zero;

    for (int r0 = blockIdx.x * kMlpTile; r0 < j.n; r0 += gridDim.x * kMlpTile) {
        const int rows = min(kMlpTile, j.n - r0);
        __syncthreads();
        // keeps the loads' addresses as one offset each: as loop invariants they would be held in
        // two hundred registers
        asm volatile("" : "+v"(fwd), "+v"(out));
        // weights of this wave's columns, B[k][n] = W[k][n0 + n], asked for while the rows are
        // normalised
        float w1[2], w2[32], w3[32], w4[32];
#pragma unroll
        for (int k = 0; k < 2; ++k) w1[k] = 4 * k + q < kMlpIn ? (j.p + kW1 + 4 * k * kMlpHid)[fwd] : 0.0f;
#pragma unroll
        for (int k = 0; k < 32; ++k) w2[k] = (j.p + kW2 + 4 * k * kMlpHid)[fwd];
#pragma unroll
        for (int k = 0; k < 32; ++k) w3[k] = (j.p + kW3 + 4 * k * kMlpHid)[fwd];
        if (wv == 0)
#pragma unroll
            for (int k = 0; k < 32; ++k) w4[k] = (j.p + kW4 + 4 * k * kMlpOut)[out];
        if (threadIdx.x < kMlpTile) {
            const int t = threadIdx.x, row = t < rows ? (j.idx ? j.idx[r0 + t] : r0 + t) : 0;
            int ok = 1;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                float z = 0.0f;
                if (k < kMlpIn && t < rows) {
                    z = j.X[(long long)row * kMlpIn + k];
                    if (j.raw) {
                        const float lo = j.norm[k], hi = j.norm[kMlpIn + k];
                        z = 2.0f * (z - lo) / (hi - lo) - 1.0f;
                        ok &= (z >= -1.0f && z <= 1.0f) ? 1 : 0;
                    }
                }
                xn[t][k] = z;
            }
            if (j.inside && t < rows) j.inside[r0 + t] = ok;
        }
        if (TRAIN && threadIdx.x >= 256) {
            const int t = (threadIdx.x - 256) >> 4, k = threadIdx.x & 15;
            float v = 0.0f;
            if (t < rows) {
                const int row = j.idx ? j.idx[r0 + t] : r0 + t;
                v = j.T[(long long)row * kMlpOut + k];
            }
            tt[t][k] = v;
        }
        __syncthreads();
        // hidden layers
        mlp4 a = zero;
#pragma unroll
        for (int k = 0; k < 2; ++k) a = mlp_mfma(xn[c][4 * k + q], w1[k], a);
#pragma unroll
        for (int r = 0; r < 4; ++r) h[0][4 * q + r][n0 + c] = tanhf(a[r] + b1);
        __syncthreads();
        a = mlp_dot(&h[0][c][q], w2);
#pragma unroll
        for (int r = 0; r < 4; ++r) h[1][4 * q + r][n0 + c] = tanhf(a[r] + b2);
        __syncthreads();
        a = mlp_dot(&h[1][c][q], w3);
#pragma unroll
        for (int r = 0; r < 4; ++r) h[2][4 * q + r][n0 + c] = tanhf(a[r] + b3);
        __syncthreads();
        // the backward pass's weights, transposed: B[k][n] = W[n0 + n][k]
        float u2[TRAIN ? 32 : 1], u3[TRAIN ? 32 : 1], u4[TRAIN ? 4 : 1];
        if constexpr (TRAIN) {
#pragma unroll
            for (int k = 0; k < 4; ++k) u4[k] = (j.pt + kW4 + 4 * k * kMlpHid)[fwd];
#pragma unroll
            for (int k = 0; k < 32; ++k) u3[k] = (j.pt + kW3 + 4 * k * kMlpHid)[fwd];
#pragma unroll
            for (int k = 0; k < 32; ++k) u2[k] = (j.pt + kW2 + 4 * k * kMlpHid)[fwd];
        }
        if (wv == 0) {
            a = mlp_dot(&h[2][c][q], w4);
            if (TRAIN) {
#pragma unroll
                for (int r = 0; r < 4; ++r) y[4 * q + r][c] = a[r] + b4;
            } else {
                const float mu = j.norm[2 * kMlpIn + c], sd = j.norm[2 * kMlpIn + kMlpOut + c];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (4 * q + r < rows) j.Y[(long long)(r0 + 4 * q + r) * kMlpOut + c] = (a[r] + b4) * sd + mu;
            }
        }
        if constexpr (TRAIN) {
            __syncthreads();
            // squared error per row and its gradient 2 (Y - T) / (n outputs)
            if (threadIdx.x < kMlpTile * kMlpOut) {
                const int t = threadIdx.x >> 4, k = threadIdx.x & 15;
                const float d = y[t][k] - tt[t][k];
                float e = d * d;
#pragma unroll
                for (int m = 8; m >= 1; m >>= 1) e += __shfl_xor(e, m, 16);
                if (k == 0 && t < rows) j.err[r0 + t] = e;
                y[t][k] = t < rows ? 2.0f / (float)(j.n * kMlpOut) * d : 0.0f;
            }
            __syncthreads();
            // layer 4: W4's rows n0.., and dZ3 = (dY W4^T) (1 - H3^2)
            a = zero;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                g4 = mlp_mfma(h[2][4 * k + q][n0 + c], y[4 * k + q][c], g4);
                a = mlp_mfma(y[c][4 * k + q], u4[k], a);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = h[2][4 * q + r][n0 + c];
                dz[2][4 * q + r][n0 + c] = a[r] * (1.0f - v * v);
            }
            __syncthreads();
            // layer 3: W3's rows n0.., and dZ2
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float x = h[1][4 * k + q][n0 + c];
#pragma unroll
                for (int t = 0; t < 8; ++t) g3[t] = mlp_mfma(x, dz[2][4 * k + q][16 * t + c], g3[t]);
            }
            a = mlp_dot(&dz[2][c][q], u3);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = h[1][4 * q + r][n0 + c];
                dz[1][4 * q + r][n0 + c] = a[r] * (1.0f - v * v);
            }
            __syncthreads();
            // layer 2: W2's rows n0.., and dZ1
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float x = h[0][4 * k + q][n0 + c];
#pragma unroll
                for (int t = 0; t < 8; ++t) g2[t] = mlp_mfma(x, dz[1][4 * k + q][16 * t + c], g2[t]);
            }
            a = mlp_dot(&dz[1][c][q], u2);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = h[0][4 * q + r][n0 + c];
                dz[0][4 * q + r][n0 + c] = a[r] * (1.0f - v * v);
            }
            __syncthreads();
            // layer 1: W1's columns n0.. (rows beyond the five inputs stay zero); biases
#pragma unroll
            for (int k = 0; k < 4; ++k) g1 = mlp_mfma(c < 8 ? xn[4 * k + q][c & 7] : 0.0f, dz[0][4 * k + q][n0 + c], g1);
            {
                const int layer = threadIdx.x >> 7, col = threadIdx.x & 127;
                if (layer < 3) {
                    for (int t = 0; t < kMlpTile; ++t) gb += dz[layer][t][col];
                } else if (col < kMlpOut) {
                    for (int t = 0; t < kMlpTile; ++t) gb += y[t][col];
                }
            }
        }
    }
    if constexpr (TRAIN) {
        float* o = j.part + (long long)blockIdx.x * kMlpParams;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 4 * q + r;
            if (m < kMlpIn) o[kW1 + m * kMlpHid + n0 + c] = g1[r];
            o[kW4 + (n0 + m) * kMlpOut + c] = g4[r];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                o[kW2 + (n0 + m) * kMlpHid + 16 * t + c] = g2[t][r];
                o[kW3 + (n0 + m) * kMlpHid + 16 * t + c] = g3[t][r];
            }
        }
        const int layer = threadIdx.x >> 7, col = threadIdx.x & 127;
        if (layer < 3)
            o[(layer == 0 ? kB1 : layer == 1 ? kB2 : kB3) + col] = gb;
        else if (col < kMlpOut)
            o[kB4 + col] = gb;
    }
}

// Place of parameter i in the copy with transposed W2 .. W4.
__device__ __forceinline__ int mlp_transposed(int i)
{
    if (i >= kW2 && i < kB2) return kW2 + ((i - kW2) & 127) * kMlpHid + ((i - kW2) >> 7);
    if (i >= kW3 && i < kB3) return kW3 + ((i - kW3) & 127) * kMlpHid + ((i - kW3) >> 7);
    if (i >= kW4 && i < kB4) return kW4 + ((i - kW4) & 15) * kMlpHid + ((i - kW4) >> 4);
    return i;
}

__global__ __launch_bounds__(256) void mlp_transpose_kernel(const float* __restrict__ p, float* __restrict__ pt)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < kMlpParams) pt[mlp_transposed(i)] = p[i];
}

// Training rows, once per call: inputs to [-1, 1] in the box, targets
// standardised, in place.
__global__ __launch_bounds__(256) void mlp_normalize_kernel(float* __restrict__ X, float* __restrict__ T, long long n,
                                                            const float* __restrict__ norm)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n * kMlpIn) {
        const int k = (int)(i % kMlpIn);
        const float lo = norm[k], hi = norm[kMlpIn + k];
        X[i] = 2.0f * (X[i] - lo) / (hi - lo) - 1.0f;
    }
    if (i < n * kMlpOut) {
        const int k = (int)(i % kMlpOut);
        T[i] = (T[i] - norm[2 * kMlpIn + k]) / norm[2 * kMlpIn + kMlpOut + k];
    }
}

// The gradient (the blocks' shares in block order) and, with ADAM, the update
// of the flat parameter vector (bias-corrected moments).
template <bool ADAM>
__global__ __launch_bounds__(256) void adam_kernel(const float* __restrict__ part, int blocks, float* __restrict__ g,
                                                   float* __restrict__ p, float* __restrict__ pt,
                                                   float* __restrict__ m, float* __restrict__ v, float lr, float b1, float b2, float eps,
                                                   float c1, float c2)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= kMlpParams) return;
    float gi = part[i];
    for (int b = 1; b < blocks; ++b) gi += part[(long long)b * kMlpParams + i];
    if (!ADAM) {
        g[i] = gi;
        return;
    }
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    pt[mlp_transposed(i)] = pi;
}

// Glorot-uniform weights from Philox (key (seed, 0x4d4c50), counter (parameter
// index, 0, 5, 0)), zero biases, zero moments.
__global__ __launch_bounds__(256) void mlp_init_kernel(uint64_t seed, float* __restrict__ p, float* __restrict__ m,
                                                       float* __restrict__ v)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= kMlpParams) return;
    int fan = 0;
    if (i < kB1) fan = kMlpIn + kMlpHid;
    else if ((i >= kW2 && i < kB2) || (i >= kW3 && i < kB3)) fan = 2 * kMlpHid;
    else if (i >= kW4 && i < kB4) fan = kMlpHid + kMlpOut;
    float w = 0.0f;
    if (fan) {
        const double lim = sqrt(6.0 / fan);
        w = (float)((2.0 * unit(philox((uint64_t)i, 0, 5, 0, seed, 0x4d4c50ull).w[0]) - 1.0) * lim);
    }
    p[i] = w;
    m[i] = 0.0f;
    v[i] = 0.0f;
}

}  // namespace odk
